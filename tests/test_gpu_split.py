"""GPU parity: fp32 products on the bf16 matrix pipe, every value in three parts (gemm_split.hip), against the oracle at the contract's
tolerance, against the fp32 kernels' error, and on operands that are no finite numbers or next to the largest one."""
import numpy as np
import pytest

from test_gpu_layer import Case, dev, gcn, run_bwd, run_fwd, tuned          # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


def rows_alone(gcn, dev, rows):
    return Case(gcn, dev, np.zeros(0, np.int32), np.zeros(0, np.int32), rows)          # A^ = I


# Steps of 32 k with and without a tail, W whole in LDS and two steps at a time, each number of column tiles, more columns than one panel,
# columns that end inside a group of four; W as it is and transposed; rows around a tile, a workgroup and a pass over all of them.
@pytest.mark.parametrize("rows", [1, 31, 257, 4099, 70001])
@pytest.mark.parametrize("d_in,d_out", [(1, 5), (33, 65), (64, 128), (100, 173), (602, 41), (200, 300), (129, 192), (256, 256)])
def test_products_in_three_parts(gcn, dev, tuned, rows, d_in, d_out):
    case = rows_alone(gcn, dev, rows)
    tuned("GCN_GEMM_SPLIT", 2)
    run_fwd(gcn, dev, case, d_in, d_out, bias=True, save_ah=True)
    run_fwd(gcn, dev, case, d_in, d_out, act="none", want_z=False)
    run_bwd(gcn, dev, case, d_in, d_out, saved_ah=True, dbias=True)
    run_bwd(gcn, dev, case, d_in, d_out, mask=False)
    case.A.free()


# Every shape of the weight gradient's workgroups; widths around pairs of columns and blocks; rows around a chunk, a split, many splits.
@pytest.mark.parametrize("rows", [1, 15, 33, 2049, 40001])
@pytest.mark.parametrize("d_in,d_out", [(65, 67), (128, 128), (256, 100), (100, 256), (250, 256), (602, 128), (384, 128), (44, 300), (520, 260)])
def test_weight_gradient_in_three_parts(gcn, dev, tuned, rows, d_in, d_out):
    case = rows_alone(gcn, dev, rows)
    tuned("GCN_GEMM_SPLIT", 2)
    run_bwd(gcn, dev, case, d_in, d_out, want_dh=False, saved_ah=True)
    case.A.free()


def error(a, ref):
    return ((a.double() - ref).norm() / ref.norm()).item()


# the 2-norm of the error against 64 bits, of terms of either sign, after a ReLU, and all positive
@pytest.mark.parametrize("kind", ["signed", "relu", "positive"])
@pytest.mark.parametrize("rows,d_in,d_out", [(20000, 128, 200), (20000, 602, 128), (70001, 256, 256), (262144, 100, 130)])
def test_no_less_exact_than_the_fp32_pipe(gcn, dev, tuned, kind, rows, d_in, d_out):
    import torch
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows + d_in)
    X = torch.randn(rows, d_in, generator=gen, device=dev)
    W = torch.randn(d_in, d_out, generator=gen, device=dev)
    G = torch.randn(rows, d_out, generator=gen, device=dev)
    if kind != "signed":
        X.clamp_(min=0)
    if kind == "positive":
        W.abs_(), G.abs_()
    case = rows_alone(gcn, dev, rows)
    err = {}
    for mode in (0, 2):
        tuned("GCN_GEMM_SPLIT", mode)
        out, dW = torch.empty(rows, d_out, device=dev), torch.empty(d_in, d_out, device=dev)
        gcn.gcn_dense_fwd(X, W, out)
        gcn.gcn_layer_bwd(case.A, X, W, G, dW, AH_saved=X)
        err[mode] = (error(out, X.double() @ W.double()), error(dW, X.double().T @ G.double()))
    print(kind, rows, d_in, d_out, err, flush=True)
    assert err[2][0] <= err[0][0] and err[2][1] <= err[0][1]
    case.A.free()


# Rows (for a gradient, columns) of few terms, the others zero.  The six products of a term lack 2^-27 of it as a rule, a quarter of a rounding
# (in the 2-norm sqrt(1 + 1/16) of one: 1.04 with its spread), and a step's sum is rounded before it is added: with two to eight terms one
# rounding more for each but the first, of a part of the sum (at most sqrt(2) of the fp32 pipe's, where all roundings are as large).
@pytest.mark.parametrize("terms,bound", [(1, 1.04), (2, 1.42), (3, 1.42), (8, 1.42), (32, 1.0)])
@pytest.mark.parametrize("d_in,d_out", [(100, 130), (602, 128), (256, 256)])
def test_sums_of_few_terms(gcn, dev, tuned, terms, bound, d_in, d_out):
    import torch
    rows = 8192
    gen = torch.Generator(device=dev)
    gen.manual_seed(terms + d_in)
    X = torch.randn(rows, d_in, generator=gen, device=dev)
    W = torch.randn(d_in, d_out, generator=gen, device=dev)
    G = torch.randn(rows, d_out, generator=gen, device=dev)
    place = torch.rand(rows, d_in, generator=gen, device=dev)
    by_row = torch.where(place.argsort(1).argsort(1) < terms, X, torch.zeros_like(X))
    by_col = torch.where(place.argsort(0).argsort(0) < terms, X, torch.zeros_like(X))
    case = rows_alone(gcn, dev, rows)
    err = {}
    for mode in (0, 2):
        tuned("GCN_GEMM_SPLIT", mode)
        out, dW = torch.empty(rows, d_out, device=dev), torch.empty(d_in, d_out, device=dev)
        gcn.gcn_dense_fwd(by_row, W, out)
        gcn.gcn_layer_bwd(case.A, by_col, W, G, dW, AH_saved=by_col)
        err[mode] = (error(out, by_row.double() @ W.double()), error(dW, by_col.double().T @ G.double()))
    print(terms, d_in, d_out, err, flush=True)
    assert err[2][0] <= bound * err[0][0]
    # (a gradient's terms lie in the parts of different workgroups: few terms each)
    assert err[2][1] <= (1.04 if terms == 1 else 1.42) * err[0][1]
    case.A.free()


# Errors that are small each but of one sign are not small in a sum over rows (what a sparse product forms of H W) or over columns (what the next
# dense product forms): no larger there either than on the fp32 pipe.
@pytest.mark.parametrize("kind", ["signed", "relu", "positive"])
@pytest.mark.parametrize("d_in,d_out", [(48, 130), (100, 173), (602, 128), (256, 256)])
def test_errors_average_out_in_sums(gcn, dev, tuned, kind, d_in, d_out):
    import torch
    rows = 512 * 128
    gen = torch.Generator(device=dev)
    gen.manual_seed(d_in + d_out)
    X = torch.randn(rows, d_in, generator=gen, device=dev)
    W = torch.randn(d_in, d_out, generator=gen, device=dev)
    G = torch.randn(rows, d_out, generator=gen, device=dev)
    if kind != "signed":
        X.clamp_(min=0)
    if kind == "positive":
        W.abs_()
    some = torch.randperm(rows, generator=gen, device=dev)
    sums = {"neighbours": lambda t: t.view(-1, 512, d_out).sum(1), "any rows": lambda t: t[some].view(-1, 512, d_out).sum(1),
            "every fourth": lambda t: t.view(-1, 4, d_out)[:, 0].reshape(-1, 128, d_out).sum(1)}
    case = rows_alone(gcn, dev, rows)
    err = {}
    for mode in (0, 2):
        tuned("GCN_GEMM_SPLIT", mode)
        out, dW = torch.empty(rows, d_out, device=dev), torch.empty(d_in, d_out, device=dev)
        gcn.gcn_dense_fwd(X, W, out)
        gcn.gcn_layer_bwd(case.A, X, W, G, dW, AH_saved=X)
        ref, ref_w = X.double() @ W.double(), X.double().T @ G.double()
        err[mode] = {k: error(f(out.double()), f(ref)) for k, f in sums.items()}
        if kind != "positive":             # (there both have the rounding of the sum over the workgroups' parts, 4e-9, and nothing else)
            err[mode]["gradient's rows"] = error(dW.double().sum(0), ref_w.sum(0))
            err[mode]["gradient's columns"] = error(dW.double().sum(1), ref_w.sum(1))
    print(kind, d_in, d_out, err, flush=True)
    for k in err[0]:
        assert err[2][k] <= err[0][k], k
    case.A.free()


# Values beyond the range of their first part: the rows (for a gradient, the workgroups' ranges of rows) that hold one are multiplied on the fp32
# pipe.  Infinities and NaN come out where 64 bits have them; a product next to the largest number as it is.
@pytest.mark.parametrize("d_in,d_out", [(100, 173), (256, 256), (130, 64)])
def test_infinities_nan_and_the_largest_numbers(gcn, dev, tuned, d_in, d_out):
    import torch
    rows = 3001
    gen = torch.Generator(device=dev)
    gen.manual_seed(d_in)
    X = torch.randn(rows, d_in, generator=gen, device=dev)
    W = torch.randn(d_in, d_out, generator=gen, device=dev) * 0.01
    G = torch.randn(rows, d_out, generator=gen, device=dev) * 0.01
    X[5, 3], X[6, 7], X[2999, d_in - 1], X[3000, 0] = float("inf"), float("-inf"), float("nan"), 3.4e38
    X[40, 2], X[40, 9] = float("inf"), float("-inf")
    tuned("GCN_GEMM_SPLIT", 2)
    out, dW = torch.empty(rows, d_out, device=dev), torch.empty(d_in, d_out, device=dev)
    gcn.gcn_dense_fwd(X, W, out)
    case = rows_alone(gcn, dev, rows)
    gcn.gcn_layer_bwd(case.A, X, W, G, dW, AH_saved=X)
    for got, ref, scale in ((out, X.double() @ W.double(), X.double().abs() @ W.double().abs()),
                            (dW, X.double().T @ G.double(), X.double().abs().T @ G.double().abs())):
        inf, nan = torch.isinf(ref), torch.isnan(ref)
        assert torch.equal(torch.isnan(got), nan)
        assert torch.equal(got[inf].double(), ref[inf])
        ok = ~(inf | nan)
        assert ok.any() and bool(((got.double() - ref).abs()[ok] <= 1e-5 * scale[ok]).all())
    case.A.free()


# Operands (either of the two) so small that a part of theirs would lie below the smallest bf16 number, some of them below the smallest normal fp32
# one: as on the fp32 pipe, to the rounding of numbers of that size.  Beside a large operand their sums are ordinary numbers; 1e-41 has no bf16 part
# at all; 2^-107 is the least with all of its parts.
@pytest.mark.parametrize("small_x,small_w", [(1e-34, 1.0), (1e-36, 1e3), (1e-38, 1.0), (1.0, 1e-37), (1e-20, 1e-17), (2.0**-120, 2.0**40), (2.0**40, 2.0**-120),
                                             (2.0**-137, 2.0**60), (2.0**60, 2.0**-137), (1e-38, 1e12), (1e12, 1e-38), (1e-41, 1e30), (1e30, 1e-41),
                                             (1e-41, 1.0), (1.0, 1e-41), (2.0**-107, 2.0**80), (2.0**80, 2.0**-107), (2.0**-70, 2.0**-70)])
def test_operands_near_the_smallest_number(gcn, dev, tuned, small_x, small_w):
    import torch
    rows, d_in, d_out = 2500, 100, 130
    gen = torch.Generator(device=dev)
    gen.manual_seed(9)
    X = torch.randn(rows, d_in, generator=gen, device=dev) * small_x
    W = torch.randn(d_in, d_out, generator=gen, device=dev) * small_w
    G = torch.randn(rows, d_out, generator=gen, device=dev) * small_w
    tuned("GCN_GEMM_SPLIT", 2)
    out, dW = torch.empty(rows, d_out, device=dev), torch.empty(d_in, d_out, device=dev)
    gcn.gcn_dense_fwd(X, W, out)
    case = rows_alone(gcn, dev, rows)
    gcn.gcn_layer_bwd(case.A, X, W, G, dW, AH_saved=X)
    for got, a, b in ((out, X.double(), W.double()), (dW, X.double().T, G.double())):
        tiny = a.shape[1] * 2.0 ** -149                        # a rounding of each term to a multiple of the smallest number
        assert bool(((got.double() - a @ b).abs() <= 1e-5 * (a.abs() @ b.abs()) + tiny).all())
    case.A.free()


# So many of them that a gradient's workgroups form their whole ranges of rows again (more than 32 chunks of 16 or 32 rows in each).
@pytest.mark.parametrize("d_in,d_out", [(100, 130), (256, 100)])
def test_small_operands_in_every_row(gcn, dev, tuned, d_in, d_out):
    import torch
    rows = 300001
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    X = torch.randn(rows, d_in, generator=gen, device=dev)
    X[:, 5] *= 2.0**-120
    G = torch.randn(rows, d_out, generator=gen, device=dev) * 2.0**40
    case = rows_alone(gcn, dev, rows)
    tuned("GCN_GEMM_SPLIT", 2)
    dW = torch.empty(d_in, d_out, device=dev)
    gcn.gcn_layer_bwd(case.A, X, torch.zeros(d_in, d_out, device=dev), G, dW, AH_saved=X)
    assert bool(((dW.double() - X.double().T @ G.double()).abs() <= 1e-5 * (X.double().abs().T @ G.double().abs())).all())
    case.A.free()


# One such operand among ordinary ones: in every place of the row tiles, steps and passes of H W, and of the chunks and workgroups of A^T B; and in W.
@pytest.mark.parametrize("d_in,d_out", [(100, 130), (602, 65), (256, 256)])
def test_one_small_operand_among_ordinary_ones(gcn, dev, tuned, d_in, d_out):
    import torch
    rows = 70001                                               # more than one pass over them
    gen = torch.Generator(device=dev)
    gen.manual_seed(d_in)
    X = torch.randn(rows, d_in, generator=gen, device=dev)
    W = torch.randn(d_in, d_out, generator=gen, device=dev)
    G = torch.randn(rows, d_out, generator=gen, device=dev)
    at = [(0, 0), (31, d_in - 1), (32, 33), (255, 64), (256, 1), (20000, 31), (65535, 32), (65536, 5), (65541, d_in - 2), (69999, 2), (70000, d_in - 3)]
    for r, k in at + [(17, 40)]:                               # a row and a column for each, empty but for it, and its partner large
        X[r], X[:, k] = 0, 0
    for r, k in at:
        X[r, k] = 1e-40
        W[k] *= 1e32
        G[r] *= 1e32
    W[40, 3], X[17, 40] = 1e-40, 1e32
    tuned("GCN_GEMM_SPLIT", 2)
    out, dW = torch.empty(rows, d_out, device=dev), torch.empty(d_in, d_out, device=dev)
    gcn.gcn_dense_fwd(X, W, out)
    case = rows_alone(gcn, dev, rows)
    gcn.gcn_layer_bwd(case.A, X, W, G, dW, AH_saved=X)
    for got, a, b in ((out, X.double(), W.double()), (dW, X.double().T, G.double())):
        assert bool(((got.double() - a @ b).abs() <= 1e-5 * (a.abs() @ b.abs())).all())
    W[40, 3] = 1.0                                             # (W without one, A with: only the tiles that hold them are formed again)
    gcn.gcn_dense_fwd(X, W, out)
    assert bool(((out.double() - X.double() @ W.double()).abs() <= 1e-5 * (X.double().abs() @ W.double().abs())).all())
    case.A.free()


# The same of G W^T, which a layer hands down (A^ = I: the sparse product changes nothing): K = d_out terms to d_in columns.
def handed_down(gcn, dev, G, W, Zprev=None):
    import torch
    rows, d_in = G.shape[0], W.shape[0]
    case = rows_alone(gcn, dev, rows)
    dH = torch.empty(rows, d_in, device=dev)
    H = torch.zeros(rows, d_in, device=dev)
    gcn.gcn_layer_bwd(case.A, H, W, G, torch.empty_like(W), dH=dH, Zprev=Zprev)
    torch.cuda.synchronize()
    case.A.free()
    return dH


def draw(dev, seed, rows, d_in, d_out, kind="signed"):
    import torch
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    G = torch.randn(rows, d_out, generator=gen, device=dev)
    W = torch.randn(d_in, d_out, generator=gen, device=dev)
    if kind != "signed":
        G.clamp_(min=0)
    if kind == "positive":
        W.abs_()
    return gen, G, W


@pytest.mark.parametrize("kind", ["signed", "relu", "positive"])
@pytest.mark.parametrize("rows,d_in,d_out", [(20000, 200, 128), (20000, 128, 602), (70144, 256, 256), (65536, 130, 48)])
def test_gradient_handed_down_is_no_less_exact(gcn, dev, tuned, kind, rows, d_in, d_out):
    gen, G, W = draw(dev, rows + d_in, rows, d_in, d_out, kind)
    ref, err, summed = G.double() @ W.double().T, {}, {}
    few = rows // 512 * 512
    for mode in (0, 2):
        tuned("GCN_GEMM_SPLIT", mode)
        dH = handed_down(gcn, dev, G, W)
        err[mode] = error(dH, ref)
        summed[mode] = error(dH[:few].double().view(-1, 512, d_in).sum(1), ref[:few].view(-1, 512, d_in).sum(1))
    print(kind, rows, d_in, d_out, err, summed, flush=True)
    assert err[2] <= err[0] and summed[2] <= summed[0]


@pytest.mark.parametrize("terms,bound", [(1, 1.04), (2, 1.42), (3, 1.42), (8, 1.42), (32, 1.0)])
@pytest.mark.parametrize("d_in,d_out", [(130, 100), (128, 602), (256, 256)])
def test_gradient_handed_down_of_few_terms(gcn, dev, tuned, terms, bound, d_in, d_out):
    import torch
    rows = 8193
    gen, G, W = draw(dev, terms + d_in, rows, d_in, d_out)
    G = torch.where(torch.rand(rows, d_out, generator=gen, device=dev).argsort(1).argsort(1) < terms, G, torch.zeros_like(G))
    err = {}
    for mode in (0, 2):
        tuned("GCN_GEMM_SPLIT", mode)
        err[mode] = error(handed_down(gcn, dev, G, W), G.double() @ W.double().T)
    print(terms, d_in, d_out, err, flush=True)
    assert err[2] <= bound * err[0]


@pytest.mark.parametrize("d_in,d_out", [(173, 100), (256, 256), (64, 130), (300, 64)])
@pytest.mark.parametrize("masked", [False, True])
def test_gradient_handed_down_of_infinities_nan_and_the_largest_numbers(gcn, dev, tuned, d_in, d_out, masked):
    import torch
    rows = 9000
    gen, G, W = draw(dev, 7, rows, d_in, d_out)
    G[3, 5], G[40, 0], G[41, d_out - 1], G[rows - 1, 7] = float("inf"), float("-inf"), float("nan"), float("inf")
    G[100] = 0
    G[100, 2], W[:, 2] = 3.4e38, W[:, 2].sign()                # a product next to the largest number; its first part is none
    Z = torch.randn(rows, d_in, generator=gen, device=dev) if masked else None
    ref, scale = G.double() @ W.double().T, G.double().abs() @ W.double().abs().T
    tuned("GCN_GEMM_SPLIT", 2)
    got = handed_down(gcn, dev, G, W, Zprev=Z)
    if masked:
        assert bool((got[Z <= 0] == 0).all())                  # whatever the product was
        got, ref, scale = got[Z > 0], ref[Z > 0], scale[Z > 0]
    inf, nan = torch.isinf(ref), torch.isnan(ref)
    assert inf.any() and nan.any() and torch.equal(torch.isnan(got), nan)
    assert torch.equal(got[inf].double(), ref[inf])
    ok = ~(inf | nan)
    assert bool(((got.double() - ref).abs()[ok] <= 1e-5 * scale[ok]).all())


@pytest.mark.parametrize("small_g,small_w", [(1e-34, 1.0), (1e-38, 1.0), (1.0, 1e-37), (1e-20, 1e-17), (2.0**-120, 2.0**40), (2.0**40, 2.0**-120), (2.0**-137, 2.0**60),
                                             (2.0**60, 2.0**-137), (1e-41, 1e30), (1e30, 1e-41), (2.0**-107, 2.0**80), (2.0**-70, 2.0**-70)])
def test_gradient_handed_down_of_operands_near_the_smallest_number(gcn, dev, tuned, small_g, small_w):
    gen, G, W = draw(dev, 11, 9000, 130, 100)
    G, W = G * small_g, W * small_w
    tuned("GCN_GEMM_SPLIT", 2)
    got, a, b = handed_down(gcn, dev, G, W), G.double(), W.double().T
    tiny = a.shape[1] * 2.0 ** -149
    assert bool(((got.double() - a @ b).abs() <= 1e-5 * (a.abs() @ b.abs()) + tiny).all())


@pytest.mark.parametrize("d_in,d_out", [(130, 100), (65, 602), (256, 256)])
def test_gradient_handed_down_of_one_small_operand_among_ordinary_ones(gcn, dev, tuned, d_in, d_out):
    rows = 70001
    gen, G, W = draw(dev, d_in, rows, d_in, d_out)
    at = [(0, 0), (31, d_out - 1), (32, 33), (255, 64), (256, 1), (20000, 31), (65535, 32), (65536, 5), (65541, d_out - 2), (69999, 2), (70000, d_out - 3)]
    for r, k in at + [(17, 40)]:
        G[r], G[:, k] = 0, 0
    for r, k in at:
        G[r, k] = 1e-40
        W[:, k] *= 1e32
    W[3, 40], G[17, 40] = 1e-40, 1e32
    tuned("GCN_GEMM_SPLIT", 2)
    for last in (1e-40, 1.0):                                  # W with one, and without: then only the tiles that hold them are formed again
        W[3, 40] = last
        a, b = G.double(), W.double().T
        got = handed_down(gcn, dev, G, W).double()
        assert bool(((got - a @ b).abs() <= 1e-5 * (a.abs() @ b.abs())).all())
