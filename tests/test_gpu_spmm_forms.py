"""GPU parity of the request forms of the row-per-wavefront sparse product, and of device memory kept between calls.

Which form runs depends on the width, the pitch and the start address of the rows, on how long the rows are and on the
size of the operand, so the products here go over those: widths at and beside each number of vectors a row can have,
rows that start 4 / 8 / 12 bytes off a 16-byte boundary (bf16: between words as well), rows of 0 to 9 entries and long
ones, 32-bit and 64-bit gather addresses, both forms of short rows.  Padding of the operand holds NaN, padding of the
result must keep what it held.  Tolerance: that of the product itself, 1e-5 (fp32) / 2e-2 (bf16) times sum |terms|.
"""
import threading

import numpy as np
import pytest

import oracle
from test_gpu_spmm import Case
from util import TOL_BF16, TOL_F32, bf16_round, check_bound, hub_graph, say, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gcn():
    import paper_2212_05009_amd as g
    return g


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available()
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def short(gcn, dev):
    rng = np.random.default_rng(31)
    n, m = 5003, 9000                                 # 1 to about 10 entries a row, the diagonal included
    u = rng.integers(0, n, m); v = rng.integers(0, n, m)
    return Case(gcn, dev, np.r_[u, v], np.r_[v, u], n)


@pytest.fixture(scope="module")
def hubs(gcn, dev):
    src, dst = hub_graph(5003, 2, 30.0, seed=7)       # rows of 5003 and 2501 entries beside rows of about 30
    return Case(gcn, dev, src, dst, 5003)


@pytest.fixture(scope="module")
def directed(gcn, dev):
    rng = np.random.default_rng(37)
    n, m = 4001, 30000                                # columns with no entry: empty rows of the transpose
    src = rng.integers(0, n, m); dst = rng.integers(0, n // 2, m)
    whole = oracle.graph_build(src, dst, n)
    return Case(gcn, dev, src, dst, n, 500, 2500, deg_global=whole.deg)


def product(gcn, dev, case, d, bf16, transpose, off, pad):
    """Rows of X and Y at element offset `off` in rows of d + pad elements."""
    import torch
    og, A = case.og, case.A
    rng = np.random.default_rng(100 * d + 10 * off + pad)
    n_in, n_out = (og.nr, og.nc) if transpose else (og.nc, og.nr)
    X = rng.standard_normal((n_in, d)).astype(np.float32)
    if bf16:
        X = bf16_round(X)
    ptr, idx, val = (og.colptr, og.rowidx, og.val_t) if transpose else (og.rowptr, og.col, og.val)
    ref, bound = oracle.spmm(ptr, idx, val, X)
    tdt = torch.bfloat16 if bf16 else torch.float32
    Xf = torch.full((n_in * (d + pad) + off,), float("nan"), dtype=tdt, device=dev)
    Yf = torch.full((n_out * (d + pad) + off,), float("nan"), dtype=tdt, device=dev)
    Xd = Xf[off:].view(n_in, d + pad)[:, :d]
    Yd = Yf[off:].view(n_out, d + pad)[:, :d]
    Xd.copy_(to_dev(X, dev, bf16))
    say(f"spmm form rows={n_out} nnz={og.nnz} d={d} bf16={bf16} t={transpose} off={off} pad={pad}")
    (gcn.gcn_spmm_t if transpose else gcn.gcn_spmm)(A, Xd, Yd)
    torch.cuda.synchronize()
    check_bound(to_np(Yd), ref, bound, TOL_BF16 if bf16 else TOL_F32, what=f"form d={d} off={off} pad={pad}")
    assert bool(torch.isnan(Yf[:off].float()).all())
    if pad:
        assert bool(torch.isnan(Yf[off:].view(n_out, d + pad)[:, d:].float()).all()), "wrote outside the d columns"
    return Yd.clone()


# widths with 1, 2, 3, 4, 5, 8, 9, 15, 16, 17, 33 and 65 vectors, whole and ragged
WIDTHS = [3, 4, 5, 7, 8, 9, 13, 17, 18, 33, 36, 50, 61, 64, 66, 81, 131, 258]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", WIDTHS)
def test_forms_widths_and_offsets(gcn, dev, short, hubs, directed, d, bf16):
    for off, pad in [(0, 0), (1, 0), (2, 1), (3, 3), (0, 2), (4, 6)]:
        product(gcn, dev, short, d, bf16, False, off, pad)
    for case, transpose in [(hubs, False), (directed, False), (directed, True)]:
        product(gcn, dev, case, d, bf16, transpose, 0, 0)
        product(gcn, dev, case, d, bf16, transpose, 2, 1)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d", [5, 34, 50, 68, 128])
def test_forms_agree_with_the_general_path(gcn, dev, short, hubs, d, bf16):
    """64-bit addresses change no association, so results are the same bits; short-row groups do, so the bound holds."""
    import torch
    for case in (short, hubs):
        a = product(gcn, dev, case, d, bf16, False, 0, 0)
        for name, value, same in [("GCN_SPMM_WIDE", 1, True), ("GCN_SPMM_SHORT", 0, False), ("GCN_SPMM_SHORT", 1, False)]:
            gcn.gcn_debug_set_tuning(name, value)
            try:
                b = product(gcn, dev, case, d, bf16, False, 0, 0)
            finally:
                gcn.gcn_debug_set_tuning(name, None)
            assert not same or torch.equal(a, b), (name, value)


@pytest.mark.parametrize("bf16", [False, True])
def test_infinities_stay_in_the_rows_that_hold_them(gcn, dev, short, bf16):
    """A lane without an entry adds zero times zero: an infinity of one row reaches its neighbours' rows alone."""
    import torch
    og = short.og
    tdt = torch.bfloat16 if bf16 else torch.float32
    for d in (3, 17, 50, 64):
        X = torch.ones(og.nc, d, dtype=tdt, device=dev)
        X[[0, og.nc // 2, og.nc - 1]] = float("inf")
        Y = torch.empty(og.nr, d, dtype=tdt, device=dev)
        gcn.gcn_spmm(short.A, X, Y)
        torch.cuda.synchronize()
        hit = np.zeros(og.nr, bool)
        rows = np.repeat(np.arange(og.nr), np.diff(og.rowptr))
        hit[rows[np.isin(og.col, [0, og.nc // 2, og.nc - 1])]] = True
        got = Y.float().cpu().numpy()
        assert np.isposinf(got[hit]).all() and np.isfinite(got[~hit]).all()


@pytest.mark.parametrize("rows,k,n", [(1, 3, 5), (63, 64, 16), (65, 17, 33), (700, 64, 16), (4097, 128, 128), (520, 602, 41),
                                      (16385, 64, 16), (33001, 50, 7), (50001, 128, 41)])
@pytest.mark.parametrize("bf16", [False, True])
def test_dw_of_few_rows_against_fp64(gcn, dev, rows, k, n, bf16):
    """A^T G over few rows, whose split depends on the size of the output; an edgeless graph makes A the identity."""
    import torch
    A = gcn.gcn_csr_build(torch.zeros(1, dtype=torch.int32, device=dev), torch.zeros(1, dtype=torch.int32, device=dev), rows)
    rng = np.random.default_rng(rows + k)
    H = rng.standard_normal((rows, k)).astype(np.float32); G = rng.standard_normal((rows, n)).astype(np.float32)
    W = rng.standard_normal((k, n)).astype(np.float32)
    if bf16:
        H, G = bf16_round(H), bf16_round(G)
    dW = torch.empty(k, n, device=dev)
    dH = torch.empty(rows, k, dtype=torch.bfloat16 if bf16 else torch.float32, device=dev)
    say(f"dW rows={rows} {k}x{n} bf16={bf16}")
    gcn.gcn_layer_bwd(A, to_dev(H, dev, bf16), to_dev(W, dev), to_dev(G, dev, bf16), dW, dH=dH)
    torch.cuda.synchronize()
    tol = TOL_BF16 if bf16 else TOL_F32
    H64, G64, W64 = H.astype(np.float64), G.astype(np.float64), W.astype(np.float64)
    check_bound(dW.cpu().numpy(), H64.T @ G64, np.abs(H64).T @ np.abs(G64), tol, what="dW")
    check_bound(to_np(dH), G64 @ W64.T, np.abs(G64) @ np.abs(W64).T, tol, what="dH = G W^T")
    A.free()


@pytest.mark.parametrize("bf16", [False, True])
def test_dw_is_summed_over_no_more_parts_than_it_needs(gcn, dev, bf16):
    """Parts of less than 512 rows only as far as they give every compute unit a workgroup: each part is written and read."""
    import torch
    tdt = torch.bfloat16 if bf16 else torch.float32
    for rows in (4096, 60_000, 130_000):
        A = gcn.gcn_csr_build(torch.zeros(1, dtype=torch.int32, device=dev), torch.zeros(1, dtype=torch.int32, device=dev), rows)
        for k, n in [(64, 16), (50, 7), (50, 50), (128, 41)]:
            AH, G, W = torch.ones(rows, k, dtype=tdt, device=dev), torch.ones(rows, n, dtype=tdt, device=dev), torch.ones(k, n, device=dev)
            dW = torch.empty(k, n, device=dev)
            say(f"parts of dW rows={rows} {k}x{n} bf16={bf16}")
            gcn.gcn_profile_enable(True)
            gcn.gcn_layer_bwd(A, AH, W, G, dW, AH_saved=AH)
            gcn.gcn_profile_enable(False)
            parts = [r["inner"] for r in gcn.gcn_profile_records()[0] if r["kind"] == "gemm_tn_sum"]
            assert len(parts) == 1 and 8 < parts[0] <= 256, (rows, k, n, parts)
            assert bool((dW == rows).all())
        A.free()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("k,n", [(3, 5), (4, 4), (5, 16), (6, 7), (7, 33), (18, 50), (50, 50), (50, 7), (63, 64), (66, 17), (127, 130), (128, 41)])
def test_dense_rows_that_start_on_any_word(gcn, dev, k, n, bf16):
    """H W with rows of every alignment on both sides: the last request of a row of H ends with the row (NaN follows), the
    last columns of a row of the result leave what follows as it was."""
    import torch
    rng = np.random.default_rng(10 * k + n)
    rows = 1003
    X = rng.standard_normal((rows, k)).astype(np.float32)
    if bf16:
        X = bf16_round(X)
    W = rng.standard_normal((k, n)).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float32)
    X64, W64 = X.astype(np.float64), W.astype(np.float64)
    ref, bound = X64 @ W64 + bias, np.abs(X64) @ np.abs(W64) + np.abs(bias)
    tdt = torch.bfloat16 if bf16 else torch.float32
    # the last three: result rows on 16 bytes, with a whole request of room behind column n and without, beside operands of
    # either kind
    for off, px, py in [(0, 0, 0), (1, 0, 0), (2, 2, 2), (0, 3, 3), (1, 1, 1), (0, 0, -n % 8 + 8), (0, -k % 8, -n % 8), (0, -k % 8, -n % 4)]:
        Xf = torch.full((rows * (k + px) + off,), float("nan"), dtype=tdt, device=dev)
        Yf = torch.full((rows * (n + py) + off,), float("nan"), dtype=tdt, device=dev)
        Xd = Xf[off:].view(rows, k + px)[:, :k]
        Yd = Yf[off:].view(rows, n + py)[:, :n]
        Xd.copy_(to_dev(X, dev, bf16))
        say(f"dense rows {k}x{n} bf16={bf16} off={off} pads={px},{py}")
        gcn.gcn_dense_fwd(Xd, to_dev(W, dev), Yd, bias=to_dev(bias, dev))
        torch.cuda.synchronize()
        check_bound(to_np(Yd), ref, bound, TOL_BF16 if bf16 else TOL_F32, what=f"dense {k}x{n} off={off} pads={px},{py}")
        assert bool(torch.isnan(Yf[:off].float()).all())
        assert bool(torch.isnan(Yf[off:].view(rows, n + py)[:, n:].float()).all()), "wrote outside the n columns"


# ---- device memory kept between calls ------------------------------------------------------------------------------

def test_builds_in_reused_memory_give_the_same_arrays(gcn, dev):
    """Large and small graphs in turn, so that arrays land in blocks that held others; each against the oracle."""
    import torch
    graphs = []
    for n, m, seed in [(3000, 40000, 1), (64, 100, 2), (20000, 150000, 3), (2900, 41000, 4), (1, 1, 5)]:
        rng = np.random.default_rng(seed)
        src = rng.integers(0, n, m).astype(np.int32); dst = rng.integers(0, n, m).astype(np.int32)
        graphs.append((n, src, dst, oracle.graph_build(src, dst, n)))
    for _ in range(3):
        for n, src, dst, og in graphs:
            say(f"build in reused memory n={n} m={len(src)}")
            A = gcn.gcn_csr_build(to_dev(src, dev), to_dev(dst, dev), n)
            X = torch.randn(n, 20, device=dev); Y = torch.empty_like(X)
            gcn.gcn_spmm(A, X, Y)                    # still running when the handle is freed
            arr = {k: v.cpu().numpy() for k, v in A.arrays().items() if v is not None}
            A.free()
            for name in ["rowptr", "col", "deg", "colptr", "rowidx"]:
                assert np.array_equal(arr[name], getattr(og, name)), name
            for name in ["val", "val_t"]:
                assert np.array_equal(arr[name].view(np.int32), getattr(og, name).view(np.int32)), name
            ref, bound = oracle.spmm(og.rowptr, og.col, og.val, X.cpu().numpy())
            check_bound(Y.cpu().numpy(), ref, bound, TOL_F32, what="product in reused memory")


def test_threads_and_streams_share_kept_memory(gcn, dev):
    """Four threads build, multiply and free on streams of their own; every product against one made alone."""
    import torch
    rng = np.random.default_rng(3)
    work, errors = [], []
    for t in range(4):
        n, m = 2000 + 700 * t, 30000
        src = to_dev(rng.integers(0, n, m).astype(np.int32), dev); dst = to_dev(rng.integers(0, n, m).astype(np.int32), dev)
        X = torch.randn(n, 33, device=dev); want = torch.empty_like(X)
        A = gcn.gcn_csr_build(src, dst, n)
        gcn.gcn_spmm(A, X, want)
        A.free()
        work.append((n, src, dst, X, want))
    torch.cuda.synchronize()

    def loop(t):
        try:
            n, src, dst, X, want = work[t]
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(8):
                    A = gcn.gcn_csr_build(src, dst, n)
                    Y = torch.empty_like(X)
                    gcn.gcn_spmm(A, X, Y)
                    A.free()
                    assert torch.equal(Y, want)
        except BaseException as e:            # noqa: BLE001 (reported by the main thread)
            errors.append((t, repr(e)))

    say("four threads build and free")
    threads = [threading.Thread(target=loop, args=(t,)) for t in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert not errors, errors
