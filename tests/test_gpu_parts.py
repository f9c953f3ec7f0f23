"""GPU parity: the sparse product in two steps (owned columns first, halo columns second) and the dense
half of a layer, against the oracle.

Sec. 4.1 writes a processor's product as A_mm H_m + sum_n A_mn H_nm; the first term needs no remote
rows.  The expected values come from the oracle's plain product applied to the stored entries
whose local column is below nr (first step) and to all entries (both steps).  Same tolerance
as the one-step product: |gpu - oracle| <= 1e-5 * sum |terms| in fp32, 2e-2 * the same sum for
bf16 features.
"""
import numpy as np
import pytest

import oracle
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


def build_both(gcn, dev, src, dst, n, lo, hi, deg_global=None):
    import torch
    og = oracle.graph_build(src, dst, n, lo, hi, deg_global=deg_global)
    dg = None if deg_global is None else torch.from_numpy(np.ascontiguousarray(deg_global, np.int32)).to(dev)
    A = gcn.gcn_csr_build(torch.from_numpy(np.ascontiguousarray(src, np.int32)).to(dev),
                          torch.from_numpy(np.ascontiguousarray(dst, np.int32)).to(dev), n, lo, hi, deg_global=dg)
    return og, A


@pytest.fixture(scope="module")
def block(gcn, dev):
    rng = np.random.default_rng(23)
    n, m = 7000, 120000
    src = rng.integers(0, n, m); dst = rng.integers(0, n, m)
    whole = oracle.graph_build(np.r_[src, dst], np.r_[dst, src], n)
    return build_both(gcn, dev, np.r_[src, dst], np.r_[dst, src], n, 2000, 4777, deg_global=whole.deg)


@pytest.fixture(scope="module")
def hub_block(gcn, dev):
    src, dst = hub_graph(9000, 3, 6.0, seed=11)      # the hubs are vertices 0..2: rows of several thousand entries
    whole = oracle.graph_build(src, dst, 9000)
    return build_both(gcn, dev, src, dst, 9000, 0, 3000, deg_global=whole.deg)


@pytest.fixture(scope="module")
def whole_graph(gcn, dev):
    rng = np.random.default_rng(29)
    n, m = 3000, 30000
    src = rng.integers(0, n, m); dst = rng.integers(0, n, m)
    return build_both(gcn, dev, src, dst, n, 0, n)


def owned_entries(og):
    """CSR arrays of the entries whose local column is an owned row (column < nr)."""
    keep = og.col < og.nr
    rows = np.repeat(np.arange(og.nr), np.diff(og.rowptr))
    ptr = np.zeros(og.nr + 1, np.int64)
    np.add.at(ptr, rows[keep] + 1, 1)
    return np.cumsum(ptr), og.col[keep], og.val[keep]


def run_parts(gcn, dev, og, A, d, bf16=False, epilogue="none", bias=False, pad=0, seed=0):
    import torch
    rng = np.random.default_rng(500 + seed + d)
    X = rng.standard_normal((og.nc, d)).astype(np.float32)
    if bf16:
        X = bf16_round(X)
    tol = TOL_BF16 if bf16 else TOL_F32
    tdt = torch.bfloat16 if bf16 else torch.float32
    lptr, lcol, lval = owned_entries(og)
    ref_l, bound_l = oracle.spmm(lptr, lcol, lval, X)
    ref, bound = oracle.spmm(og.rowptr, og.col, og.val, X)
    b = None
    if bias:
        b = rng.standard_normal(d).astype(np.float32)
        ref = ref + b.astype(np.float64); bound = bound + np.abs(b.astype(np.float64))
    Zp = None
    if epilogue == "relu":
        ref = np.maximum(ref, 0.0)
    elif epilogue == "mask":
        Zp = rng.standard_normal((og.nr, d)).astype(np.float32)
        if bf16:
            Zp = bf16_round(Zp)
        ref = ref.copy(); ref[~(Zp > 0)] = 0.0
    # bf16: the first step rounds its sums to bf16 before the second adds to them; 2^-9 |local sum| is
    # well inside 2e-2 * bound

    Xfull = torch.zeros(og.nc, d + pad, dtype=tdt, device=dev)
    Xfull[:, :d] = to_dev(X, dev, bf16)
    Xd = Xfull[:, :d]
    # during the first step the halo rows hold NaN: a single read of them would poison the sums
    Xl = Xfull.clone()
    Xl[og.nr:] = float("nan")
    Yfull = torch.full((og.nr, d + pad), float("nan"), dtype=tdt, device=dev)
    Yd = Yfull[:, :d]
    say(f"spmm_part rows={og.nr} halo={og.nh} nnz={og.nnz} d={d} bf16={bf16} epi={epilogue} bias={bias} pad={pad}")
    gcn.gcn_spmm_part(A, gcn.PART_LOCAL, Xl[:, :d], Yd)
    torch.cuda.synchronize()
    check_bound(to_np(Yd), ref_l, bound_l, tol, what=f"local part d={d}")
    code = {"none": gcn.EPI_NONE, "relu": gcn.EPI_RELU, "mask": gcn.EPI_MASK}[epilogue]
    gcn.gcn_spmm_part(A, gcn.PART_HALO, Xd, Yd, epilogue=code, bias=None if b is None else to_dev(b, dev),
                      Zprev=None if Zp is None else to_dev(Zp, dev, bf16))
    torch.cuda.synchronize()
    check_bound(to_np(Yd), ref, bound, tol, what=f"both parts d={d}")
    if pad:
        assert bool(torch.isnan(Yfull[:, d:].float()).all()), "wrote outside the d columns"


@pytest.mark.parametrize("d", [1, 3, 16, 41, 64, 100, 128, 130, 256, 602])
def test_parts_widths_fp32(gcn, dev, block, d):
    og, A = block
    assert og.nh > 0 and 0 < (og.col < og.nr).sum() < og.nnz
    run_parts(gcn, dev, og, A, d)


@pytest.mark.parametrize("d", [7, 41, 64, 128, 256])
def test_parts_widths_bf16(gcn, dev, block, d):
    og, A = block
    run_parts(gcn, dev, og, A, d, bf16=True)


@pytest.mark.parametrize("epilogue", ["relu", "mask"])
@pytest.mark.parametrize("bf16", [False, True])
def test_parts_epilogues(gcn, dev, block, epilogue, bf16):
    og, A = block
    run_parts(gcn, dev, og, A, 48, bf16=bf16, epilogue=epilogue)
    run_parts(gcn, dev, og, A, 128, bf16=bf16, epilogue=epilogue, bias=True)


@pytest.mark.parametrize("d,pad", [(16, 1), (41, 3), (128, 4)])
def test_parts_padded_leading_dimension(gcn, dev, block, d, pad):
    og, A = block
    run_parts(gcn, dev, og, A, d, pad=pad)


@pytest.mark.parametrize("d", [1, 47, 128])
def test_parts_hub_rows(gcn, dev, hub_block, d):
    og, A = hub_block
    assert og.deg.max() > 2048 and og.nh > 0
    run_parts(gcn, dev, og, A, d, epilogue="relu", bias=True)
    run_parts(gcn, dev, og, A, d, bf16=True)


@pytest.mark.parametrize("d", [16, 100])
def test_parts_without_halo(gcn, dev, whole_graph, d):
    """No halo columns: the first step is the whole product, the second only applies bias and epilogue."""
    og, A = whole_graph
    assert og.nh == 0
    run_parts(gcn, dev, og, A, d, epilogue="relu", bias=True)


def test_parts_argument_errors(gcn, dev, block):
    import torch
    og, A = block
    X = torch.zeros(og.nc, 8, device=dev); Y = torch.zeros(og.nr, 8, device=dev)
    with pytest.raises(gcn.GcnError):
        gcn.gcn_spmm_part(A, 0, X, Y)
    with pytest.raises(gcn.GcnError):
        gcn.gcn_spmm_part(A, 3, X, Y)
    with pytest.raises(gcn.GcnError):
        gcn.gcn_spmm_part(A, gcn.PART_LOCAL, X, Y, epilogue=gcn.EPI_RELU)
    with pytest.raises(gcn.GcnError):
        gcn.gcn_spmm_part(A, gcn.PART_LOCAL, X, Y, bias=torch.zeros(8, device=dev))
    with pytest.raises(gcn.GcnError):
        gcn.gcn_spmm_part(A, gcn.PART_HALO, X, Y, epilogue=gcn.EPI_MASK)
    with pytest.raises(TypeError):
        gcn.gcn_spmm_part(A, gcn.PART_HALO, X[:-1], Y)


# Rows that start on 16 bytes whatever their width: the streaming kernels, whose copy of W and last group of columns have edges
# of their own (fewer than 4 columns, a cut last block of W in either direction, 256 columns, K no whole number of steps).
@pytest.mark.parametrize("d_in,d_out", [(16, 1), (32, 2), (64, 3), (1, 4), (3, 5), (5, 17), (20, 33), (100, 130), (128, 47), (33, 255), (256, 129)])
@pytest.mark.parametrize("bf16", [False, True])
def test_dense_fwd_of_pitched_rows(gcn, dev, d_in, d_out, bf16):
    import torch
    rows = 8 * 16 * 512 + 16 * 3 + 5                      # more tiles than wavefronts, the last of them cut
    rng = np.random.default_rng(100 * d_in + d_out)
    X = rng.standard_normal((rows, d_in)).astype(np.float32)
    if bf16:
        X = bf16_round(X)
    W = (rng.standard_normal((d_in, d_out)) / np.sqrt(d_in)).astype(np.float32)
    b = rng.standard_normal(d_out).astype(np.float32)
    ref, bound = oracle.gemm("nn", X, W)
    ref = ref + b.astype(np.float64); bound = bound + np.abs(b.astype(np.float64))
    tdt = torch.bfloat16 if bf16 else torch.float32
    up = lambda d: (d + 7) // 8 * 8 + 8
    Xd = torch.full((rows, up(d_in)), float("nan"), dtype=tdt, device=dev); Xd[:, :d_in] = to_dev(X, dev, bf16)
    Wd = torch.full((d_in + 1, d_out), float("nan"), device=dev); Wd[:d_in] = to_dev(W, dev)
    Out = torch.full((rows + 1, up(d_out)), 7.0, dtype=tdt, device=dev)
    say(f"dense_fwd of pitched rows d_in={d_in} d_out={d_out} bf16={bf16}")
    gcn.gcn_dense_fwd(Xd[:, :d_in], Wd[:d_in], Out[:rows, :d_out], bias=to_dev(b, dev), act=gcn.ACT_RELU)
    torch.cuda.synchronize()
    check_bound(to_np(Out[:rows, :d_out]), np.maximum(ref, 0.0), bound, TOL_BF16 if bf16 else TOL_F32, what="dense_fwd Out")
    assert (Out[rows] == 7).all() and (Out[:, d_out:] == 7).all()


@pytest.mark.parametrize("rows,d_in,d_out", [(1, 5, 3), (777, 41, 16), (5000, 128, 128), (3001, 602, 47), (4097, 16, 41)])
@pytest.mark.parametrize("bf16", [False, True])
def test_dense_fwd(gcn, dev, rows, d_in, d_out, bf16):
    import torch
    rng = np.random.default_rng(rows + d_in)
    X = rng.standard_normal((rows, d_in)).astype(np.float32)
    if bf16:
        X = bf16_round(X)
    W = (rng.standard_normal((d_in, d_out)) / np.sqrt(d_in)).astype(np.float32)
    b = rng.standard_normal(d_out).astype(np.float32)
    ref, bound = oracle.gemm("nn", X, W)
    ref = ref + b.astype(np.float64); bound = bound + np.abs(b.astype(np.float64))
    tdt = torch.bfloat16 if bf16 else torch.float32
    Out = torch.full((rows, d_out), float("nan"), dtype=tdt, device=dev)
    Z = torch.full((rows, d_out), float("nan"), dtype=tdt, device=dev)
    say(f"dense_fwd rows={rows} d_in={d_in} d_out={d_out} bf16={bf16}")
    gcn.gcn_dense_fwd(to_dev(X, dev, bf16), to_dev(W, dev), Out, bias=to_dev(b, dev), act=gcn.ACT_RELU, Z=Z)
    torch.cuda.synchronize()
    tol = TOL_BF16 if bf16 else TOL_F32
    check_bound(to_np(Z), ref, bound, tol, what="dense_fwd Z")
    check_bound(to_np(Out), np.maximum(ref, 0.0), bound, tol, what="dense_fwd Out")
    assert gcn.gcn_dense_fwd(torch.zeros(0, d_in, dtype=tdt, device=dev), to_dev(W, dev),
                             torch.zeros(0, d_out, dtype=tdt, device=dev)) is not None
