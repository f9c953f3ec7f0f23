"""GPU parity: gcn_csr_induced (Sec. 4.3.3: a mini-batch is an induced subgraph treated as a graph of its own)
and mini-batch training steps on a directed graph against the oracle.

Structure arrays and values must be bit-identical to the oracle's build of the relabelled edge list
(integer work; values are one fp32 product of two correctly rounded factors on both sides).  The
sampler is the tests' own (uniform distinct vertices, seeded): the paper does not fix one.
"""
import numpy as np
import pytest

import oracle
from util import hub_graph, say

pytestmark = pytest.mark.gpu
NAMES = ["rowptr", "col", "deg", "colptr", "rowidx"]


@pytest.fixture(scope="module")
def gcn():
    import paper_2212_05009_amd as g
    return g


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available()
    return torch.device("cuda:0")


def dev_i32(a, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(dev)


def check_induced(gcn, dev, A, src, dst, n, V):
    og = oracle.graph_build(*oracle.induced_edges(src, dst, n, V), len(V))
    say(f"csr_induced n={n} n_sub={len(V)} nnz_sub={og.nnz}")
    B = gcn.gcn_csr_induced(A, dev_i32(V, dev))
    assert (B.nr, B.nh, B.nnz) == (og.nr, 0, og.nnz)
    arr = B.arrays()
    for name in NAMES:
        assert np.array_equal(arr[name].cpu().numpy(), getattr(og, name)), name
    for name in ["val", "val_t"]:
        assert np.array_equal(arr[name].cpu().numpy().view(np.int32), getattr(og, name).view(np.int32)), name
    return og, B


def check_selected(A, V, total, kept, og):
    """The case is the one meant: entries of the selected rows in the parent, and those off the diagonal that stay."""
    rowptr = A.arrays()["rowptr"].cpu().numpy()
    assert int((rowptr[V + 1] - rowptr[V]).sum()) == total
    assert og.nnz - len(V) == kept


@pytest.mark.parametrize("total", [2047, 2048, 2049, 4096, 6145])
@pytest.mark.parametrize("kept", ["none", "all"])
def test_induced_at_the_edges_of_its_blocks(gcn, dev, total, kept):
    """A whole number of blocks of 2048 selected entries and beside it: in rows of one entry (as many rows as a block can hold),
    and in k rows of k entries that are all kept, the first and the last of every block among them.  (Rows of falling
    ids: a row's diagonal is neither the first entry of the first row nor the last of the others.)"""
    n = 9200
    k = 0 if kept == "none" else int(total ** 0.5)
    ids = 3000 + np.arange(k)
    src, dst = np.repeat(ids, k), np.tile(ids, k)
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    V = np.r_[ids[::-1][:k // 2], np.r_[np.arange(3000), np.arange(4000, n)][:total - k * k], ids[::-1][k // 2:]]
    og, B = check_induced(gcn, dev, A, src, dst, n, V)
    check_selected(A, V, total, k * (k - 1), og)
    B.free()
    A.free()


@pytest.mark.parametrize("length", [2047, 2048, 2049, 4096, 4097])
@pytest.mark.parametrize("before", [0, 1, 2047])
def test_induced_keeps_the_ends_of_its_blocks(gcn, dev, length, before):
    """One row of several blocks, behind `before` rows of one entry: only the first and the last entry of every block of 2048 that
    lies in it are kept, and the row's ends."""
    n, hub = 12000, 4000
    cols = hub - length // 3 + np.arange(length)          # its entries, the diagonal among them
    ends = [s for s in range(length) if s in (0, length - 1) or (before + s) % 2048 in (0, 2047)]
    ends = [s for s in ends if cols[s] != hub]
    src, dst = np.full(length, hub), cols
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    V = np.r_[9000 + np.arange(before), hub, cols[ends]]
    og, B = check_induced(gcn, dev, A, src, dst, n, V)
    check_selected(A, V, before + length + len(ends), len(ends), og)
    assert len(ends) >= 2
    B.free()
    A.free()


@pytest.mark.parametrize("n,m,k,directed,seed", [
    (64, 300, 1, True, 1), (500, 4000, 37, True, 2), (5000, 60000, 1000, False, 3), (30000, 400000, 30000, True, 4),
    (30000, 400000, 4096, False, 5), (100000, 2000000, 25000, True, 6)])
def test_induced_matches_oracle(gcn, dev, n, m, k, directed, seed):
    rng = np.random.default_rng(seed)
    u = rng.integers(0, n, m); v = rng.integers(0, n, m)
    src, dst = (u, v) if directed else (np.r_[u, v], np.r_[v, u])
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    V = rng.permutation(n)[:k]
    check_induced(gcn, dev, A, src, dst, n, V)
    check_induced(gcn, dev, A, src, dst, n, np.sort(V))


def test_induced_with_hub_rows(gcn, dev):
    src, dst = hub_graph(9000, 3, 6.0, seed=21)
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), 9000)
    rng = np.random.default_rng(2)
    V = np.unique(np.r_[[0, 1, 2], rng.permutation(9000)[:6000]])
    og, _ = check_induced(gcn, dev, A, src, dst, 9000, V)
    assert og.deg.max() > 2048


def test_induced_argument_errors(gcn, dev):
    import torch
    rng = np.random.default_rng(3)
    n = 200
    src, dst = rng.integers(0, n, 900), rng.integers(0, n, 900)
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    for bad in ([3, 7, 3], [0, 200], [-1, 5], []):
        with pytest.raises(gcn.GcnError):
            gcn.gcn_csr_induced(A, dev_i32(np.array(bad, np.int32), dev))
    with pytest.raises(gcn.GcnError):
        gcn.gcn_csr_induced(A, dev_i32(np.arange(n + 1) % n, dev))
    blk = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n, 20, 90, deg_global=A.arrays()["deg"])
    with pytest.raises(gcn.GcnError):
        gcn.gcn_csr_induced(blk, dev_i32([1, 2], dev))
    torch.cuda.synchronize()


def test_minibatch_training_on_a_directed_graph(gcn, dev):
    """Three mini-batches of a directed graph (A^^T != A^): subgraph build, feature and label rows fetched
    through the vertex list, forward, loss, backward through the column-major copy, update - losses and final
    weights against the oracle's loop run on its own subgraphs."""
    import torch
    rng = np.random.default_rng(11)
    n, m, dims, lr = 6000, 50000, [24, 16, 5], 0.5
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    X = rng.standard_normal((n, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[2], n).astype(np.int32)
    W0 = [(rng.standard_normal((dims[k], dims[k + 1])) / np.sqrt(dims[k])).astype(np.float32) for k in range(2)]
    batches = [rng.permutation(n)[:1500] for _ in range(3)]

    Wo, want = [w.copy() for w in W0], []
    for V in batches:
        og = oracle.graph_build(*oracle.induced_edges(src, dst, n, V), len(V))
        assert not np.array_equal(og.col, og.rowidx)              # the batch graph really is asymmetric
        losses, Wo = oracle.train(og, X[V], Wo, y[V], lr, 1)
        want.append(losses[0])

    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    Xd = torch.from_numpy(X).to(dev)
    yd = torch.from_numpy(y.view(np.float32).reshape(n, 1).copy()).to(dev)       # labels ride the row gather as 4-byte rows
    Ws = [torch.from_numpy(w.copy()).to(dev) for w in W0]
    dWs = [torch.empty_like(w) for w in Ws]
    loss = torch.zeros(1, device=dev)
    got = []
    for V in batches:
        k = len(V)
        Vd = dev_i32(V, dev)
        say(f"mini-batch of {k} vertices")
        B = gcn.gcn_csr_induced(A, Vd)
        Xb = torch.empty(k, dims[0], device=dev); yb = torch.empty(k, 1, device=dev)
        gcn.gcn_halo_gather(Xd, Vd, Xb)
        gcn.gcn_halo_gather(yd, Vd, yb)
        H1 = torch.empty(k, dims[1], device=dev); Z2 = torch.empty(k, dims[2], device=dev)
        G2 = torch.empty_like(Z2); G1 = torch.empty_like(H1)
        gcn.gcn_layer_fwd(B, Xb, Ws[0], H1, act=gcn.ACT_RELU)
        gcn.gcn_layer_fwd(B, H1, Ws[1], Z2, act=gcn.ACT_NONE)
        gcn.gcn_softmax_xent(Z2, yb.view(torch.int32).reshape(k), 1.0 / k, loss, G2)
        got.append(float(loss.item()))
        gcn.gcn_layer_bwd(B, H1, Ws[1], G2, dWs[1], dH=G1, Zprev=H1)
        gcn.gcn_layer_bwd(B, Xb, Ws[0], G1, dWs[0])
        for W, dW in zip(Ws, dWs):
            gcn.gcn_sgd_update(W, dW, lr)
        torch.cuda.synchronize()
        B.free()
    for e, (a, b) in enumerate(zip(got, want)):
        assert abs(a - b) <= 1e-5 * (1 + e) * abs(b), (e, a, b)
    for W, Wref in zip(Ws, Wo):
        assert np.max(np.abs(W.cpu().numpy() - Wref)) <= 1e-4


@pytest.mark.parametrize("n_sub_all", [False, True])
def test_induced_rows_of_every_length(gcn, dev, n_sub_all):
    """Parent rows and what is kept of them at the bounds of the ways they are taken: 64 entries (16 lanes / a wavefront), 1024 (one piece /
    several), 256 kept (ranked / marked in a bitmap); rows and columns of different lengths."""
    lens = [0, 1, 62, 63, 64, 254, 255, 256, 257, 1022, 1023, 1024, 2048, 5000]
    n = 12000
    rng = np.random.default_rng(11)
    rows = rng.permutation(n)[:6 * len(lens)]
    src = np.concatenate([np.full(k, r) for r, k in zip(rows, 6 * lens)])
    dst = np.concatenate([rng.permutation(n)[:k] for r, k in zip(rows, 6 * lens)])
    back = rng.random(len(src)) < 0.5                                                  # half of them as columns
    src, dst = np.where(back, dst, src), np.where(back, src, dst)
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    V = rng.permutation(n) if n_sub_all else np.concatenate([rows, np.setdiff1d(rng.permutation(n)[:3000], rows)])
    check_induced(gcn, dev, A, src, dst, n, V)


@pytest.mark.parametrize("n_sub", [1, 15, 31, 32768, 32769, 70000])
def test_induced_around_the_sizes_of_its_blocks(gcn, dev, n_sub):
    """One block and less, and both sides of the line from which offsets are scanned and blocks are larger."""
    n = 80000
    rng = np.random.default_rng(n_sub)
    src, dst = rng.integers(0, n, 400000), rng.integers(0, n, 400000)
    hub = rng.integers(0, n, 30000)
    src, dst = np.r_[src, hub, np.full(20000, 5)], np.r_[dst, np.full(30000, 7), hub[:20000]]
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    check_induced(gcn, dev, A, src, dst, n, rng.permutation(n)[:n_sub])


@pytest.mark.parametrize("parent_csc,csc", [(False, True), (False, False), (True, False)])
def test_induced_with_and_without_column_major_arrays(gcn, dev, parent_csc, csc):
    """A parent without them has its subgraphs sorted; a subgraph without them has its rows alone."""
    n = 9000
    rng = np.random.default_rng(5)
    src, dst = rng.integers(0, n, 90000), rng.integers(0, n, 90000)
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n, flags=gcn.BUILD_CSC if parent_csc else 0)
    V = rng.permutation(n)[:4000]
    og = oracle.graph_build(*oracle.induced_edges(src, dst, n, V), len(V))
    arr = gcn.gcn_csr_induced(A, dev_i32(V, dev), flags=gcn.BUILD_CSC if csc else 0).arrays()
    for name in NAMES if csc else NAMES[:3]:
        assert np.array_equal(arr[name].cpu().numpy(), getattr(og, name)), name
    assert np.array_equal(arr["val"].cpu().numpy().view(np.int32), og.val.view(np.int32))


def sparse_parent_with_long_rows(n, degree, long_rows, length, seed):
    rng = np.random.default_rng(seed)
    m = n * degree // 2
    src, dst = rng.integers(0, n, m), rng.integers(0, n, m)
    hubs = rng.permutation(n)[:long_rows]
    src = np.r_[src, np.repeat(hubs, length)]
    dst = np.r_[dst, rng.integers(0, n, long_rows * length)]
    return src.astype(np.int32), dst.astype(np.int32), hubs, rng


@pytest.mark.parametrize("n_sub", [1 << 17, (1 << 17) + 1, 600_000, (1 << 20) + 1])
def test_induced_with_large_bitmaps(gcn, dev, n_sub):
    """Long rows whose bitmaps stand two and one in a block's LDS, take more than 64 KB of it, and no longer fit (subgraphs by keys)."""
    n = max(200_000, n_sub + 5)
    src, dst, hubs, rng = sparse_parent_with_long_rows(n, 4, 40, 3000, n_sub)
    A = gcn.gcn_csr_build(dev_i32(src, dev), dev_i32(dst, dev), n)
    V = np.concatenate([hubs, np.setdiff1d(rng.permutation(n)[:n_sub], hubs)])[:n_sub]
    V = np.concatenate([V, np.setdiff1d(np.arange(n), V)[:n_sub - len(V)]])
    _, B = check_induced(gcn, dev, A, src, dst, n, rng.permutation(V))
    B.free()
    A.free()


@pytest.mark.parametrize("n,n_sub,long_rows", [(150_000, 1 << 17, 300), (150_000, 1 << 17, 1200), (150_000, (1 << 17) + 1, 300), (150_000, (1 << 17) + 1, 1200),
                                               ((1 << 20) + 1, 1 << 16, 3000), ((1 << 20) + 1, (1 << 16) + 1, 3000)])
def test_induced_of_parents_with_many_long_rows(gcn, dev, n, n_sub, long_rows):
    """Both sides of the line between the two ways: subgraphs of more than 2^17 vertices (2^16 of parents of more than 2^20) of a parent whose long rows
    (512 entries and more, rows and columns counted) are fewer or more than one in 200."""
    src, dst, hubs, rng = sparse_parent_with_long_rows(n, 4, long_rows, 700, long_rows)
    A = gcn.gcn_csr_build(dev_i32(np.r_[src, dst], dev), dev_i32(np.r_[dst, src], dev), n)
    V = rng.permutation(n)[:n_sub]
    _, B = check_induced(gcn, dev, A, np.r_[src, dst], np.r_[dst, src], n, V)
    B.free()
    A.free()


@pytest.mark.parametrize("rows,length", [(1, 98304), (1, 98400), (1, 196500), (1, 196700), (1, 300000), (33, 6000)])
@pytest.mark.parametrize("n_sub", [500, 20000, 40000])
@pytest.mark.parametrize("csc", [True, False])
def test_induced_with_more_entries_than_a_block_takes(gcn, dev, rows, length, n_sub, csc):
    """Rows (for an edge list turned round: columns) of more than 96 pieces of 1024 entries (and one for every 1024 vertices) among the 32 that a block has,
    alone and several in a row, at the line and beyond it, and at that of giant rows (192 pieces); a vertex out of range and one listed twice (or 5000 times) are refused there as elsewhere."""
    n = 400_000
    rng = np.random.default_rng(rows + length)
    long = rng.permutation(n)[:rows]
    src = np.r_[rng.integers(0, n, 800_000), np.repeat(long, length)].astype(np.int32)
    dst = np.r_[rng.integers(0, n, 800_000), np.concatenate([rng.permutation(n)[:length] for _ in long])].astype(np.int32)
    V = np.concatenate([np.setdiff1d(rng.permutation(n)[:n_sub], long)[:100], long])
    V = np.concatenate([V, np.setdiff1d(rng.permutation(n), V)[:n_sub - len(V)]])
    for s, d in ((src, dst), (dst, src)):
        A = gcn.gcn_csr_build(dev_i32(s, dev), dev_i32(d, dev), n)
        og = oracle.graph_build(*oracle.induced_edges(s, d, n, V), len(V))
        B = gcn.gcn_csr_induced(A, dev_i32(V, dev), flags=gcn.BUILD_CSC if csc else 0)
        arr = B.arrays()
        for name in NAMES if csc else NAMES[:3]:
            assert np.array_equal(arr[name].cpu().numpy(), getattr(og, name)), name
        assert np.array_equal(arr["val"].cpu().numpy().view(np.int32), og.val.view(np.int32))
        B.free()
        for bad, what in ((np.r_[V[:-1], n], "outside"), (np.r_[V[:-1], V[0]], "twice"), (np.r_[V[:-1], np.full(5000, long[0])], "twice")):
            with pytest.raises(Exception, match=what):
                gcn.gcn_csr_induced(A, dev_i32(bad, dev))
        A.free()
