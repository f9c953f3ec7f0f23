"""GPU parity: gcn_partition_stats against the oracle's net-by-net count (Sec. 4.3.2 column-net model, Sec. 5
communication metrics).  Integer work: every figure must be equal."""
import os

import numpy as np
import pytest

import oracle
from util import say

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")
KEYS = ("load", "send_rows", "recv_rows", "send_msgs", "recv_msgs")


@pytest.fixture(scope="module")
def gcn():
    import paper_2212_05009_amd as g
    return g


@pytest.fixture(scope="module")
def dev():
    import torch
    assert torch.cuda.is_available()
    return torch.device("cuda:0")


def both(gcn, dev, src, dst, n, part, p):
    import torch
    og = oracle.graph_build(src, dst, n)
    A = gcn.gcn_csr_build(torch.from_numpy(np.ascontiguousarray(src, np.int32)).to(dev),
                          torch.from_numpy(np.ascontiguousarray(dst, np.int32)).to(dev), n, 0, n)
    want = oracle.partition_stats(og.colptr, og.rowidx, og.rowptr, part, p)
    say(f"partition_stats n={n} nnz={og.nnz} p={p}")
    got = gcn.gcn_partition_stats(A, torch.from_numpy(np.ascontiguousarray(part, np.int32)).to(dev), p)
    torch.cuda.synchronize()
    for k in KEYS:
        assert got[k].cpu().numpy().tolist() == want[k].tolist(), k
    assert got["totals"].cpu().numpy().tolist() == [want["volume"], want["cut_entries"]]
    return og, A, want


def test_paper_example(gcn, dev):
    facts = {}
    for line in open(os.path.join(GOLDEN, "halo_example.txt")):
        if line.strip() and not line.startswith("#"):
            k, *rest = line.split()
            facts[k] = rest
    e = np.array([[int(x) for x in q.split("-")] for q in facts["edges"]]) - 1
    src = np.concatenate([e[:, 0], e[:, 1]]); dst = np.concatenate([e[:, 1], e[:, 0]])
    part = np.zeros(6, int)
    for m, q in enumerate(facts["parts"]):
        part[[int(x) - 1 for x in q.split(",")]] = m
    _, _, want = both(gcn, dev, src, dst, 6, part, 3)
    assert want["recv_rows"][2] == 3 and want["send_rows"][1] == int(facts["transfers_row4"][0])


@pytest.mark.parametrize("n,m,p,directed,seed", [
    (50, 200, 1, False, 1), (500, 3000, 2, True, 2), (5000, 60000, 7, True, 3), (20000, 300000, 64, False, 4),
    (20000, 150000, 1000, True, 5), (3000, 20000, 3000, False, 6), (70000, 900000, 16, True, 7)])
def test_random_partitions(gcn, dev, n, m, p, directed, seed):
    rng = np.random.default_rng(seed)
    u = rng.integers(0, n, m); v = (u + rng.geometric(0.01, m)) % n if seed % 2 else rng.integers(0, n, m)
    src, dst = (u, v) if directed else (np.r_[u, v], np.r_[v, u])
    part = rng.integers(0, max(1, p - p // 8), n)               # the last eighth of the parts stays empty
    if p == n:
        part = rng.permutation(n)                               # every vertex its own part
    both(gcn, dev, src, dst, n, part, p)


def test_contiguous_parts_match_block_builds(gcn, dev):
    """The rows a contiguous part receives are the halo list of its block build, bit for bit in size."""
    import torch
    rng = np.random.default_rng(9)
    n, m = 30000, 400000
    u = rng.integers(0, n, m); v = (u + rng.geometric(0.002, m)) % n
    src, dst = np.r_[u, v], np.r_[v, u]
    cuts = [0, 5000, 5001, 17000, 30000]
    part = np.zeros(n, int)
    for k in range(4):
        part[cuts[k]:cuts[k + 1]] = k
    og, A, want = both(gcn, dev, src, dst, n, part, 4)
    sd, dd = torch.from_numpy(src.astype(np.int32)).to(dev), torch.from_numpy(dst.astype(np.int32)).to(dev)
    dg = torch.from_numpy(og.deg).to(dev)
    for k in range(4):
        B = gcn.gcn_csr_build(sd, dd, n, cuts[k], cuts[k + 1], deg_global=dg)
        assert (B.nh, B.nnz) == (int(want["recv_rows"][k]), int(want["load"][k]))


def test_config2_random_and_contiguous_partitions(gcn, dev):
    """The bench graph (R-MAT, 2^18 vertices), 8 parts: a random partition against contiguous ranges."""
    from workloads import configs
    w = configs.get("c2_rmat18")
    n = w["n"]
    rng = np.random.default_rng(1)
    _, _, rnd = both(gcn, dev, w["src"], w["dst"], n, rng.integers(0, 8, n), 8)
    assert rnd["volume"] <= rnd["cut_entries"] and rnd["send_rows"].sum() == rnd["recv_rows"].sum() == rnd["volume"]
    assert rnd["send_msgs"].tolist() == [7] * 8


def test_argument_errors(gcn, dev):
    import torch
    rng = np.random.default_rng(2)
    n = 100
    src = torch.from_numpy(rng.integers(0, n, 400).astype(np.int32)).to(dev)
    dst = torch.from_numpy(rng.integers(0, n, 400).astype(np.int32)).to(dev)
    A = gcn.gcn_csr_build(src, dst, n, 0, n)
    part = torch.zeros(n, dtype=torch.int32, device=dev)
    with pytest.raises(gcn.GcnError):
        gcn.gcn_partition_stats(A, part, 0)
    part[17] = 3
    with pytest.raises(gcn.GcnError):
        gcn.gcn_partition_stats(A, part, 3)                     # part id 3 with p = 3
    part[17] = -1
    with pytest.raises(gcn.GcnError):
        gcn.gcn_partition_stats(A, part, 3)
    with pytest.raises(TypeError):
        gcn.gcn_partition_stats(A, part[:-1], 3)
    whole_deg = A.arrays()["deg"]
    B = gcn.gcn_csr_build(src, dst, n, 10, 60, deg_global=whole_deg)
    with pytest.raises(gcn.GcnError):
        gcn.gcn_partition_stats(B, torch.zeros(50, dtype=torch.int32, device=dev), 2)


@pytest.mark.parametrize("p", [1, 2, 31, 32, 33, 64, 511, 1025, 4096, 4097])
@pytest.mark.parametrize("directed", [False, True])
def test_counting_by_columns_equals_sorting(gcn, dev, p, directed):
    """Columns of 1 to 9000 entries (chunks of long columns included), part counts at the edges of a bitmap word and of
    the form itself; against the oracle, against the sort, and against a handle without column-major arrays."""
    import torch
    from util import hub_graph
    rng = np.random.default_rng(p)
    n = 9001
    src, dst = hub_graph(n, 3, 9.0, seed=11)
    if directed:
        keep = rng.random(src.size) < 0.7
        src, dst = src[keep], dst[keep]
    part = rng.integers(0, p, n)
    og, A, want = both(gcn, dev, src, dst, n, part, p)
    assert np.diff(og.colptr).max() > 2048
    part_d = torch.from_numpy(part.astype(np.int32)).to(dev)
    gcn.gcn_debug_set_tuning("GCN_PARTITION_SORT", 1)
    try:
        by_sort = gcn.gcn_partition_stats(A, part_d, p)
    finally:
        gcn.gcn_debug_set_tuning("GCN_PARTITION_SORT", None)
    rows_only = gcn.gcn_csr_build(torch.from_numpy(src.astype(np.int32)).to(dev), torch.from_numpy(dst.astype(np.int32)).to(dev), n, flags=0)
    for other in (gcn.gcn_partition_stats(A, part_d, p), gcn.gcn_partition_stats(rows_only, part_d, p)):
        for k in by_sort:
            assert torch.equal(by_sort[k], other[k]), k


# Columns whose lengths lie at the bounds of the ways they are counted in (4 lanes, 16, a wavefront with one and more batches, chunks of hub
# columns), every neighbour in another part and all of them in few; part counts around whole words and where the pair table leaves LDS.
@pytest.mark.parametrize("p", [1, 31, 33, 512, 513, 4096])
def test_columns_of_every_length_class(gcn, dev, p):
    lens = [0, 1, 2, 3, 4, 7, 11, 14, 15, 16, 47, 61, 62, 63, 64, 127, 255, 511, 512, 513, 1023, 1024, 2046, 2047, 2048, 3071, 5000]
    n = 8000
    rng = np.random.default_rng(p)
    cols = rng.permutation(n)[:3 * len(lens)]
    src = np.concatenate([rng.permutation(n)[:k] for c, k in zip(cols, 3 * lens)])
    dst = np.concatenate([np.full(k, c) for c, k in zip(cols, 3 * lens)])
    for part in (rng.integers(0, p, n), np.minimum(rng.integers(0, 3, n), p - 1), np.arange(n) % p):
        both(gcn, dev, src, dst, n, part, p)


def test_a_part_out_of_range_is_refused_wherever_it_is(gcn, dev):
    import torch
    n, p = 3000, 40
    rng = np.random.default_rng(3)
    src, dst = rng.integers(0, n, 9000), rng.integers(0, n, 9000)
    src, dst = np.r_[src, np.arange(n)], np.r_[dst, np.full(n, 7)]                     # vertex 7: a hub column
    A = gcn.gcn_csr_build(torch.from_numpy(src.astype(np.int32)).to(dev), torch.from_numpy(dst.astype(np.int32)).to(dev), n, 0, n)
    for at, bad in ((0, -1), (7, p), (n - 1, 2**31 - 1), (1234, -2**31)):
        part = rng.integers(0, p, n)
        part[at] = bad
        with pytest.raises(Exception, match="part id"):
            gcn.gcn_partition_stats(A, torch.from_numpy(part.astype(np.int32)).to(dev), p)
    A.free()
