"""What is timed of this library: the calls that a training or inference program makes, over the range they are made for.

A case is a plain dict.  Its "kind" says which program it is:
  step       one full-batch training step: forward, loss, backward, weight update (the epoch of bench.py plus the update)
  infer      the forward pass alone, on plain contiguous tensors, with biases
  block      one processor's row block: halo rows gathered from a device table beside the owned-column product
             (Algorithm 1), loss, push-form backward
  minibatch  one mini-batch step: induced subgraph of a vertex list, its feature rows, a training step on it
  build      the normalised adjacency block (CSR and CSC) from an edge list, and its arrays
  stats      communication figures of a row partition of a built graph
"graph" is the law of the edges (er: uniform ends, rmat: power law, lognormal: dense neighbourhoods, degrees spread by a
log-normal law), "n" the vertices, "degree" the mean number of distinct neighbours, "dims" the layer widths.
"""
from __future__ import annotations

import math

import torch

import paper_2212_05009_amd as gcn

LR = 0.05


def listed():
    return [
        # the smallest graph of the benchmark: launches and host work count, not bytes
        dict(name="step_er4k", kind="step", graph="er", n=4096, degree=16.0, dims="64,16,8", dtype="f32"),
        # a citation-network-sized graph served forward only: two small calls, ragged sizes
        dict(name="infer_2708", kind="infer", graph="er", n=2708, degree=4.0, dims="100,50,7", dtype="f32"),
        # a power-law graph of ordinary size (the benchmark's second workload)
        dict(name="step_rmat18", kind="step", graph="rmat", n=1 << 18, degree=44.0, dims="128,128,16", dtype="f32"),
        # the same size served forward only with bf16 features
        dict(name="infer_rmat18_bf16", kind="infer", graph="rmat", n=1 << 18, degree=44.0, dims="128,128,16", dtype="bf16"),
        # road-network-like: very short rows, several layers of one odd width (depth L > 2 and d = 50 in the paper's runs)
        dict(name="step_deep_d50", kind="step", graph="er", n=500_009, degree=5.6, dims="50,50,50,50,7", dtype="f32"),
        # dense neighbourhoods: 490 entries per row, wide and odd input features (the benchmark's third workload)
        dict(name="step_dense233k", kind="step", graph="lognormal", n=232_965, degree=492.0, dims="602,128,41", dtype="f32"),
        # the largest full graph of the benchmark, in both feature types
        dict(name="step_sparse2m4", kind="step", graph="rmat", n=2_449_029, degree=50.5, dims="100,256,256,47", dtype="f32"),
        dict(name="step_sparse2m4_bf16", kind="step", graph="rmat", n=2_449_029, degree=50.5, dims="100,256,256,47", dtype="bf16"),
        # one processor's rows of a larger graph, as in the benchmark's row block but with the table on the device
        dict(name="block_512k", kind="block", n=1 << 19, n_global=1 << 22, halo=3 << 18, degree=16.0, dims="128,128,32", dtype="f32"),
        # mini-batches of 20 K vertices (the size of the paper's mini-batch experiment)
        dict(name="minibatch_20k", kind="minibatch", graph="rmat", n=1 << 18, degree=44.0, batch=20_000, dims="128,128,16", dtype="f32"),
        # set-up of the power-law graph: sorts, normalisation, column-major copy, schedules
        dict(name="build_rmat18", kind="build", graph="rmat", n=1 << 18, degree=44.0),
        # the communication table of a 512-way partition
        dict(name="stats_p512", kind="stats", graph="rmat", n=1 << 18, degree=44.0, parts=512),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "infer", "infer", "block", "minibatch", "build", "stats"])
    for _ in range(10_000):
        depth = rng.choice([2, 2, 2, 3, 3, 4, 5])
        dims = [_log_int(rng, 16, 602)] + [rng.choice([16, 32, 64, 100, 128, 256, _log_int(rng, 12, 256)])] * (depth - 1) + [_log_int(rng, 2, 64)]
        graph = rng.choice(["er", "rmat", "rmat", "lognormal"])
        degree = round(math.exp(rng.uniform(math.log(3.0), math.log(500.0 if graph == "lognormal" else 64.0))), 2)
        case = dict(kind=kind, graph=graph, n=_log_int(rng, 2_000, 2_449_029), degree=degree, dims=",".join(map(str, dims)),
                    dtype=rng.choice(["f32", "f32", "bf16"]))
        if kind == "block":
            case = dict(case, n=_log_int(rng, 20_000, 1 << 20), degree=round(rng.uniform(6.0, 40.0), 2), dtype="f32")
            del case["graph"]
            case["n_global"] = case["n"] * rng.choice([3, 4, 8])
            case["halo"] = int(case["n"] * rng.uniform(0.2, 1.5))
        elif kind == "minibatch":
            case["n"] = _log_int(rng, 20_000, 1 << 20)
            case["batch"] = _log_int(rng, 1_000, max(2_000, case["n"] // 2))
        elif kind in ("build", "stats"):
            case = dict(kind=kind, graph=graph, n=case["n"], degree=degree)
            if kind == "stats":
                case["parts"] = _log_int(rng, 2, 2048)
        # no drawn graph beyond 60 M entries, no drawn pass beyond a fraction of the largest listed one
        rows = case["n"] + case.get("halo", 0)
        if case["n"] * degree > 6.0e7 or degree > case["n"] / 64:
            continue
        if kind in ("build", "stats"):
            return case
        w = work(case)
        if rows * sum(dims) <= 8.0e8 and w["bytes"] <= 8.0e9 and w["flops"] <= 4.0e11:
            return case
    raise RuntimeError("no case found")


# ---- inputs --------------------------------------------------------------------------------------------------------

def _pairs(case, m, gen, dev):
    """m samples of the graph's law (fewer where ends fall beyond n), duplicates and self-loops left in."""
    n = case["n"]
    if case["graph"] == "er":
        return torch.randint(n, (m,), generator=gen, device=dev), torch.randint(n, (m,), generator=gen, device=dev)
    if case["graph"] == "lognormal":
        w = torch.exp(torch.randn(n, generator=gen, device=dev, dtype=torch.float64))
        cdf = torch.cumsum(w, 0)
        cdf /= cdf[-1].clone()
        return tuple(torch.searchsorted(cdf, torch.rand(m, generator=gen, device=dev, dtype=torch.float64), right=True).clamp_(max=n - 1)
                     for _ in range(2))
    # R-MAT (0.57, 0.19, 0.19, 0.05) on a power-of-two grid
    scale = max(1, (n - 1).bit_length())
    u = torch.zeros(m, dtype=torch.int64, device=dev)
    v = torch.zeros(m, dtype=torch.int64, device=dev)
    for _ in range(scale):
        r = torch.rand(m, generator=gen, device=dev)
        u = u * 2 + (r >= 0.76).long()
        v = v * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95)).long()
    keep = (u < n) & (v < n)
    return u[keep], v[keep]


def _edges(case, gen, dev):
    """Raw directed edge list with both directions in random order: n * degree / 2 distinct pairs, an eighth of them listed
    twice, and a few self-loops, which the build has to drop."""
    n = case["n"]
    m = int(n * case["degree"] / 2)
    keys = torch.empty(0, dtype=torch.int64, device=dev)
    more = int(1.2 * m) + 16
    while keys.numel() < m:
        u, v = _pairs(case, more, gen, dev)
        new = (torch.minimum(u, v) * n + torch.maximum(u, v))[u != v]
        keys = torch.unique(torch.cat([keys, new]))
    keys = keys[torch.randperm(keys.numel(), generator=gen, device=dev)[:m]]
    loops = torch.randint(n, (n // 64 + 1,), generator=gen, device=dev)
    # new names for the vertices, or the hubs would be the lowest ids; and a random direction first
    name = torch.randperm(n, generator=gen, device=dev)
    u, v = name[keys // n], name[keys % n]
    turn = torch.rand(m, generator=gen, device=dev) < 0.5
    u, v = torch.where(turn, v, u), torch.where(turn, u, v)
    d = m // 8
    src = torch.cat([u, u[:d], loops, v, v[:d]])
    dst = torch.cat([v, v[:d], loops, u, u[:d]])
    return src.to(torch.int32), dst.to(torch.int32)


def _block_edges(case, gen, dev):
    """Rows of one processor: power-law row lengths, half of the entries owned, the rest drawn from `halo` foreign ids."""
    n, n_global, halo, degree = case["n"], case["n_global"], case["halo"], case["degree"]
    lo = n_global // 4 // 64 * 64
    raw = (1.0 - torch.rand(n, generator=gen, device=dev, dtype=torch.float64)).pow(-1.0 / 1.2).clamp_(max=1e5)
    lens = (raw * ((degree - 1.0) / raw.mean()) + 0.5).floor().clamp_(min=1).long()
    src = torch.repeat_interleave(torch.arange(lo, lo + n, device=dev), lens)
    total = src.numel()
    ids = torch.randperm(n_global - n, generator=gen, device=dev)[:halo]
    ids = torch.where(ids >= lo, ids + n, ids)
    own = torch.rand(total, generator=gen, device=dev) < 0.5
    r = torch.rand(total, generator=gen, device=dev, dtype=torch.float64)
    near = lo + (r.pow(1.5) * n).long().clamp_(max=n - 1)
    far = ids[(r.pow(3.0) * halo).long().clamp_(max=halo - 1)]
    at = torch.nonzero(~own).flatten()
    far[at[torch.randperm(at.numel(), generator=gen, device=dev)[:halo]]] = ids      # every foreign id is somebody's neighbour
    dst = torch.where(own, near, far)
    deg = torch.randint(2, int(2 * degree), (n_global,), generator=gen, device=dev).to(torch.int32)
    return src.to(torch.int32), dst.to(torch.int32), lo, deg


def _dims(case):
    return [int(d) for d in case["dims"].split(",")]


class _Net:
    """Weights, labels and the buffers of a training step on a block of nr rows with nc columns."""

    def __init__(self, dims, nr, nc, fdt, gen, dev):
        self.dims, self.L, self.nr = dims, len(dims) - 1, nr
        L = self.L
        self.W = [(torch.rand(dims[k], dims[k + 1], generator=gen, device=dev) * 2 - 1) * math.sqrt(6.0 / (dims[k] + dims[k + 1]))
                  for k in range(L)]
        self.y = torch.randint(dims[L], (nr,), generator=gen, device=dev).to(torch.int32)
        self.H = [gcn.feature_buffer(nc, dims[k], fdt, dev) for k in range(L)]
        # A^ H is kept where the forward pass computes it anyway
        self.AH = [torch.empty(nr, dims[k], dtype=fdt, device=dev) if dims[k] <= dims[k + 1] else None for k in range(L)]
        self.Z = torch.empty(nr, dims[L], dtype=fdt, device=dev)
        self.D = [gcn.feature_buffer(nc, dims[k + 1], fdt, dev) for k in range(L - 1)]
        self.G = [d[:nr] for d in self.D] + [gcn.feature_buffer(nr, dims[L], fdt, dev)]
        self.dW = [torch.empty_like(w) for w in self.W]
        self.loss = torch.zeros(1, device=dev)

    def forward(self, A):
        for k in range(self.L):
            last = k == self.L - 1
            gcn.gcn_layer_fwd_ld(A, self.H[k], self.W[k], self.Z if last else self.H[k + 1][:self.nr],
                                 act=gcn.ACT_NONE if last else gcn.ACT_RELU, AH_save=self.AH[k])

    def backward(self, A):
        nr = self.nr
        gcn.gcn_softmax_xent(self.Z, self.y, 1.0 / nr, self.loss, self.G[self.L - 1])
        for k in range(self.L - 1, -1, -1):
            gcn.gcn_layer_bwd_ld(A, self.H[k], self.W[k], self.G[k], self.dW[k], dH=self.D[k - 1] if k else None,
                                 Zprev=self.H[k][:nr] if k else None, AH_saved=self.AH[k])

    def update(self):
        for w, dw in zip(self.W, self.dW):
            gcn.gcn_sgd_update(w, dw, LR)


def prepare(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    kind, n = case["kind"], case["n"]
    fdt = torch.bfloat16 if case.get("dtype") == "bf16" else torch.float32
    st = {"kind": kind}
    if kind == "block":
        src, dst, lo, deg = _block_edges(case, gen, dev)
        A = gcn.gcn_csr_build(src, dst, case["n_global"], lo, lo + n, deg_global=deg)
        dims = _dims(case)
        net = _Net(dims, A.nr, A.nc, fdt, gen, dev)
        # rows that other processors hold, one table per layer input
        st["tables"] = [torch.randn(case["n_global"], d, generator=gen, device=dev, dtype=fdt) for d in dims[:-1]]
        net.H[0][:A.nr] = st["tables"][0][lo:lo + n]
        st.update(A=A, net=net, halo=A.arrays()["halo_gid"], side=torch.cuda.Stream(),
                  P=[None if net.AH[k] is not None else gcn.feature_buffer(A.nc, dims[k + 1], fdt, dev) for k in range(net.L)])
        return st
    src, dst = _edges(case, gen, dev)
    if kind == "build":
        st.update(src=src, dst=dst, n=n)
        return st
    A = gcn.gcn_csr_build(src, dst, n)
    del src, dst
    st["A"] = A
    if kind == "stats":
        st.update(part=torch.randint(case["parts"], (n,), generator=gen, device=dev).to(torch.int32), p=case["parts"])
        return st
    dims = _dims(case)
    if kind == "infer":
        st["X"] = torch.randn(n, dims[0], generator=gen, device=dev).to(fdt)
        st["W"] = [(torch.rand(a, b, generator=gen, device=dev) * 2 - 1) * math.sqrt(6.0 / (a + b)) for a, b in zip(dims, dims[1:])]
        st["bias"] = [torch.randn(b, generator=gen, device=dev) * 0.1 for b in dims[1:]]
        st["out"] = [torch.empty(n, b, dtype=fdt, device=dev) for b in dims[1:]]
    elif kind == "minibatch":
        b = case["batch"]
        st["verts"] = torch.randperm(n, generator=gen, device=dev)[:b].to(torch.int32)
        st["X"] = torch.randn(n, dims[0], generator=gen, device=dev).to(fdt)
        st["labels"] = torch.randint(dims[-1], (n,), generator=gen, device=dev).to(torch.int32)
        st["net"] = _Net(dims, b, b, fdt, gen, dev)
    else:
        st["net"] = _Net(dims, n, n, fdt, gen, dev)
        st["net"].H[0][:] = torch.randn(n, dims[0], generator=gen, device=dev).to(fdt)
    return st


# ---- one pass ------------------------------------------------------------------------------------------------------

def _infer(st):
    A, x, last = st["A"], st["X"], len(st["W"]) - 1
    for k, w in enumerate(st["W"]):
        x = gcn.gcn_layer_fwd(A, x, w, st["out"][k], act=gcn.ACT_NONE if k == last else gcn.ACT_RELU, bias=st["bias"][k])
    return x


def _block(st):
    A, net, nr = st["A"], st["net"], st["net"].nr
    main, side = torch.cuda.current_stream(), st["side"]
    for k in range(net.L):
        last = k == net.L - 1
        H, W, out = net.H[k], net.W[k], net.Z if last else net.H[k + 1][:nr]
        act = gcn.ACT_NONE if last else gcn.ACT_RELU
        side.wait_stream(main)             # the rows being replaced were read by the pass before
        with torch.cuda.stream(side):
            gcn.gcn_halo_gather(st["tables"][k], st["halo"], H[nr:])
        if net.AH[k] is not None:
            gcn.gcn_spmm_part(A, gcn.PART_LOCAL, H, net.AH[k])
            main.wait_stream(side)
            gcn.gcn_spmm_part(A, gcn.PART_HALO, H, net.AH[k])
            gcn.gcn_dense_fwd(net.AH[k], W, out, act=act)
        else:
            P = st["P"][k]
            gcn.gcn_dense_fwd(H[:nr], W, P[:nr])
            gcn.gcn_spmm_part(A, gcn.PART_LOCAL, P, out)
            main.wait_stream(side)
            gcn.gcn_dense_fwd(H[nr:], W, P[nr:])
            gcn.gcn_spmm_part(A, gcn.PART_HALO, P, out, epilogue=gcn.EPI_NONE if last else gcn.EPI_RELU)
    net.backward(A)
    return [net.loss, net.Z, net.dW, [d[nr:] for d in net.D]]


def _minibatch(st):
    net, verts = st["net"], st["verts"]
    sub = gcn.gcn_csr_induced(st["A"], verts)
    gcn.gcn_halo_gather(st["X"], verts, net.H[0])
    net.y = st["labels"][verts]
    net.forward(sub)
    net.backward(sub)
    net.update()
    sub.free()
    return [net.loss, net.Z, net.dW, net.W]


def run(state):
    kind = state["kind"]
    if kind == "step":
        A, net = state["A"], state["net"]
        net.forward(A)
        net.backward(A)
        net.update()
        return [net.loss, net.Z, net.dW, net.W]
    if kind == "infer":
        return _infer(state)
    if kind == "block":
        return _block(state)
    if kind == "minibatch":
        return _minibatch(state)
    if kind == "build":
        A = gcn.gcn_csr_build(state["src"], state["dst"], state["n"])
        out = A.arrays()
        A.free()
        return out
    return gcn.gcn_partition_stats(state["A"], state["part"], state["p"])


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def work(case):
    """Every operand of every product once: a product needs the whole result of the one before, so the matrix is read once
    per sparse product (8 bytes an entry) and each layer's rows are written once and read once by whoever needs them
    next, at the narrower of the layer's two widths where the sparse product may choose its side."""
    kind, n = case["kind"], case["n"]
    nnz = n * (case["degree"] + 1)
    if kind == "build":       # edge list in; CSR and CSC arrays out
        return {"bytes": 8.0 * n * case["degree"] + 16.0 * nnz + 24.0 * n, "flops": 0.0}
    if kind == "stats":       # columns, row pointers and parts in; five counters per part out
        return {"bytes": 4.0 * nnz + 12.0 * n + 40.0 * case["parts"], "flops": 0.0}
    rows, cols, extra = n, n + case.get("halo", 0), 0.0
    dims, es = _dims(case), 2 if case["dtype"] == "bf16" else 4
    if kind == "minibatch":   # the selected rows of the parent are read, the subgraph's arrays are written
        rows = cols = case["batch"]
        extra = 4.0 * nnz * rows / n + es * rows * dims[0]
        nnz = rows * (case["degree"] * rows / n + 1)
        extra += 16.0 * nnz
    b = f = 0.0
    for k, (d_in, d_out) in enumerate(zip(dims, dims[1:])):
        w = min(d_in, d_out)
        b += 8.0 * nnz + es * (cols * d_in + rows * d_out) + 4.0 * d_in * d_out
        f += 2.0 * nnz * w + 2.0 * rows * d_in * d_out
        if kind == "block":   # halo rows arrive from the table
            b += es * case["halo"] * d_in
        if kind != "infer":   # backward: H and G in, dW out, dH out beyond the first layer
            b += es * (rows * d_in + rows * d_out) + 4.0 * d_in * d_out
            f += 2.0 * rows * d_in * d_out
            if k or w < d_in:     # the gradient handed down, or dW through A^T G where A^ H was not kept
                b += 8.0 * nnz
                f += 2.0 * nnz * w
            if k:
                b += es * (cols * d_in + rows * d_in)
                f += 2.0 * rows * d_in * d_out
    return {"bytes": b + extra, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind in ("build", "stats"):
        return "exact"            # integers, and values with every operation correctly rounded
    if case["dtype"] == "bf16":
        return {"rel": 1e-2}      # features, activations and gradients are stored in bf16
    if kind == "infer":
        return {"rel": 1e-5}      # fp32 sums in another order
    # A training step masks its gradient with [Z > 0].  Sums in another order change the sign of about 2e-7 of the hidden
    # values; each such value switches one element of the gradient on or off, sqrt(2 / hidden values) of its norm.
    dims = _dims(case)
    hidden = (case.get("batch") or case["n"]) * sum(dims[1:-1])
    return {"rel": min(0.01, max(1e-3, 1.5 * math.sqrt(2.0 / hidden)))}
