// gcn_partition_stats: what a 1D row partition costs in communication, counted on the device.
//
// Sec. 4.3.2 (hypergraph model): column j of A^ is a net that joins the rows with a stored entry
// in that column; the part that owns vertex j sends row j of H (and of G) once to every other part
// in the net's connectivity set, so the rows moved per sparse product are sum_j (lambda(n_j) - 1).
// Sec. 5 reports, per processor, the volume and the number of messages sent.
//
// Two ways of counting, the same integers:
//   by columns  (handles with column-major arrays, p <= kPsMaxParts) every column's connectivity set is a bitmap of p
//               bits in LDS; one pass over the stored entries, no sort.
//   by sorting  one key per stored entry (i, j) whose ends lie in different parts:
//                   key = (part[j] * p + part[i]) << jbits | j          (sender, receiver, row)
//               Equal keys are the same transfer needed by several rows of the receiver: after a sort, the
//               distinct keys are the transfers, and the runs of equal (sender, receiver) are the messages.
#include <algorithm>

#include "common.h"

namespace gcn {

constexpr int kPsThreads = 256;
static inline dim3 ps_grid(int64_t n) { return fold_grid(ceil_div(n > 0 ? n : 1, kPsThreads)); }

struct PsOut { int64_t *load, *send_rows, *recv_rows, *send_msgs, *recv_msgs, *totals; };

__global__ void k_ps_zero(PsOut o, int p) {
  const int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < p) o.load[i] = o.send_rows[i] = o.recv_rows[i] = o.send_msgs[i] = o.recv_msgs[i] = 0;
  if (i < 2) o.totals[i] = 0;
}

__global__ void k_ps_zero_words(uint32_t* __restrict__ a, int64_t n) {
  const int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0u;
}

__global__ void k_ps_check(const int32_t* __restrict__ part, int64_t n, int p, int* __restrict__ bad) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < n && (part[i] < 0 || part[i] >= p)) *bad = 1;
}

__global__ void k_ps_load(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ part, int64_t n,
                          int64_t* __restrict__ load) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i >= n) return;
  atomicAdd(reinterpret_cast<unsigned long long*>(load + part[i]), (unsigned long long)(rowptr[i + 1] - rowptr[i]));
}

// entries whose ends share a part get the key of the pair id p*p, which sorts behind every real pair
__global__ void k_ps_keys(const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t nnz, int64_t n,
                          const int32_t* __restrict__ part, int p, int jbits, uint64_t* __restrict__ keys) {
  int64_t e = block_id() * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  int64_t lo = 0, hi = n;                  // row i: the last one with rowptr[i] <= e
  while (hi - lo > 1) {
    const int64_t m = (lo + hi) >> 1;
    if (rowptr[m] <= e) lo = m; else hi = m;
  }
  const int64_t j = col[e];
  const uint64_t ps = (uint64_t)part[j], pr = (uint64_t)part[lo];
  const uint64_t pair = ps != pr ? ps * (uint64_t)p + pr : (uint64_t)p * (uint64_t)p;
  keys[e] = (pair << jbits) | (uint64_t)j;
}

__global__ void k_ps_flags(const uint64_t* __restrict__ keys, int64_t nnz, uint64_t first_invalid,
                           uint32_t* __restrict__ flag) {
  int64_t e = block_id() * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const uint64_t k = keys[e];
  flag[e] = k < first_invalid && (e == 0 || keys[e - 1] != k) ? 1u : 0u;
}

// pos[e] = distinct transfers before position e.  A run of one (sender, receiver) pair spans [a, b]: it
// holds pos[b + 1] - pos[a] transfers, added as two terms by the threads at its two ends.
__global__ void k_ps_pairs(const uint64_t* __restrict__ keys, const int64_t* __restrict__ pos, int64_t nnz, int p,
                           int jbits, uint64_t first_invalid, int64_t* __restrict__ send_rows,
                           int64_t* __restrict__ recv_rows, int64_t* __restrict__ send_msgs,
                           int64_t* __restrict__ recv_msgs, int64_t* __restrict__ totals) {
  int64_t e = block_id() * blockDim.x + threadIdx.x;
  if (e >= nnz) return;
  const uint64_t k = keys[e];
  if (k >= first_invalid) return;
  const uint64_t pair = k >> jbits;
  const int ps = (int)(pair / (uint64_t)p), pr = (int)(pair % (uint64_t)p);
  typedef unsigned long long u64;
  const bool first = e == 0 || (keys[e - 1] >> jbits) != pair;
  const bool last = e == nnz - 1 || (keys[e + 1] >> jbits) != pair;
  if (first) {
    atomicAdd(reinterpret_cast<u64*>(send_rows + ps), (u64)(-pos[e]));
    atomicAdd(reinterpret_cast<u64*>(recv_rows + pr), (u64)(-pos[e]));
    atomicAdd(reinterpret_cast<u64*>(send_msgs + ps), (u64)1);
    atomicAdd(reinterpret_cast<u64*>(recv_msgs + pr), (u64)1);
  }
  if (last) {
    atomicAdd(reinterpret_cast<u64*>(send_rows + ps), (u64)pos[e + 1]);
    atomicAdd(reinterpret_cast<u64*>(recv_rows + pr), (u64)pos[e + 1]);
  }
  if (e == nnz - 1 || keys[e + 1] >= first_invalid) {      // the last entry that crosses parts
    totals[0] = pos[e + 1];
    totals[1] = e + 1;
  }
}

// ---- counting by columns -------------------------------------------------------------------------------------------
// What bounds it is the two gathers per entry (the part of the row's vertex, and the word of the pair table), served by
// L2, and the LDS atomics; the sort it replaces moved every entry's 8-byte key through memory ten times and more.
// Lanes per column: a wavefront holds four columns at once, each lane four entries in flight, because most columns are
// shorter than a wavefront (5 to 50 entries) and a column costs a chain of three dependent loads whatever its length.
// Columns come in the order of the schedule, so that the four of a wavefront are of like length.
constexpr int kPsLanes = 16;
constexpr int kPsGroups = kPsThreads / kPsLanes;
// The counters of a workgroup (entries, rows sent and rows received of every part) and its 16 bitmaps have to fit 64 KB
// of LDS: 3 p words + p / 2 words.
constexpr int kPsMaxParts = 4096;
static size_t ps_lds_bytes(int p) { return sizeof(uint32_t) * ((size_t)3 * p + 2 + (size_t)kPsGroups * ceil_div(p, 32)); }

// Connectivity sets of the long columns, which the schedule cuts into chunks of kHubChunkNnz entries: one workgroup per
// chunk; a chunk's bitmap is OR-ed into its column's.
__global__ __launch_bounds__(kPsThreads) void k_ps_hubs(const int64_t* __restrict__ colptr, const int32_t* __restrict__ rowidx,
                                                        const int32_t* __restrict__ hub_cols, const int64_t* __restrict__ hub_chunk_ptr,
                                                        const int32_t* __restrict__ chunk_hub, int64_t n_chunks,
                                                        const int32_t* __restrict__ part, int pw, uint32_t* __restrict__ hub_bits,
                                                        uint32_t* __restrict__ chunk_cut) {
  __shared__ uint32_t bm[kPsMaxParts / 32];
  __shared__ uint32_t cut;
  const int64_t c = block_id();
  if (c >= n_chunks) return;
  const int32_t h = chunk_hub[c];
  const int64_t j = hub_cols[h];
  for (int w = threadIdx.x; w < pw; w += kPsThreads) bm[w] = 0u;
  if (threadIdx.x == 0) cut = 0u;
  __syncthreads();
  const int ps = part[j];
  const int64_t s = colptr[j] + (c - hub_chunk_ptr[h]) * kHubChunkNnz, end = colptr[j + 1];
  uint32_t cross = 0;
#pragma unroll
  for (int u = 0; u < kHubChunkNnz / kPsThreads; ++u) {
    const int64_t e = s + u * kPsThreads + threadIdx.x;
    if (e >= end) continue;
    const int q = part[rowidx[e]];
    if (q == ps) continue;
    ++cross;
    atomicOr(&bm[q >> 5], 1u << (q & 31));
  }
  if (cross) atomicAdd(&cut, cross);
  __syncthreads();
  for (int w = threadIdx.x; w < pw; w += kPsThreads)
    if (bm[w]) atomicOr(&hub_bits[(int64_t)h * pw + w], bm[w]);
  if (threadIdx.x == 0) chunk_cut[c] = cut;          // (one counter for all chunks: 54 us of atomics on it, 2^18 R-MAT)
}

// partial[block] = { entries[p], rows sent[p], rows received[p], cut entries, rows moved } of the columns it took: 32
// bits each, since a block has seen fewer than 2^32 entries.
__global__ __launch_bounds__(kPsThreads) void k_ps_columns(const int64_t* __restrict__ colptr, const int32_t* __restrict__ rowidx,
                                                           const int64_t* __restrict__ rowptr, const int32_t* __restrict__ cols,
                                                           int64_t n_cols, const int32_t* __restrict__ hub_cols, int64_t n_hub,
                                                           const uint32_t* __restrict__ hub_bits, const uint32_t* __restrict__ chunk_cut,
                                                           int64_t n_chunks, const int32_t* __restrict__ part, int p, int pw, uint32_t* pair, uint32_t* __restrict__ partial) {
  extern __shared__ uint32_t ps_lds[];
  uint32_t* load = ps_lds;
  uint32_t* send = ps_lds + p;
  uint32_t* recv = ps_lds + 2 * p;
  uint32_t* sums = ps_lds + 3 * p;                   // cut entries, rows moved
  const int g = threadIdx.x / kPsLanes, l = threadIdx.x % kPsLanes;
  uint32_t* bm = ps_lds + 3 * p + 2 + g * pw;
  const int words = 3 * p + 2;
  for (int i = threadIdx.x; i < words + kPsGroups * pw; i += kPsThreads) ps_lds[i] = 0u;
  __syncthreads();

  uint32_t cross = 0, moved = 0;
  // part `ps` sends one more row to part q
  auto transfer = [&](int ps, int q) {
    atomicAdd(&recv[q], 1u);
    uint32_t* word = pair + (int64_t)ps * pw + (q >> 5);
    const uint32_t bit = 1u << (q & 31);
    if (!(*word & bit)) atomicOr(word, bit);         // (an old value costs one more atomic, no more)
  };
  const int64_t stride = (int64_t)gridDim.x * kPsGroups;
  const int64_t first = (int64_t)blockIdx.x * kPsGroups + g;
  for (int64_t it = first; it < n_cols; it += stride) {
    const int64_t j = cols[it];
    const int ps = part[j];
    const int64_t s = colptr[j];
    const int n = (int)(colptr[j + 1] - s);          // at most kHubRowNnz
    uint32_t fresh = 0;
    for (int base = 0; base < n; base += 4 * kPsLanes) {
      int q[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = base + u * kPsLanes + l;
        q[u] = k < n ? rowidx[s + k] : (int)j;       // (a vertex of the column's own part counts for nothing)
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) q[u] = part[q[u]];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (q[u] == ps) continue;
        ++cross;
        const uint32_t bit = 1u << (q[u] & 31);
        if (!(atomicOr(&bm[q[u] >> 5], bit) & bit)) { ++fresh; transfer(ps, q[u]); }
      }
    }
    if (fresh) { atomicAdd(&send[ps], fresh); moved += fresh; }
    if (l == 0) atomicAdd(&load[ps], (uint32_t)(rowptr[j + 1] - rowptr[j]));
    // the lanes of a column are lanes of one wavefront, whose LDS operations are carried out in order
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    for (int w = l; w < pw; w += kPsLanes) bm[w] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
  for (int64_t h = first; h < n_hub; h += stride) {
    const int64_t j = hub_cols[h];
    const int ps = part[j];
    uint32_t fresh = 0;
    for (int w = l; w < pw; w += kPsLanes) {
      uint32_t bits = hub_bits[h * pw + w];
      fresh += (uint32_t)__popc(bits);
      for (; bits; bits &= bits - 1) transfer(ps, w * 32 + __ffs(bits) - 1);
    }
    if (fresh) { atomicAdd(&send[ps], fresh); moved += fresh; }
    if (l == 0) atomicAdd(&load[ps], (uint32_t)(rowptr[j + 1] - rowptr[j]));
  }
  for (int64_t c = (int64_t)blockIdx.x * kPsThreads + threadIdx.x; c < n_chunks; c += (int64_t)gridDim.x * kPsThreads) cross += chunk_cut[c];
  if (cross) atomicAdd(&sums[0], cross);
  if (moved) atomicAdd(&sums[1], moved);
  __syncthreads();
  for (int i = threadIdx.x; i < words; i += kPsThreads) partial[(int64_t)blockIdx.x * words + i] = ps_lds[i];
}

constexpr int kPsSplit = 32;         // blocks in y that share a sum over workgroups or over the rows of the pair table

__global__ void k_ps_sum(const uint32_t* __restrict__ partial, int64_t n_blocks, int p, PsOut o) {
  const int words = 3 * p + 2;
  const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= words) return;
  unsigned long long v = 0;
  for (int64_t b = blockIdx.y; b < n_blocks; b += kPsSplit) v += partial[b * words + c];
  int64_t* to = c < p ? o.load + c : c < 2 * p ? o.send_rows + (c - p) : c < 3 * p ? o.recv_rows + (c - 2 * p) : o.totals + (c == 3 * p ? 1 : 0);
  if (v) atomicAdd(reinterpret_cast<unsigned long long*>(to), v);
}

// bit (s, r) of the pair table: s sends to r
__global__ void k_ps_messages(const uint32_t* __restrict__ pair, int p, int pw, PsOut o) {
  const int r = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  unsigned long long got = 0;
  for (int s = (int)blockIdx.y; s < p; s += kPsSplit) {
    const bool bit = r < p && ((pair[(int64_t)s * pw + (r >> 5)] >> (r & 31)) & 1u);
    got += bit ? 1u : 0u;
    const unsigned long long sent = (unsigned long long)__popcll(__ballot(bit));
    if ((threadIdx.x & 63) == 0 && sent) atomicAdd(reinterpret_cast<unsigned long long*>(o.send_msgs + s), sent);
  }
  if (got) atomicAdd(reinterpret_cast<unsigned long long*>(o.recv_msgs + r), got);
}

static int count_by_columns(const gcn_csr_t* A, const int32_t* d_part, int p, const PsOut& o, CallScope& sc) {
  hipStream_t s = sc.s;
  const Schedule& t = A->sched_t;
  const int pw = (int)ceil_div(p, 32);
  const size_t lds = ps_lds_bytes(p);
  // as many workgroups as the chip holds at once (256 compute units of 160 KB of LDS and 8 such workgroups)
  const int64_t per_cu = std::min<int64_t>(8, (int64_t)((size_t)160 * 1024 / lds));
  const int64_t blocks = std::min<int64_t>(256 * per_cu, std::max<int64_t>(1, ceil_div(std::max(t.n_wave_rows, t.n_hub_rows), kPsGroups)));
  const int64_t pair_words = (int64_t)p * pw, hub_words = t.n_hub_rows * pw;
  DevBuf bits, partial;
  GCN_TRY(bits.alloc(sc, sizeof(uint32_t) * (size_t)(pair_words + hub_words + t.n_chunks)));
  GCN_TRY(partial.alloc(sc, sizeof(uint32_t) * (size_t)blocks * (size_t)(3 * (int64_t)p + 2)));
  uint32_t* pair = bits.as<uint32_t>();
  uint32_t* hub_bits = pair + pair_words;
  uint32_t* chunk_cut = hub_bits + hub_words;
  k_ps_zero_words<<<ps_grid(pair_words + hub_words), kPsThreads, 0, s>>>(pair, pair_words + hub_words);
  if (t.n_chunks > 0)
    k_ps_hubs<<<fold_grid(t.n_chunks), kPsThreads, 0, s>>>(A->colptr, A->rowidx, t.hub_rows, t.hub_chunk_ptr, t.chunk_hub, t.n_chunks,
                                                          d_part, pw, hub_bits, chunk_cut);
  k_ps_columns<<<(unsigned)blocks, kPsThreads, lds, s>>>(A->colptr, A->rowidx, A->rowptr, t.wave_rows, t.n_wave_rows, t.hub_rows,
                                                        t.n_hub_rows, hub_bits, chunk_cut, t.n_chunks, d_part, p, pw, pair, partial.as<uint32_t>());
  k_ps_sum<<<dim3((unsigned)ceil_div(3 * (int64_t)p + 2, kPsThreads), kPsSplit), kPsThreads, 0, s>>>(partial.as<uint32_t>(), blocks, p, o);
  k_ps_messages<<<dim3((unsigned)ceil_div(p, kPsThreads), kPsSplit), kPsThreads, 0, s>>>(pair, p, pw, o);
  GCN_CHECK_LAUNCH();
  GCN_HIP(hipStreamSynchronize(s));      // the temporaries go back on return
  sc.done = true;
  return GCN_OK;
}

}  // namespace gcn

using namespace gcn;

extern "C" int gcn_partition_stats(const gcn_csr_t* A, const int32_t* d_part, int p, int64_t* d_load,
                                   int64_t* d_send_rows, int64_t* d_recv_rows, int64_t* d_send_msgs,
                                   int64_t* d_recv_msgs, int64_t* d_totals, void* stream) {
  clear_error();
  if (!A || !d_part) return fail(GCN_EINVAL, "gcn_partition_stats: NULL argument");
  if (A->nh != 0 || A->nr != A->n_global)
    return fail(GCN_EINVAL, "gcn_partition_stats: needs the handle of a whole graph (every row, no halo columns)");
  if (p < 1 || p > 32768) return fail(GCN_EINVAL, "gcn_partition_stats: the number of parts must be in [1, 32768]");
  hipStream_t s = (hipStream_t)stream;
  const int64_t n = A->nr, nnz = A->nnz;

  // results the caller does not ask for still have to land somewhere
  CallScope sc(s);
  DevBuf spare;
  GCN_TRY(spare.alloc(sc, sizeof(int64_t) * (size_t)(5 * (int64_t)p + 2)));
  int64_t* sp = spare.as<int64_t>();
  int64_t* load = d_load ? d_load : sp;
  int64_t* send_rows = d_send_rows ? d_send_rows : sp + p;
  int64_t* recv_rows = d_recv_rows ? d_recv_rows : sp + 2 * (int64_t)p;
  int64_t* send_msgs = d_send_msgs ? d_send_msgs : sp + 3 * (int64_t)p;
  int64_t* recv_msgs = d_recv_msgs ? d_recv_msgs : sp + 4 * (int64_t)p;
  int64_t* totals = d_totals ? d_totals : sp + 5 * (int64_t)p;
  const PsOut o{load, send_rows, recv_rows, send_msgs, recv_msgs, totals};
  k_ps_zero<<<ps_grid(p), kPsThreads, 0, s>>>(o, p);
  GCN_CHECK_LAUNCH();

  DevBuf bad;
  GCN_TRY(bad.alloc(sc, sizeof(int)));
  GCN_HIP(hipMemsetAsync(bad.p, 0, sizeof(int), s));
  k_ps_check<<<ps_grid(n), kPsThreads, 0, s>>>(d_part, n, p, bad.as<int>());
  GCN_CHECK_LAUNCH();
  int h_bad = 0;
  GCN_HIP(hipMemcpyAsync(&h_bad, bad.p, sizeof(int), hipMemcpyDeviceToHost, s));
  GCN_HIP(hipStreamSynchronize(s));
  if (h_bad) return fail(GCN_EINVAL, "gcn_partition_stats: a part id lies outside [0, p)");

  if (A->colptr && p <= kPsMaxParts && !tune().partition_sort) return count_by_columns(A, d_part, p, o, sc);

  k_ps_load<<<ps_grid(n), kPsThreads, 0, s>>>(A->rowptr, d_part, n, load);
  GCN_CHECK_LAUNCH();
  if (nnz == 0) { GCN_HIP(hipStreamSynchronize(s)); sc.done = true; return GCN_OK; }

  int jbits = 1;
  while (((int64_t)1 << jbits) < n) ++jbits;
  int pair_bits = 1;
  while (((uint64_t)1 << pair_bits) <= (uint64_t)p * (uint64_t)p) ++pair_bits;
  const uint64_t first_invalid = ((uint64_t)p * (uint64_t)p) << jbits;

  DevBuf ka, kb, tmp, flag, pos;
  GCN_TRY(ka.alloc(sc, sizeof(uint64_t) * (size_t)nnz));
  GCN_TRY(kb.alloc(sc, sizeof(uint64_t) * (size_t)nnz));
  GCN_TRY(tmp.alloc(sc, std::max(sort_tmp_bytes(nnz), scan_tmp_bytes(nnz))));
  GCN_TRY(flag.alloc(sc, sizeof(uint32_t) * (size_t)nnz));
  GCN_TRY(pos.alloc(sc, sizeof(int64_t) * (size_t)(nnz + 1)));
  k_ps_keys<<<ps_grid(nnz), kPsThreads, 0, s>>>(A->rowptr, A->col, nnz, n, d_part, p, jbits, ka.as<uint64_t>());
  GCN_CHECK_LAUNCH();
  uint64_t* sorted = nullptr; uint32_t* unused = nullptr;
  GCN_TRY(radix_sort_u64(ka.as<uint64_t>(), kb.as<uint64_t>(), nullptr, nullptr, nnz, 0, jbits + pair_bits, tmp.p, s,
                         &sorted, &unused));
  k_ps_flags<<<ps_grid(nnz), kPsThreads, 0, s>>>(sorted, nnz, first_invalid, flag.as<uint32_t>());
  GCN_CHECK_LAUNCH();
  GCN_TRY(exclusive_scan_u32(flag.as<uint32_t>(), pos.as<int64_t>(), nnz, tmp.p, s));
  k_ps_pairs<<<ps_grid(nnz), kPsThreads, 0, s>>>(sorted, pos.as<int64_t>(), nnz, p, jbits, first_invalid, send_rows,
                                               recv_rows, send_msgs, recv_msgs, totals);
  GCN_CHECK_LAUNCH();
  GCN_HIP(hipStreamSynchronize(s));      // the temporaries go back on return
  sc.done = true;
  return GCN_OK;
}
