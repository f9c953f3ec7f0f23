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
// What bounds it is the gather of a part per entry, out of L2 (11.8 M entries: about 70 us at the 160 G requests/s it answers); the
// figures of a column are kept in registers and LDS.  A column costs a chain of dependent requests (its number, its ends and part,
// its rows, their parts), so it gets the lanes that leave it one step of that chain: a wavefront for 64 entries and more (8 a lane), 16
// lanes for 16 to 63, four lanes below, where equal parts are found by comparing registers.  Columns come in the order of the schedule,
// whose length classes are those bounds.  Whole calls, against 16 lanes for every column, the pair table in memory and its word asked for
// entry by entry, 2048 workgroups and the ids checked by a launch and a wait of their own, us before / now: 2^18 R-MAT columns of
// 45 entries, 512 parts 226 / 131 (this kernel 130 / 92); 1.2 M of 13, 27 parts 702 / 185; 82 K uniform ones of 24, 15 parts 621 / 78; 67 K
// log-normal ones of 444, 1692 parts 519 / 275.
constexpr int kPsColThreads = 1024, kPsWaves = kPsColThreads / 64;
constexpr int kPsLanes = 16, kPsFew = 4;         // lanes of a column of 16 to 63 entries; of fewer
constexpr int kPsGroups = kPsColThreads / kPsLanes;
// The counters of a workgroup (entries, rows sent and rows received of every part) and its 64 bitmaps take 3 p + 2 words and 2 p words of its
// LDS: 80 KB at most, and up to 4095 parts a second workgroup fits the compute unit.
constexpr int kPsMaxParts = 4096;
// The pair table fits LDS up to 512 parts: a workgroup marks its pairs there and looks at the table in memory once, at the end.
constexpr int kPsPairLds = 512;
static size_t ps_lds_bytes(int p) {
  const size_t pw = (size_t)ceil_div(p, 32);
  return sizeof(uint32_t) * ((size_t)3 * p + 2 + (size_t)kPsGroups * pw + (p <= kPsPairLds ? (size_t)p * pw : 0));
}

struct PsColumns {
  const int64_t* colptr; const int32_t* rowidx; const int64_t* rowptr;
  const int32_t* cols; int64_t n_long, n_mid, n_cols;      // columns of 64 entries and more, of 16 and more, all but the hub columns
  const int32_t* hub_cols; const int64_t* hub_chunk_ptr; const int32_t* chunk_hub; int64_t n_hub, n_chunks;
  const int32_t* part; int p, pw;
  uint32_t* pair;            // [p][pw] bit (s, r): part s sends to part r
  uint32_t* hub_bits;        // [n_hub][pw] connectivity sets of the hub columns
  uint32_t* partial;         // [workgroups][3 p + 2] entries, rows sent, rows received of every part, cut entries, rows moved
  int* bad;
};

// Clears the results, the tables and the verdict.
__global__ void k_ps_clear(PsOut o, int p, uint32_t* __restrict__ words, int64_t n, int* __restrict__ bad) {
  const int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < p) o.load[i] = o.send_rows[i] = o.recv_rows[i] = o.send_msgs[i] = o.recv_msgs[i] = 0;
  if (i < 2) o.totals[i] = 0;
  if (i == 0) *bad = 0;
  if (i < n) words[i] = 0u;
}

// LDS operations of one wavefront are carried out in order; this keeps the compiler to it
__device__ __forceinline__ void ps_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// A block has seen fewer than 2^32 entries: 32 bits a counter.  A part id out of range counts as part 0 and is reported.
template <bool PAIR_LDS>
__global__ __launch_bounds__(kPsColThreads) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ps_columns(PsColumns a) {
  extern __shared__ uint32_t ps_lds[];
  const int p = a.p, pw = a.pw;
  uint32_t* load = ps_lds;
  uint32_t* send = ps_lds + p;
  uint32_t* recv = ps_lds + 2 * p;
  uint32_t* sums = ps_lds + 3 * p;                   // cut entries, rows moved
  const int words = 3 * p + 2;
  uint32_t* sets = ps_lds + words;                   // bitmaps of the groups; a wavefront's own are those of its four groups
  uint32_t* pairs = sets + kPsGroups * pw;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i < words + kPsGroups * pw + (PAIR_LDS ? p * pw : 0); i += kPsColThreads) ps_lds[i] = 0u;
  __syncthreads();

  uint32_t cross = 0, moved = 0;
  auto part_of = [&](int64_t i) {
    const int q = a.part[i];
    return (uint32_t)q < (uint32_t)p ? q : 0;
  };
  auto own_part = [&](int64_t j) {
    const int q = a.part[j];
    if ((uint32_t)q < (uint32_t)p) return q;
    *a.bad = 1;
    return 0;
  };
  // Part `ps` sends one more row to each part q[u] that is fresh.  The pair table in memory is looked at for all of them together, and
  // written where a bit is missing (an old value costs one more atomic, no more).
  auto transfer = [&](int ps, const auto& q, const auto& fresh) -> uint32_t {
    constexpr int U = sizeof(q) / sizeof(q[0]);
    uint32_t n = 0, old[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (!PAIR_LDS) old[u] = fresh[u] ? a.pair[ps * pw + (q[u] >> 5)] : ~0u;
      if (!fresh[u]) continue;
      ++n;
      atomicAdd(&recv[q[u]], 1u);
      if constexpr (PAIR_LDS) atomicOr(&pairs[ps * pw + (q[u] >> 5)], 1u << (q[u] & 31));
    }
    if constexpr (!PAIR_LDS) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (!(old[u] & (1u << (q[u] & 31)))) atomicOr(&a.pair[ps * pw + (q[u] >> 5)], 1u << (q[u] & 31));
    }
    return n;
  };
  auto column_done = [&](int64_t j, int ps, uint32_t fresh, bool first) {
    if (fresh) { atomicAdd(&send[ps], fresh); moved += fresh; }
    if (first) atomicAdd(&load[ps], (uint32_t)(a.rowptr[j + 1] - a.rowptr[j]));
  };
  const int64_t wave0 = (int64_t)blockIdx.x * kPsWaves + w, waves = (int64_t)gridDim.x * kPsWaves;

  // hub columns, a chunk of entries per wavefront, and columns of 64 entries and more
  {
    uint32_t* set = sets + (w * (64 / kPsLanes)) * pw;
    constexpr int kU = 8;                            // (16 a lane: no second workgroup on a compute unit)
    for (int64_t it = wave0; it < a.n_chunks + a.n_long; it += waves) {
      const bool hub = it < a.n_chunks;
      const int32_t hc = hub ? a.chunk_hub[it] : 0;
      const int64_t j = hub ? a.hub_cols[hc] : a.cols[it - a.n_chunks];
      const int ps = own_part(j);
      const int64_t c0 = a.colptr[j], c1 = a.colptr[j + 1];
      const int64_t s = hub ? c0 + (it - a.hub_chunk_ptr[hc]) * kHubChunkNnz : c0;
      const int n = (int)(hub && c1 - s > kHubChunkNnz ? kHubChunkNnz : c1 - s);
      uint32_t fresh = 0;
      for (int base = 0; base < n; base += kU * 64) {
        int q[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int k = base + u * 64 + lane;
          q[u] = base + u * 64 < n ? a.rowidx[s + (k < n ? k : n - 1)] : 0;
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
          if (base + u * 64 < n) q[u] = part_of(q[u]);
        bool is_new[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          is_new[u] = false;
          if (base + u * 64 + lane >= n || q[u] == ps) continue;
          ++cross;
          const uint32_t bit = 1u << (q[u] & 31);
          is_new[u] = !(atomicOr(&set[q[u] >> 5], bit) & bit) && !hub;
        }
        if (!hub) fresh += transfer(ps, q, is_new);
      }
      ps_order();
      for (int k = lane; k < pw; k += 64) {
        const uint32_t bits = set[k];
        if (hub && bits) atomicOr(&a.hub_bits[(int64_t)hc * pw + k], bits);
        set[k] = 0u;
      }
      ps_order();
      if (!hub) column_done(j, ps, fresh, lane == 0);
    }
  }
  // columns of 16 to 63 entries
  {
    const int l = lane % kPsLanes;
    const int g = (int)threadIdx.x / kPsLanes;
    uint32_t* set = sets + g * pw;
    constexpr int kU = 64 / kPsLanes;
    const int64_t groups = (int64_t)gridDim.x * kPsGroups;
    for (int64_t it = a.n_long + (int64_t)blockIdx.x * kPsGroups + g; it < a.n_mid; it += groups) {
      const int64_t j = a.cols[it];
      const int ps = own_part(j);
      const int64_t s = a.colptr[j];
      const int n = (int)(a.colptr[j + 1] - s);
      int q[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int k = u * kPsLanes + l;
        q[u] = a.rowidx[s + (k < n ? k : n - 1)];
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) q[u] = part_of(q[u]);
      bool is_new[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        is_new[u] = false;
        if (u * kPsLanes + l >= n || q[u] == ps) continue;
        ++cross;
        const uint32_t bit = 1u << (q[u] & 31);
        is_new[u] = !(atomicOr(&set[q[u] >> 5], bit) & bit);
      }
      column_done(j, ps, transfer(ps, q, is_new), l == 0);
      ps_order();
      // (what was set, by whom it was set; more parts than entries as a rule)
#pragma unroll
      for (int u = 0; u < kU; ++u) set[q[u] >> 5] = 0u;
      ps_order();
    }
  }
  // columns of up to 15 entries
  {
    const int l = lane % kPsFew;
    constexpr int kU = 4;
    const int64_t groups = (int64_t)gridDim.x * (kPsColThreads / kPsFew);
    for (int64_t it = a.n_mid + ((int64_t)blockIdx.x * kPsColThreads + threadIdx.x) / kPsFew; it < a.n_cols; it += groups) {
      const int64_t j = a.cols[it];
      const int ps = own_part(j);
      const int64_t s = a.colptr[j];
      const int n = (int)(a.colptr[j + 1] - s);
      int q[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int k = u * kPsFew + l;
        q[u] = n > 0 ? a.rowidx[s + (k < n ? k : n - 1)] : (int)j;
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        q[u] = part_of(q[u]);
        if (u * kPsFew + l >= n) q[u] = ps;          // (a vertex of the column's own part counts for nothing)
      }
      bool is_new[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        // an equal part in an earlier step, of any lane of the four, or in this one, of a lane before this
        bool seen = q[u] == ps;
        cross += seen ? 0u : 1u;
#pragma unroll
        for (int v = 0; v <= u; ++v)
#pragma unroll
          for (int o = 0; o < kPsFew; ++o) {
            const int other = __shfl_xor(q[v], o, kPsFew);
            seen = seen || (other == q[u] && (v < u || (l ^ o) < l));
          }
        is_new[u] = !seen;
      }
      column_done(j, ps, transfer(ps, q, is_new), l == 0);
    }
  }
  if (cross) atomicAdd(&sums[0], cross);
  if (moved) atomicAdd(&sums[1], moved);
  __syncthreads();
  for (int i = threadIdx.x; i < words; i += kPsColThreads) a.partial[(int64_t)blockIdx.x * words + i] = ps_lds[i];
  if constexpr (PAIR_LDS)
    for (int i = threadIdx.x; i < p * pw; i += kPsColThreads) {
      const uint32_t bits = pairs[i];
      if (bits & ~a.pair[i]) atomicOr(&a.pair[i], bits);
    }
}

// The hub columns, whose connectivity sets are complete: counters into the rows of `partial` behind those of the columns' workgroups.
constexpr int kPsHubBlocks = 32;
__global__ __launch_bounds__(kPsColThreads) void k_ps_hubs(PsColumns a, int64_t row0) {
  extern __shared__ uint32_t ps_lds[];
  const int p = a.p, pw = a.pw, words = 3 * p + 2;
  uint32_t *load = ps_lds, *send = ps_lds + p, *recv = ps_lds + 2 * p, *sums = ps_lds + 3 * p;
  for (int i = threadIdx.x; i < words; i += kPsColThreads) ps_lds[i] = 0u;
  __syncthreads();
  uint32_t moved = 0;
  for (int64_t i = (int64_t)blockIdx.x * kPsColThreads + threadIdx.x; i < a.n_hub * pw; i += (int64_t)gridDim.x * kPsColThreads) {
    const int64_t h = i / pw, k = i % pw, j = a.hub_cols[h];
    const int own = a.part[j], ps = (uint32_t)own < (uint32_t)p ? own : 0;
    uint32_t bits = a.hub_bits[i];
    if (k == 0) atomicAdd(&load[ps], (uint32_t)(a.rowptr[j + 1] - a.rowptr[j]));
    if (!bits) continue;
    const uint32_t fresh = (uint32_t)__popc(bits);
    atomicAdd(&send[ps], fresh);
    moved += fresh;
    if (bits & ~a.pair[(int64_t)ps * pw + k]) atomicOr(&a.pair[(int64_t)ps * pw + k], bits);
    // (full sets: from the first bit on, the lanes' counters would lie on one bank)
    const uint32_t turn = (uint32_t)i & 31u;
    bits = __builtin_rotateright32(bits, turn);
    for (; bits; bits &= bits - 1) atomicAdd(&recv[k * 32 + (((uint32_t)__ffs(bits) - 1u + turn) & 31u)], 1u);
  }
  if (moved) atomicAdd(&sums[1], moved);
  __syncthreads();
  for (int i = threadIdx.x; i < words; i += kPsColThreads) a.partial[(row0 + blockIdx.x) * words + i] = ps_lds[i];
}

constexpr int kPsSplit = 32;         // blocks in y that share a sum over workgroups or over the rows of the pair table

// The first `sum_blocks` blocks of x add up the workgroups' counters, the others count the messages: bit (s, r) of the pair table says
// that s sends to r.
__global__ void k_ps_finish(const uint32_t* __restrict__ partial, int64_t n_rows, int sum_blocks, const uint32_t* __restrict__ pair, int p, int pw, PsOut o) {
  typedef unsigned long long u64;
  if ((int)blockIdx.x < sum_blocks) {
    const int words = 3 * p + 2;
    const int c = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (c >= words) return;
    u64 v = 0;
#pragma unroll 8
    for (int64_t b = blockIdx.y; b < n_rows; b += kPsSplit) v += partial[b * words + c];
    int64_t* to = c < p ? o.load + c : c < 2 * p ? o.send_rows + (c - p) : c < 3 * p ? o.recv_rows + (c - 2 * p) : o.totals + (c == 3 * p ? 1 : 0);
    if (v) atomicAdd(reinterpret_cast<u64*>(to), v);
    return;
  }
  const int r = (int)((blockIdx.x - sum_blocks) * blockDim.x + threadIdx.x);
  u64 got = 0;
  constexpr int kU = 8;                              // rows asked for together
  for (int s0 = (int)blockIdx.y; s0 < p; s0 += kU * kPsSplit) {
    uint32_t word[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int s = s0 + u * kPsSplit;
      word[u] = r < p && s < p ? pair[(int64_t)s * pw + (r >> 5)] : 0u;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const bool bit = (word[u] >> (r & 31)) & 1u;
      got += bit ? 1u : 0u;
      const u64 sent = (u64)__popcll(__ballot(bit));
      if ((threadIdx.x & 63) == 0 && sent) atomicAdd(reinterpret_cast<u64*>(o.send_msgs + s0 + u * kPsSplit), sent);
    }
  }
  if (got) atomicAdd(reinterpret_cast<u64*>(o.recv_msgs + r), got);
}

// Four launches and one wait: the ids are checked where the columns are counted, and the verdict is read with the end of the call.
static int count_by_columns(const gcn_csr_t* A, const int32_t* d_part, int p, const PsOut& o, CallScope& sc) {
  hipStream_t s = sc.s;
  const Schedule& t = A->sched_t;
  PsColumns a{A->colptr, A->rowidx, A->rowptr, t.wave_rows, t.class_begin[26], t.class_begin[28], t.n_wave_rows,
              t.hub_rows, t.hub_chunk_ptr, t.chunk_hub, t.n_hub_rows, t.n_chunks, d_part, p, (int)ceil_div(p, 32), nullptr, nullptr, nullptr, nullptr};
  const size_t lds = ps_lds_bytes(p);
  // as many workgroups as the chip holds at once (256 compute units of 160 KB of LDS and 2 such workgroups), and no more than have work
  const int64_t per_cu = std::min<int64_t>(2, std::max<int64_t>(1, (int64_t)((size_t)160 * 1024 / lds)));
  const int64_t work = ceil_div(a.n_chunks + a.n_long, kPsWaves) + ceil_div(a.n_mid - a.n_long, kPsGroups) +
                       ceil_div(a.n_cols - a.n_mid, kPsColThreads / kPsFew);
  const int64_t blocks = std::min<int64_t>(256 * per_cu, std::max<int64_t>(1, work));
  const int64_t hub_blocks = a.n_hub > 0 ? kPsHubBlocks : 0, rows = blocks + hub_blocks;
  const int64_t pair_words = (int64_t)p * a.pw, hub_words = a.n_hub * a.pw, words = 3 * (int64_t)p + 2;
  PinnedPage page;
  GCN_TRY(page.take(sc));
  DevBuf bits, partial;
  GCN_TRY(bits.alloc(sc, sizeof(uint32_t) * (size_t)(pair_words + hub_words + 1)));
  GCN_TRY(partial.alloc(sc, sizeof(uint32_t) * (size_t)(rows * words)));
  a.pair = bits.as<uint32_t>();
  a.hub_bits = a.pair + pair_words;
  a.bad = (int*)(a.hub_bits + hub_words);
  a.partial = partial.as<uint32_t>();
  k_ps_clear<<<ps_grid(std::max<int64_t>(p, pair_words + hub_words)), kPsThreads, 0, s>>>(o, p, a.pair, pair_words + hub_words, a.bad);
  auto kern = p <= kPsPairLds ? k_ps_columns<true> : k_ps_columns<false>;
  GCN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  kern<<<(unsigned)blocks, kPsColThreads, lds, s>>>(a);
  if (hub_blocks) k_ps_hubs<<<(unsigned)hub_blocks, kPsColThreads, sizeof(uint32_t) * (size_t)words, s>>>(a, blocks);
  const int sum_blocks = (int)ceil_div(words, kPsThreads);
  k_ps_finish<<<dim3((unsigned)(sum_blocks + ceil_div(p, kPsThreads)), kPsSplit), kPsThreads, 0, s>>>(a.partial, rows, sum_blocks, a.pair, p, a.pw, o);
  GCN_CHECK_LAUNCH();
  GCN_HIP(hipMemcpyAsync(page.p, a.bad, sizeof(int), hipMemcpyDeviceToHost, s));
  GCN_HIP(hipStreamSynchronize(s));      // the temporaries go back on return
  if (*(const int*)page.p) {
    k_ps_clear<<<ps_grid(p), kPsThreads, 0, s>>>(o, p, nullptr, 0, a.bad);
    GCN_CHECK_LAUNCH();
    return fail(GCN_EINVAL, "gcn_partition_stats: a part id lies outside [0, p)");
  }
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
  if (A->colptr && p <= kPsMaxParts && !tune().partition_sort) return count_by_columns(A, d_part, p, o, sc);

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
