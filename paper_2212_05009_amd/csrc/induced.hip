// gcn_csr_induced: the normalised adjacency of the subgraph induced by a vertex list, built on the
// device from a whole-graph handle (Sec. 4.3.3: a mini-batch is a subgraph G' = (V', E') of the input
// graph, and convolutions run on it as they do on the whole graph in full-batch training).
//
// The subgraph is a graph of its own: vertex k is vertices[k], its edges are the stored entries
// (vertices[a], vertices[b]) of the parent, and degrees, self-loops and D^-1/2 (A'+I) D^-1/2 are
// those of the subgraph.  Two ways, the same arrays:
//   row by row   the parent's selected rows and columns, each filtered and sorted by itself, two passes over them;
//   by keys      the entries of the selected rows whose columns are selected too become (row, column) keys in subgraph
//                numbering, one pass over those rows, and the keys go through the builder's second half, so sorting,
//                normalisation and the column-major copy are the builder's.
#include <algorithm>
#include <new>
#include <type_traits>

#include "common.h"

namespace gcn {

constexpr int kIndThreads = 256;
static inline dim3 ind_grid(int64_t n) { return fold_grid(ceil_div(n > 0 ? n : 1, kIndThreads)); }

// lid[v] = -1 for every vertex of the parent; the flags and the number of keys (the diagonals come first)
__global__ void k_ind_init(int32_t* __restrict__ lid, int64_t n, int64_t n_sub, int* __restrict__ bad, int64_t* __restrict__ cursor, int cursors) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < n) lid[i] = -1;
  if (i == 0) bad[0] = bad[1] = 0;
  if (i < cursors) cursor[i] = n_sub;
}

// lid[vertices[k]] = k; ids out of range are reported, never used as an index
__global__ void k_ind_scatter(const int32_t* __restrict__ vertices, int64_t n_sub, int64_t n,
                              int32_t* __restrict__ lid, int* __restrict__ bad) {
  int64_t k = block_id() * blockDim.x + threadIdx.x;
  if (k >= n_sub) return;
  const int32_t v = vertices[k];
  if (v < 0 || v >= n) { bad[0] = 1; return; }
  lid[v] = (int32_t)k;
}

// (an id outside the graph has been reported: it counts for no entry here)
// a vertex listed twice keeps one of its two positions in lid: the other one sees a mismatch.
// Also the number of stored entries of each selected row.
__global__ void k_ind_rows(const int32_t* __restrict__ vertices, int64_t n_sub, int64_t n, const int32_t* __restrict__ lid,
                           const int64_t* __restrict__ rowptr, uint32_t* __restrict__ len, int* __restrict__ bad) {
  int64_t k = block_id() * blockDim.x + threadIdx.x;
  if (k >= n_sub) return;
  const int32_t v = vertices[k];
  if (v < 0 || v >= n) { len[k] = 0u; return; }
  if (lid[v] != (int32_t)k) bad[1] = 1;
  len[k] = (uint32_t)(rowptr[v + 1] - rowptr[v]);
}

// Keys of the diagonal, then of every entry of the selected rows whose column is selected too (order within the list does
// not matter: it is sorted, and no key occurs twice).  A block takes kIndTile consecutive entries of the selected rows; every
// row holds its diagonal, so they lie in at most as many rows, whose offsets fit LDS.  What is kept of a block leaves in
// one piece, one addition to the cursor per block: with every entry in the list (those not selected as self-loops, which
// the builder drops) a mini-batch of 20 K of 2^18 vertices sorted 914 K keys instead of 106 K.
constexpr int kIndItems = 8;
constexpr int kIndTile = kIndThreads * kIndItems;
__global__ __launch_bounds__(kIndThreads) void k_ind_keys(const int32_t* __restrict__ vertices, int64_t n_sub,
                                                          const int64_t* __restrict__ off, int64_t total, int64_t nb,
                                                          const int64_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                                          const int32_t* __restrict__ lid, int colbits,
                                                          uint64_t* __restrict__ keys, int64_t* __restrict__ cursor) {
  const int64_t blk = block_id();
  if (blk >= nb) return;
  for (int64_t k = blk * kIndThreads + threadIdx.x; k < n_sub; k += nb * kIndThreads) keys[k] = ((uint64_t)k << colbits) | (uint64_t)k;
  __shared__ int row_off[kIndTile + 1];              // first entry of row lo + i, counted from the block's first
  __shared__ int64_t row_pos[kIndTile + 1];          // where entry t0 + t of row lo + i is stored, less t
  __shared__ uint32_t wave_cnt[kIndItems][kIndThreads / 64];
  __shared__ int64_t base;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t t0 = blk * kIndTile, t1 = t0 + kIndTile < total ? t0 + kIndTile : total;
  int64_t lo = 0, hi = n_sub;                        // selected row lo: the last one with off[lo] <= t0 (64 probes a step)
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + 63) >> 6, at = lo + lane * step;
    const int below = __popcll(__ballot(at < hi && off[at < hi ? at : lo] <= t0));
    lo += (below - 1) * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  const int rows = (int)(n_sub - lo < kIndTile + 1 ? n_sub - lo : kIndTile + 1);
  for (int i = threadIdx.x; i < rows; i += kIndThreads) {
    const int64_t o = off[lo + i] - t0;
    row_off[i] = (int)(o < -1 ? -1 : o > kIndTile ? kIndTile : o);
    if (o < kIndTile) row_pos[i] = rowptr[vertices[lo + i]] - o;
  }
  __syncthreads();
  // the requests of all items are in flight together: columns, then their numbers in the subgraph
  int row[kIndItems], at[kIndItems];
#pragma unroll
  for (int i = 0; i < kIndItems; ++i) {
    const int t = i * kIndThreads + threadIdx.x;
    int a = 0, b = t0 + t < t1 ? rows : 1;           // row lo + a: the last one that starts at or before t
    while (b - a > 1) {
      const int m = (a + b) >> 1;
      if (row_off[m] <= t) a = m; else b = m;
    }
    row[i] = a;
  }
#pragma unroll
  for (int i = 0; i < kIndItems; ++i) {
    const int t = i * kIndThreads + threadIdx.x;
    at[i] = t0 + t < t1 ? col[row_pos[row[i]] + t] : -1;
  }
#pragma unroll
  for (int i = 0; i < kIndItems; ++i) at[i] = at[i] >= 0 ? lid[at[i]] : -1;
  uint64_t key[kIndItems];
  uint64_t kept[kIndItems];
#pragma unroll
  for (int i = 0; i < kIndItems; ++i) {
    const uint64_t r = (uint64_t)(lo + row[i]);
    key[i] = (r << colbits) | (uint64_t)(uint32_t)at[i];
    kept[i] = __ballot(at[i] >= 0 && (uint64_t)(uint32_t)at[i] != r);
    if (lane == 0) wave_cnt[i][w] = (uint32_t)__popcll(kept[i]);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t run = 0;
    for (int i = 0; i < kIndItems; ++i)
      for (int j = 0; j < kIndThreads / 64; ++j) { const uint32_t c = wave_cnt[i][j]; wave_cnt[i][j] = run; run += c; }
    base = run ? (int64_t)atomicAdd((unsigned long long*)cursor, (unsigned long long)run) : 0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kIndItems; ++i)
    if ((kept[i] >> lane) & 1ull) keys[base + wave_cnt[i][w] + __popcll(kept[i] & ((1ull << lane) - 1ull))] = key[i];
}

// ---- row by row ------------------------------------------------------------------------------------------------------
// A parent with both copies: the rows (columns) of the subgraph are what is left of the parent's selected rows (columns), each sorted by
// itself.  Two passes over them, one that counts and one that sorts and writes, with the call's wait for the number of entries between:
// seven launches and two waits up to the schedules' read-back, where making keys and sorting them by radix, twice, took 28 and three.  20 K of 2^18
// R-MAT vertices, training step included: 398 -> 286 us (count 20, fill 36; the sorts, counts and copies they replace 190).
//
// A block takes the rows of one side, kIndLanes lanes each (a step of the chain vertex, ends, columns, numbers in the subgraph serves up to 64
// entries), then those of up to kIndWave entries with a wavefront each, then the longer ones, cut into pieces of kIndWave entries, a wavefront
// each.  What is kept of a row is ranked by comparing all pairs, out of LDS, up to kIndRank entries; longer lists are marked in a bitmap of
// the subgraph's vertices, whose set bits are the sorted list (at most 2^20 vertices: 128 KB of LDS; several rows at a time where their bitmaps fit
// 32 KB).
constexpr int kIndLanes = 16, kIndShort = 64;              // lanes of a short row; its entries
constexpr int kIndWave = 1024;                             // entries that a wavefront takes of a row
constexpr int kIndRank = 256;
// A block with more pieces than these, and one more for every 1024 vertices, leaves its hub rows to launches of their own, whose blocks share the
// pieces of every such row: the call would wait for that one block, 1.1 us a piece in both passes.  Us with the pieces of a block as they come / this way /
// by keys: the 1000 vertices of 2^20 R-MAT ones with the longest rows, longest first 1738 / 375 / 520, in random order 741 / 347 / 526; 20 K of 2^18
// 871 / 406 / 661, 405 / 395 / 670; random ones 119 / 118 / 204.  Leaving every hub row to them costs a launch and a longer chain of requests
// where none is that long (134).  Slower than by keys: 20 K of 2.45 M, longest first, 50 M entries of which few stay, 5177 / 2727 / 2141 (columns are
// read too, and both twice).
constexpr int kIndOver = 96, kIndShare = 16;               // (blocks that share a row)
static_assert(kIndOver >= 32 * kHubRowNnz / kIndWave, "what a block keeps is fewer pieces");
constexpr int kIndU = 8;                                   // entries a lane asks for together
// The number of entries is added up on so many words, whose sum the host takes: additions to one word are 14 ns each, one after the other
constexpr int kIndSums = 128;
constexpr int64_t kIndMaxSub = (int64_t)1 << 20;
// Up to here a block adds up the counts before its rows itself (128 KB out of L2 at most): a scan is a launch of 12 us.  Bitmaps of more vertices
// leave room for few blocks on a compute unit: the rows that take one are then done by a launch of their own.
constexpr int64_t kIndOwnOffsets = (int64_t)1 << 15;
constexpr int kIndThreadsRows = 512, kIndMany = 1024;
constexpr int kIndWaves = kIndThreadsRows / 64, kIndJobs = kIndThreadsRows / kIndLanes;      // of a block: wavefronts, rows
// staging: 64 entries a row, or kIndRank a wavefront
constexpr size_t kIndStage = sizeof(int32_t) * kIndJobs * kIndShort;
static_assert(kIndStage == sizeof(int32_t) * kIndWaves * kIndRank, "one staging area");

struct IndRows {
  const int32_t* vertices; int64_t n_sub, n; const int32_t* lid;
  const int64_t* ptr[2]; const int32_t* idx[2];            // the parent's rows, then its columns
  int64_t blocks; int sides;                               // blocks of a side
  uint32_t* cnt; int64_t cnt_ld;                           // [sides][cnt_ld] entries kept; sides start on 16 bytes
  int32_t* deg; float* dinv;
  int* bad; int64_t* nnz;
  int64_t* out_ptr[2]; int scanned;                        // (scanned: out_ptr holds the sums already)
  int32_t* out_idx[2]; float* out_val[2];
  int maps;                                                // bitmaps side by side, a power of two up to the wavefronts
  // rows that take one, where they are done by themselves: kIndSums lists of up to map_ld
  int64_t* map_list; int64_t map_ld; int* map_count;
  // hub rows left over by the counting blocks: their number, [rows], and of each the pieces counted (from bit 40 on) and entries kept
  int64_t* n_over; int64_t* over; unsigned long long* over_kept; int64_t max_over;
  int hubs_listed;                                         // every hub row is left to k_ind_maps
};

// a row of the parent: its ends
struct IndJob { int64_t s, len; };
__device__ __forceinline__ IndJob ind_job(const IndRows& a, int side, int64_t k) {
  IndJob j{0, 0};
  if (k >= a.n_sub) return j;
  const int32_t v = a.vertices[k];
  if (v < 0 || v >= a.n) return j;                         // (reported: it has no entries here)
  j.s = a.ptr[side][v];
  j.len = a.ptr[side][v + 1] - j.s;
  return j;
}
// entries e0 + 64 u + lane of a row, of which those below `end` are asked for: their numbers in the subgraph, or -1
__device__ __forceinline__ void ind_entries(const int32_t* __restrict__ idx, const int32_t* __restrict__ lid, int64_t s, int64_t e0, int64_t end,
                                            int lane, int32_t (&c)[kIndU]) {
#pragma unroll
  for (int u = 0; u < kIndU; ++u) {
    const int64_t e = e0 + 64 * u + lane;
    c[u] = e < end ? idx[s + e] : -1;
  }
#pragma unroll
  for (int u = 0; u < kIndU; ++u) c[u] = c[u] >= 0 ? lid[c[u]] : -1;
}

constexpr uint32_t kIndHub = 0xffffffffu;                  // in the place of a count
__device__ __forceinline__ void ind_counted(const IndRows& a, int side, int64_t k, uint32_t n) {
  a.cnt[side * a.cnt_ld + k] = n;
  if (side == 0) { a.deg[k] = (int32_t)n; a.dinv[k] = inv_sqrt_deg(n > 0 ? (int32_t)n : 1); }
}

__global__ __launch_bounds__(kIndThreadsRows) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ind_count(IndRows a) {
  __shared__ uint32_t kept[kIndJobs];
  __shared__ int pieces[kIndJobs + 1];                     // (rows in pieces, their number; then a running sum)
  __shared__ int piece_job[kIndJobs];
  __shared__ int n_rows;
  __shared__ IndJob ends[kIndJobs];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = threadIdx.x / kIndLanes, l = threadIdx.x % kIndLanes;
  const int64_t blk = block_id();
  if (blk >= a.sides * a.blocks) return;
  const int side = blk >= a.blocks ? 1 : 0;
  const int64_t k0 = (blk - side * a.blocks) * kIndJobs;
  if (threadIdx.x == 0) n_rows = 0;
  if (threadIdx.x < kIndJobs) kept[threadIdx.x] = 0u;
  __syncthreads();
  {
    const int64_t k = k0 + g;
    const IndJob j = ind_job(a, side, k);
    if (k < a.n_sub && l == 0 && side == 0) {
      const int32_t v = a.vertices[k];
      if (v >= 0 && v < a.n && a.lid[v] != (int32_t)k) a.bad[1] = 1;         // listed twice: one of its places is not in lid
    }
    if (j.len > kIndShort) {
      if (l == 0) {
        ends[g] = j;
        const int at = atomicAdd(&n_rows, 1);
        piece_job[at] = g;
        pieces[at] = (int)((j.len + kIndWave - 1) / kIndWave);
      }
    } else {
      int32_t c[kIndShort / kIndLanes];
#pragma unroll
      for (int u = 0; u < kIndShort / kIndLanes; ++u) {
        const int e = u * kIndLanes + l;
        c[u] = e < j.len ? a.idx[side][j.s + e] : -1;
      }
      uint32_t n = 0;
#pragma unroll
      for (int u = 0; u < kIndShort / kIndLanes; ++u) n += c[u] >= 0 && a.lid[c[u]] >= 0 ? 1u : 0u;
#pragma unroll
      for (int o = 1; o < kIndLanes; o <<= 1) n += __shfl_xor(n, o, kIndLanes);
      if (l == 0) kept[g] = n;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < n_rows; ++i) { const int c = pieces[i]; pieces[i] = run; run += c; }
    pieces[n_rows] = run;
  }
  __syncthreads();
  const bool over = pieces[n_rows] > kIndOver + (int)(a.n_sub >> 10);
  for (int i = w, row = 0; i < pieces[n_rows]; i += kIndWaves) {
    while (pieces[row + 1] <= i) ++row;
    const int at = piece_job[row];
    const IndJob j = ends[at];
    if (over && j.len > kHubRowNnz) {
      if (i == pieces[row] && lane == 0) {
        kept[at] = kIndHub;
        const int64_t to = (int64_t)atomicAdd(reinterpret_cast<unsigned long long*>(a.n_over), 1ull);
        if (to < a.max_over) a.over[to] = side * a.n_sub + k0 + at;            // (more only of a vertex listed again)
      }
      continue;
    }
    const int64_t e_lo = (int64_t)(i - pieces[row]) * kIndWave, e_hi = e_lo + kIndWave < j.len ? e_lo + kIndWave : j.len;
    uint32_t n = 0;
    for (int64_t e0 = e_lo; e0 < e_hi; e0 += 64 * kIndU) {
      int32_t c[kIndU];
      ind_entries(a.idx[side], a.lid, j.s, e0, e_hi, lane, c);
#pragma unroll
      for (int u = 0; u < kIndU; ++u) n += c[u] >= 0 ? 1u : 0u;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0) atomicAdd(&kept[at], n);
  }
  __syncthreads();
  if (w == 0) {
    static_assert(kIndJobs <= 64, "a row per lane");
    const int64_t k = k0 + lane;
    const bool mine = lane < kIndJobs && k < a.n_sub && kept[lane] != kIndHub;
    uint32_t n = mine ? kept[lane] : 0u;
    if (mine) ind_counted(a, side, k, n);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0 && side == 0) atomicAdd(reinterpret_cast<unsigned long long*>(a.nnz + blk % kIndSums), (unsigned long long)n);
  }
}

// The hub rows left over: whoever counts a row's last piece writes its number down.
__global__ __launch_bounds__(kIndThreadsRows) void k_ind_count_over(IndRows a, int64_t rows) {
  const int lane = threadIdx.x & 63;
  for (int64_t r = blockIdx.x; r < rows; r += gridDim.x) {
    const int64_t job = a.over[r], side = job >= a.n_sub ? 1 : 0, k = job - side * a.n_sub;
    const IndJob j = ind_job(a, (int)side, k);
    const int64_t pieces = (j.len + kIndWave - 1) / kIndWave;
    uint32_t n = 0;
    int64_t done = 0;
    for (int64_t p = (int64_t)blockIdx.y * kIndWaves + (threadIdx.x >> 6); p < pieces; p += kIndShare * kIndWaves, ++done) {
      const int64_t e_hi = (p + 1) * kIndWave < j.len ? (p + 1) * kIndWave : j.len;
      for (int64_t e0 = p * kIndWave; e0 < e_hi; e0 += 64 * kIndU) {
        int32_t c[kIndU];
        ind_entries(a.idx[side], a.lid, j.s, e0, e_hi, lane, c);
#pragma unroll
        for (int u = 0; u < kIndU; ++u) n += c[u] >= 0 ? 1u : 0u;
      }
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) n += __shfl_xor(n, o, 64);
    if (lane == 0 && done > 0) {
      typedef unsigned long long u64;
      const u64 mine = ((u64)done << 40) + n, now = atomicAdd(a.over_kept + r, mine) + mine;
      if ((int64_t)(now >> 40) == pieces) {
        const uint32_t all = (uint32_t)(now & (((u64)1 << 40) - 1));
        ind_counted(a, (int)side, k, all);
        if (side == 0) atomicAdd(reinterpret_cast<u64*>(a.nnz + k % kIndSums), (u64)all);
      }
    }
  }
}

// An entry of a row at place `at`; its value is the product of the same two factors on both sides.
__device__ __forceinline__ void ind_put(const IndRows& a, int side, float dk, int64_t at, int32_t v) {
  a.out_idx[side][at] = v;
  a.out_val[side][at] = __fmul_rn(dk, a.dinv[v]);
}

struct IndMapRow { IndJob ends; int64_t first, k; int side; };
// `rows` rows side by side (written by threads of the block before), each with its bitmap: their pieces go round the wavefronts, then each bitmap
// is read by its share of them.
template <int THREADS>
__device__ __forceinline__ void ind_maps(const IndRows& a, uint32_t* __restrict__ maps, const IndMapRow* row, int rows) {
  constexpr int kWaves = THREADS / 64;
  __shared__ int pieces[kWaves + 1];
  __shared__ uint32_t wave_sum[kWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int words = (int)((a.n_sub + 31) >> 5), per_map = kWaves / a.maps;
  for (int q = threadIdx.x; q < rows * words; q += THREADS) maps[q] = 0u;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int r = 0; r < rows; ++r) {
      pieces[r] = run;
      run += (int)((row[r].ends.len + kIndWave - 1) / kIndWave);
    }
    pieces[rows] = run;
  }
  __syncthreads();
  for (int i = w, r = 0; i < pieces[rows]; i += kWaves) {
    while (pieces[r + 1] <= i) ++r;
    const IndJob j = row[r].ends;
    uint32_t* __restrict__ map = maps + r * words;
    const int64_t e_lo = (int64_t)(i - pieces[r]) * kIndWave, e_hi = e_lo + kIndWave < j.len ? e_lo + kIndWave : j.len;
    for (int64_t e0 = e_lo; e0 < e_hi; e0 += 64 * kIndU) {
      int32_t c[kIndU];
      ind_entries(a.idx[row[r].side], a.lid, j.s, e0, e_hi, lane, c);
#pragma unroll
      for (int u = 0; u < kIndU; ++u)
        if (c[u] >= 0) atomicOr(&map[c[u] >> 5], 1u << (c[u] & 31));
    }
  }
  __syncthreads();
  // the words of a wavefront are consecutive: 64 at a time, a word per lane
  const int r = w / per_map, part = w % per_map;
  const uint32_t* __restrict__ map = maps + r * words;
  const int share = (words + 64 * per_map - 1) / (64 * per_map) * 64;
  const int w0 = part * share, w1 = r < rows ? (w0 + share < words ? w0 + share : words) : 0;
  uint32_t mine = 0;
  for (int q = w0 + lane; q < w1; q += 64) mine += (uint32_t)__popc(map[q]);
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) mine += __shfl_xor(mine, o, 64);
  if (lane == 0) wave_sum[w] = mine;
  __syncthreads();
  if (r < rows) {
    int64_t at = row[r].first;
    const float dk = a.dinv[row[r].k];
    for (int q = r * per_map; q < w; ++q) at += wave_sum[q];
    for (int q0 = w0; q0 < w1; q0 += 64) {
      const int q = q0 + lane;
      uint32_t bits = q < w1 ? map[q] : 0u;
      uint32_t inc = (uint32_t)__popc(bits);
      const uint32_t own = inc;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t x = __shfl_up(inc, o, 64);
        if (lane >= o) inc += x;
      }
      int64_t to = at + (inc - own);
      for (; bits; bits &= bits - 1) ind_put(a, row[r].side, dk, to++, q * 32 + __ffs(bits) - 1);
      at += __shfl(inc, 63, 64);
    }
  }
  __syncthreads();
}

// MAPS: the rows that take a bitmap are done here too, but for listed hub rows; else they are listed for k_ind_maps.
template <bool MAPS>
__global__ __launch_bounds__(kIndThreadsRows) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ind_fill(IndRows a) {
  extern __shared__ __align__(16) int32_t ind_lds[];                     // staging, then the bitmaps
  __shared__ int64_t offset[kIndJobs];                 // first entry of a row of the block
  __shared__ uint32_t kept[kIndJobs];
  __shared__ int wave_rows[kIndJobs], map_rows[kIndJobs];
  __shared__ IndMapRow row[kIndWaves];
  __shared__ int n_wave, n_map;
  __shared__ IndJob ends[kIndJobs];
  __shared__ uint64_t before[kIndWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = threadIdx.x / kIndLanes, l = threadIdx.x % kIndLanes;
  const int64_t blk = block_id();
  if (blk >= a.sides * a.blocks) return;
  const int side = blk >= a.blocks ? 1 : 0;
  const int64_t k0 = (blk - side * a.blocks) * kIndJobs;
  const uint32_t* __restrict__ cnt = a.cnt + side * a.cnt_ld;
  if (threadIdx.x == 0) n_wave = n_map = 0;
  {
    uint64_t sum = 0;
    static_assert(kIndJobs % 4 == 0, "whole requests before the first row");
    if (!a.scanned)
#pragma unroll 4
      for (int64_t k = 4 * threadIdx.x; k < k0; k += 4 * kIndThreadsRows) {
        const uint4 x = *reinterpret_cast<const uint4*>(cnt + k);
        sum += (uint64_t)x.x + x.y + x.z + x.w;
      }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) before[w] = sum;
  }
  __syncthreads();
  if (w == 0) {
    const int64_t k = k0 + lane;
    const bool mine = lane < kIndJobs && k < a.n_sub;
    const uint32_t own = mine ? cnt[k] : 0u;
    uint64_t inc = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint64_t x = __shfl_up(inc, o, 64);
      if (lane >= o) inc += x;
    }
    uint64_t base = 0;
    if (a.scanned) base = (uint64_t)a.out_ptr[side][k0];
    else
      for (int i = 0; i < kIndWaves; ++i) base += before[i];
    if (mine) {
      kept[lane] = own;
      offset[lane] = (int64_t)(base + inc - own);
    }
    if (!a.scanned && mine) {
      a.out_ptr[side][k] = (int64_t)(base + inc - own);
      if (k == a.n_sub - 1) a.out_ptr[side][a.n_sub] = (int64_t)(base + inc);
    }
  }
  __syncthreads();
  auto put = [&](float dk, int64_t at, int32_t v) { ind_put(a, side, dk, at, v); };
  auto order = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // the n numbers of a list, up to four a lane, to their places: as many of them are smaller (four a read; behind the list lies what is not)
  auto rank = [&](const int32_t* __restrict__ list, int n, int me, auto lanes, float dk, int64_t first) {
    constexpr int LANES = decltype(lanes)::value;
    int32_t v[4];
    int at[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = me + LANES * i < n ? list[me + LANES * i] : 0;
    for (int q = 0; q < n; q += 4) {
      const int4 x = *reinterpret_cast<const int4*>(list + q);
      const int in = n - q;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        at[i] += (x.x < v[i] ? 1 : 0) + (in > 1 && x.y < v[i] ? 1 : 0) + (in > 2 && x.z < v[i] ? 1 : 0) + (in > 3 && x.w < v[i] ? 1 : 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (me + LANES * i < n) put(dk, first + at[i], v[i]);
  };
  {
    const int64_t k = k0 + g;
    const IndJob j = ind_job(a, side, k);
    if (j.len > kIndShort) {
      if (l == 0) {
        ends[g] = j;
        // (neighbours, which may all be long, in different ones; so too a vertex's row and its column)
        const int list = (int)((k + side * (kIndSums / 2)) % kIndSums);
        if (j.len <= kIndWave && kept[g] <= kIndRank) wave_rows[atomicAdd(&n_wave, 1)] = g;
        else if (MAPS && !(a.hubs_listed && j.len > kHubRowNnz)) map_rows[atomicAdd(&n_map, 1)] = g;
        else a.map_list[list * a.map_ld + atomicAdd(&a.map_count[list], 1)] = side * a.n_sub + k;
      }
    } else if (j.len > 0) {
      int32_t* stage = ind_lds + g * kIndShort;
      int32_t c[kIndShort / kIndLanes];
#pragma unroll
      for (int u = 0; u < kIndShort / kIndLanes; ++u) {
        const int e = u * kIndLanes + l;
        c[u] = e < j.len ? a.idx[side][j.s + e] : -1;
      }
      const float dk = a.dinv[k];
      int n = 0;
#pragma unroll
      for (int u = 0; u < kIndShort / kIndLanes; ++u) c[u] = c[u] >= 0 ? a.lid[c[u]] : -1;
#pragma unroll
      for (int u = 0; u < kIndShort / kIndLanes; ++u) {
        const uint32_t some = (uint32_t)(__ballot(c[u] >= 0) >> (lane & ~(kIndLanes - 1))) & ((1u << kIndLanes) - 1u);
        if (c[u] >= 0) stage[n + __popc(some & ((1u << l) - 1u))] = c[u];
        n += __popc(some);
      }
      order();
      rank(stage, n, l, std::integral_constant<int, kIndLanes>(), dk, offset[g]);
    }
  }
  __syncthreads();
  for (int i = w; i < n_wave; i += kIndWaves) {
    const int at = wave_rows[i];
    const IndJob j = ends[at];
    int32_t* stage = ind_lds + w * kIndRank;
    const float dk = a.dinv[k0 + at];
    int n = 0;
    for (int64_t e0 = 0; e0 < j.len; e0 += 64 * kIndU) {
      int32_t c[kIndU];
      ind_entries(a.idx[side], a.lid, j.s, e0, j.len, lane, c);
#pragma unroll
      for (int u = 0; u < kIndU; ++u) {
        const uint64_t some = __ballot(c[u] >= 0);
        const int to = n + __popcll(some & ((1ull << lane) - 1ull));
        if (c[u] >= 0 && to < kIndRank) stage[to] = c[u];
        n += __popcll(some);
      }
    }
    n = n < kIndRank ? n : kIndRank;
    order();
    rank(stage, n, lane, std::integral_constant<int, 64>(), dk, offset[at]);
    order();
  }
  if constexpr (MAPS) {
    uint32_t* maps = reinterpret_cast<uint32_t*>(ind_lds) + kIndStage / sizeof(int32_t);
    for (int i0 = 0; i0 < n_map; i0 += a.maps) {
      const int rows = n_map - i0 < a.maps ? n_map - i0 : a.maps;
      if (threadIdx.x < rows) {
        const int at = map_rows[i0 + threadIdx.x];
        row[threadIdx.x] = IndMapRow{ends[at], offset[at], k0 + at, side};
      }
      ind_maps<kIndThreadsRows>(a, maps, row, rows);
    }
  }
}

// The rows left over by k_ind_fill: hub rows, and those whose bitmaps leave room for few blocks on a compute unit
__global__ __launch_bounds__(kIndMany) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_ind_maps(IndRows a) {
  extern __shared__ __align__(16) int32_t ind_lds[];
  __shared__ IndMapRow row[kIndMany / 64];
  const int list = (int)blockIdx.x % kIndSums;
  const int64_t total = a.map_count[list];
  for (int64_t i0 = (int64_t)(blockIdx.x / kIndSums) * a.maps; i0 < total; i0 += (int64_t)(gridDim.x / kIndSums) * a.maps) {
    const int rows = (int)(total - i0 < a.maps ? total - i0 : a.maps);
    if (threadIdx.x < rows) {
      const int64_t job = a.map_list[list * a.map_ld + i0 + threadIdx.x];
      const int side = job >= a.n_sub ? 1 : 0;
      const int64_t k = job - side * a.n_sub;
      row[threadIdx.x] = IndMapRow{ind_job(a, side, k), a.out_ptr[side][k], k, side};
    }
    ind_maps<kIndMany>(a, reinterpret_cast<uint32_t*>(ind_lds), row, rows);
  }
}

__global__ void k_ind_giant(const int32_t* __restrict__ vertices, int64_t n_sub, int64_t n, const int64_t* __restrict__ ptr,
                            const int64_t* __restrict__ ptr_t, int64_t most, int64_t* __restrict__ host) {
  const int64_t k = block_id() * blockDim.x + threadIdx.x;
  if (k >= n_sub) return;
  const int32_t v = vertices[k];
  if (v < 0 || v >= n) return;                             // (reported by the passes)
  if (ptr[v + 1] - ptr[v] > most || (ptr_t && ptr_t[v + 1] - ptr_t[v] > most)) *host = 1;
}

// Of a parent that has giant rows: is one of them selected?  A launch and a wait, 10 us.  The list of such a row is written by one block: 2000 of 2^18
// vertices with one row of all of them 195 us by keys, 20 K of 2^22 330, in one block with its counting 320 and 4612.
static int giant_selected(const gcn_csr_t* A, const int32_t* d_vertices, int64_t n_sub, int flags, hipStream_t s, bool* yes) {
  CallScope sc(s);
  PinnedPage page;
  GCN_TRY(page.take(sc));
  int64_t* word = page.words();
  *word = 0;
  k_ind_giant<<<ind_grid(n_sub), kIndThreads, 0, s>>>(d_vertices, n_sub, A->nr, A->rowptr, (flags & GCN_BUILD_CSC) ? A->colptr : nullptr,
                                                       (int64_t)kGiantChunks * kHubChunkNnz, word);
  GCN_CHECK_LAUNCH();
  GCN_HIP(hipStreamSynchronize(s));
  sc.done = true;
  *yes = *(volatile int64_t*)word != 0;
  return GCN_OK;
}

static int induced_by_rows(const gcn_csr_t* A, const int32_t* d_vertices, int64_t n_sub, int flags, hipStream_t s, gcn_csr* B) {
  const int64_t n = A->nr;
  const int sides = (flags & GCN_BUILD_CSC) ? 2 : 1;
  const int64_t n_hubs = A->sched.n_hub_rows + (sides == 2 ? A->sched_t.n_hub_rows : 0);
  CallScope sc(s);
  DevBuf lid, cnt, dinv, words, tmp, rowptr, colptr, deg, halo_gid;
  GCN_TRY(lid.alloc(sc, sizeof(int32_t) * (size_t)n));
  GCN_TRY(cnt.alloc(sc, sizeof(uint32_t) * (size_t)(sides * round_up(n_sub, 4))));
  GCN_TRY(dinv.alloc(sc, sizeof(float) * (size_t)n_sub));
  GCN_TRY(words.alloc(sc, (2 + 2 * kIndSums + n_hubs) * sizeof(int64_t)));  // flags; rows left over; entries, in parts; listed rows; entries of rows left over
  GCN_TRY(rowptr.alloc(sc, sizeof(int64_t) * (size_t)(n_sub + 1)));
  if (sides == 2) GCN_TRY(colptr.alloc(sc, sizeof(int64_t) * (size_t)(n_sub + 1)));
  GCN_TRY(deg.alloc(sc, sizeof(int32_t) * (size_t)n_sub));
  GCN_TRY(halo_gid.alloc(sc, sizeof(int32_t)));
  PinnedPage page;
  GCN_TRY(page.take(sc));
  int64_t* read = page.words();
  const int64_t map_bytes = (int64_t)sizeof(uint32_t) * ceil_div(n_sub, 32);
  const bool few = n_sub <= kIndOwnOffsets;
  int maps = (few ? kIndThreadsRows : kIndMany) / 64;
  while (maps > 1 && maps * map_bytes > 32 * 1024) maps /= 2;
  DevBuf map_list;
  const int64_t blocks = ceil_div(n_sub, kIndJobs), map_ld = sides * ceil_div(n_sub, kIndSums);
  DevBuf over;
  GCN_TRY(over.alloc(sc, sizeof(int64_t) * (size_t)(n_hubs + 1)));
  if (!few || n_hubs > 0) GCN_TRY(map_list.alloc(sc, sizeof(int64_t) * (size_t)(kIndSums * map_ld)));
  IndRows a{d_vertices, n_sub, n, lid.as<int32_t>(), {A->rowptr, A->colptr}, {A->col, A->rowidx}, blocks, sides,
            cnt.as<uint32_t>(), round_up(n_sub, 4), deg.as<int32_t>(), dinv.as<float>(), words.as<int>(), words.as<int64_t>() + 2,
            {rowptr.as<int64_t>(), colptr.as<int64_t>()}, !few, {nullptr, nullptr}, {nullptr, nullptr}, maps, map_list.as<int64_t>(), map_ld,
            (int*)(words.as<int64_t>() + 2 + kIndSums), words.as<int64_t>() + 1, over.as<int64_t>(),
            words.as<unsigned long long>() + 2 + 2 * kIndSums, n_hubs, 0};
  const dim3 grid = fold_grid(sides * a.blocks);
  k_ind_init<<<ind_grid(std::max<int64_t>(n, 1 + 2 * kIndSums + n_hubs)), kIndThreads, 0, s>>>(lid.as<int32_t>(), n, 0, a.bad, a.n_over, (int)(1 + 2 * kIndSums + n_hubs));
  k_ind_scatter<<<ind_grid(n_sub), kIndThreads, 0, s>>>(d_vertices, n_sub, n, lid.as<int32_t>(), a.bad);
  k_ind_count<<<grid, kIndThreadsRows, 0, s>>>(a);
  GCN_CHECK_LAUNCH();
  if (a.scanned) GCN_TRY(tmp.alloc(sc, scan_tmp_bytes(n_sub)));
  auto counted = [&]() -> int {
    GCN_HIP(hipMemcpyAsync(read, words.p, (2 + kIndSums) * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    if (a.scanned)
      for (int side = 0; side < sides; ++side) GCN_TRY(exclusive_scan_u32(a.cnt + side * a.cnt_ld, a.out_ptr[side], n_sub, tmp.p, s));
    GCN_HIP(hipStreamSynchronize(s));
    return GCN_OK;
  };
  GCN_TRY(counted());
  const int* h_bad = (const int*)read;
  if (h_bad[0]) return fail(GCN_EINVAL, "gcn_csr_induced: a vertex id lies outside the graph");
  if (h_bad[1]) return fail(GCN_EINVAL, "gcn_csr_induced: a vertex is listed twice");
  if (read[1] > n_hubs) return fail(GCN_EHIP, "gcn_csr_induced: internal error (%lld long rows of %lld)", (long long)read[1], (long long)n_hubs);
  a.hubs_listed = read[1] > 0;
  if (a.hubs_listed) {
    k_ind_count_over<<<dim3((unsigned)std::min<int64_t>(read[1], 1024), kIndShare), kIndThreadsRows, 0, s>>>(a, read[1]);
    GCN_CHECK_LAUNCH();
    GCN_TRY(counted());
  }
  int64_t nnz = 0;
  for (int i = 0; i < kIndSums; ++i) nnz += read[2 + i];
  if (nnz < n_sub) return fail(GCN_EHIP, "gcn_csr_induced: internal error (nnz %lld < rows %lld)", (long long)nnz, (long long)n_sub);

  DevBuf col, val, rowidx, val_t, mid;
  GCN_TRY(col.alloc(sc, sizeof(int32_t) * (size_t)nnz + kEntrySlack));
  GCN_TRY(val.alloc(sc, sizeof(float) * (size_t)nnz + kEntrySlack));
  if (sides == 2) {
    GCN_TRY(rowidx.alloc(sc, sizeof(int32_t) * (size_t)nnz + kEntrySlack));
    GCN_TRY(val_t.alloc(sc, sizeof(float) * (size_t)nnz + kEntrySlack));
  }
  a.out_idx[0] = col.as<int32_t>(); a.out_idx[1] = rowidx.as<int32_t>();
  a.out_val[0] = val.as<float>(); a.out_val[1] = val_t.as<float>();
  const size_t stage = kIndStage, map_lds = (size_t)(maps * map_bytes);
  if (few) k_ind_fill<true><<<grid, kIndThreadsRows, stage + map_lds, s>>>(a);
  else k_ind_fill<false><<<grid, kIndThreadsRows, stage, s>>>(a);
  if (!few || a.hubs_listed) {
    GCN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_ind_maps), hipFuncAttributeMaxDynamicSharedMemorySize, (int)map_lds));
    k_ind_maps<<<dim3(4 * kIndSums), kIndMany, map_lds, s>>>(a);
  }
  GCN_CHECK_LAUNCH();
  HandleArrays h{n_sub, 0, n_sub, 0, nnz, &rowptr, &col, &val, &deg, &halo_gid, &colptr, &rowidx, &val_t, &mid};
  return adopt_arrays(h, sc, page, B);
}

static int induced_by_keys(const gcn_csr_t* A, const int32_t* d_vertices, int64_t n_sub, int flags, hipStream_t s, gcn_csr* B) {
  const int64_t n = A->nr;
  CallScope sc(s);
  DevBuf lid, len, off, tmp;
  GCN_TRY(lid.alloc(sc, sizeof(int32_t) * (size_t)n));
  GCN_TRY(len.alloc(sc, sizeof(uint32_t) * (size_t)n_sub));
  GCN_TRY(off.alloc(sc, sizeof(int64_t) * (size_t)(n_sub + 3)));      // the total, the flags and the cursor behind the offsets
  GCN_TRY(tmp.alloc(sc, scan_tmp_bytes(n_sub)));
  PinnedPage page;
  GCN_TRY(page.take(sc));
  int64_t* read = page.words();
  int* bad = (int*)(off.as<int64_t>() + n_sub + 1);
  int64_t* cursor = off.as<int64_t>() + n_sub + 2;
  k_ind_init<<<ind_grid(n), kIndThreads, 0, s>>>(lid.as<int32_t>(), n, n_sub, bad, cursor, 1);
  k_ind_scatter<<<ind_grid(n_sub), kIndThreads, 0, s>>>(d_vertices, n_sub, n, lid.as<int32_t>(), bad);
  k_ind_rows<<<ind_grid(n_sub), kIndThreads, 0, s>>>(d_vertices, n_sub, n, lid.as<int32_t>(), A->rowptr, len.as<uint32_t>(), bad);
  GCN_CHECK_LAUNCH();
  GCN_TRY(exclusive_scan_u32(len.as<uint32_t>(), off.as<int64_t>(), n_sub, tmp.p, s));
  GCN_HIP(hipMemcpyAsync(read, off.as<int64_t>() + n_sub, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
  GCN_HIP(hipStreamSynchronize(s));
  const int64_t total = read[0];
  const int* h_bad = (const int*)(read + 1);
  if (h_bad[0]) return fail(GCN_EINVAL, "gcn_csr_induced: a vertex id lies outside the graph");
  if (h_bad[1]) return fail(GCN_EINVAL, "gcn_csr_induced: a vertex is listed twice");

  if (total + n_sub >= 0xffffffffLL) return fail(GCN_EINVAL, "gcn_csr_induced: more than 2^32 - 1 entries and rows selected");

  // (total counts the diagonals of the selected rows: a bound on the keys)
  DevBuf keys_a, keys_b, words, halo_gid;
  GCN_TRY(keys_a.alloc(sc, sizeof(uint64_t) * (size_t)total));
  GCN_TRY(keys_b.alloc(sc, sizeof(uint64_t) * (size_t)total));
  GCN_TRY(words.alloc(sc, key_words_bytes(total)));
  GCN_TRY(halo_gid.alloc(sc, sizeof(int32_t)));
  const int64_t nb = ceil_div(total, kIndTile);
  k_ind_keys<<<fold_grid(nb), kIndThreads, 0, s>>>(d_vertices, n_sub, off.as<int64_t>(), total, nb, A->rowptr, A->col, lid.as<int32_t>(),
                                                  key_bits(n_sub), keys_a.as<uint64_t>(), cursor);
  GCN_CHECK_LAUNCH();
  KeyBuild in;
  in.n_global = in.nr = n_sub;
  in.keys_a = &keys_a; in.keys_b = &keys_b; in.words = &words; in.halo_gid = &halo_gid;
  in.m = total; in.count = cursor; in.flags = flags;
  return build_from_keys(in, sc, page, B);
}

}  // namespace gcn

using namespace gcn;

extern "C" int gcn_csr_induced(const gcn_csr_t* A, const int32_t* d_vertices, int64_t n_sub, int flags, void* stream,
                               gcn_csr_t** out) {
  clear_error();
  if (out) *out = nullptr;
  if (!A || !d_vertices || !out) return fail(GCN_EINVAL, "gcn_csr_induced: NULL argument");
  if (A->nh != 0 || A->nr != A->n_global)
    return fail(GCN_EINVAL, "gcn_csr_induced: needs the handle of a whole graph (every row, no halo columns)");
  if (n_sub < 1 || n_sub > A->nr) return fail(GCN_EINVAL, "gcn_csr_induced: need 1 <= n_sub <= number of vertices");
  if (flags & ~GCN_BUILD_CSC) return fail(GCN_EINVAL, "gcn_csr_induced: unknown flag");
  gcn_csr* B = new (std::nothrow) gcn_csr();
  if (!B) return fail(GCN_ENOMEM, "gcn_csr_induced: host allocation failed");
  if (hipGetDevice(&B->device) != hipSuccess) { delete B; return fail(GCN_EHIP, "hipGetDevice failed"); }
  // Row by row, but from a parent without a column-major copy, for subgraphs whose vertices no bitmap in LDS holds, and where many rows take a
  // bitmap of more than 16 KB: 500 K of 1 M vertices, R-MAT rows (one in 60 of 512 entries and more) 962 us by sorting keys, 1200 row by row;
  // uniform rows 1816 and 1330.  131 K of 262 K, R-MAT 1013 and 874.  The table of numbers is asked for four times an entry, by keys once: where it is
  // more than an XCD's L2 holds, R-MAT rows gain up to fewer vertices (of 2.45 M ones 50 K 280 and 268, 65 K 306 and 330, 131 K 387 and 468; of 4 M
  // 65 K 259 and 260, 131 K 335 and 415; of 1.5 M 90 K 335 and 308, 131 K 397 and 420).  Beyond 2^21 vertices uniform rows too, up to some 2e13
  // vertices times entries: 300 K of 2.45 M with 24 each 544 and 517, 400 K 643 and 670, 800 K 1179 and 1335; 400 K of 4 M with 12 498 and 475, 600 K
  // 634 and 684 (of 1.5 M with 24 up to 2^20 vertices 1.1 to 1.5 times as fast).
  const int64_t long_rows = A->sched.class_begin[23] + A->sched.n_hub_rows + (A->colptr ? A->sched_t.class_begin[23] + A->sched_t.n_hub_rows : 0);
  // Nor where a giant row is likely to be among the selected ones (in one call of four).
  const int64_t giants = std::max(A->sched.n_giant_rows, (flags & GCN_BUILD_CSC) && A->colptr ? A->sched_t.n_giant_rows : 0);
  const bool by_rows = (A->colptr || !(flags & GCN_BUILD_CSC)) && n_sub <= kIndMaxSub && A->nnz + n_sub < 0xffffffffLL &&
                       (n_sub <= (A->nr > 1 << 20 ? 1 << 16 : 1 << 17) || long_rows * 200 <= A->nr) && (double)giants * (double)n_sub <= 0.25 * (double)A->nr &&
                       (A->nr <= 1 << 21 || (double)A->nnz * (double)n_sub <= 2e13);
  bool by_keys = !by_rows;
  int rc = GCN_OK;
  if (!by_keys && giants > 0) rc = giant_selected(A, d_vertices, n_sub, flags, (hipStream_t)stream, &by_keys);
  if (!by_keys && rc == GCN_OK) rc = induced_by_rows(A, d_vertices, n_sub, flags, (hipStream_t)stream, B);
  if (by_keys && rc == GCN_OK) rc = induced_by_keys(A, d_vertices, n_sub, flags, (hipStream_t)stream, B);
  if (rc != GCN_OK) { gcn_csr_free(B); return rc; }
  *out = B;
  return GCN_OK;
}
