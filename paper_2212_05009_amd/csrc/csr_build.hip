// gcn_csr_build: normalised adjacency block in CSR (+CSC), halo index list, degree counts and
// the row-binned execution schedules, all built on the device (Sec. 3.1: A^ = D^-1/2 (A+I) D^-1/2;
// Sec. 4.1: the non-owned columns of the block are the rows to receive, each listed once).
#include <algorithm>
#include <new>

#include "common.h"

namespace gcn {

constexpr int kThreads = 256;
static inline dim3 grid_for(int64_t n) { return fold_grid(ceil_div(n > 0 ? n : 1, kThreads)); }

// ---- step 1: id validation ------------------------------------------------------------------
__global__ void k_validate(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                           int64_t n_edges, int64_t n_global, int* __restrict__ bad) {
  int64_t e = block_id() * blockDim.x + threadIdx.x;
  if (e >= n_edges) return;
  int32_t s = src[e], t = dst[e];
  if (s < 0 || s >= n_global || t < 0 || t >= n_global) atomicOr(bad, 1);
}

__global__ void k_validate_deg(const int32_t* __restrict__ deg, int64_t n, int* __restrict__ bad) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < n && deg[i] < 1) atomicOr(bad, 2);
}

// ---- step 2: halo set as a bitmap over global ids -------------------------------------------
__global__ void k_mark_halo(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                            int64_t n_edges, int64_t row_lo, int64_t row_hi,
                            uint32_t* __restrict__ bitmap) {
  int64_t e = block_id() * blockDim.x + threadIdx.x;
  if (e >= n_edges) return;
  int64_t s = src[e], t = dst[e];
  if (s >= row_lo && s < row_hi && (t < row_lo || t >= row_hi))
    atomicOr(&bitmap[t >> 5], 1u << (t & 31));
}

__global__ void k_popc(const uint32_t* __restrict__ bitmap, int64_t words, uint32_t* __restrict__ cnt) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < words) cnt[i] = (uint32_t)__popc(bitmap[i]);
}

__global__ void k_halo_list(const uint32_t* __restrict__ bitmap, const int64_t* __restrict__ wprefix,
                            int64_t words, int32_t* __restrict__ halo_gid) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i >= words) return;
  uint32_t w = bitmap[i];
  int64_t p = wprefix[i];
  while (w) {
    int b = __ffs(w) - 1;
    halo_gid[p++] = (int32_t)(i * 32 + b);
    w &= w - 1;
  }
}

// ---- step 3: (row, local column) keys ---------------------------------------------------------
constexpr uint64_t kInvalidKey = ~0ull;

__global__ void k_make_keys(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                            int64_t n_edges, int64_t row_lo, int64_t row_hi, int64_t nr, int colbits,
                            const uint32_t* __restrict__ bitmap, const int64_t* __restrict__ wprefix,
                            uint64_t* __restrict__ keys, int* __restrict__ bad) {
  int64_t e = block_id() * blockDim.x + threadIdx.x;
  if (e >= n_edges + nr) return;
  if (e >= n_edges) {                      // the diagonal of I, one entry per owned row
    uint64_t i = (uint64_t)(e - n_edges);
    keys[e] = (i << colbits) | i;
    return;
  }
  int64_t s = src[e], t = dst[e];
  uint64_t k = kInvalidKey;
  if (!bitmap) {                           // a whole graph, which has no halo: ids are checked here
    if (s < row_lo || s >= row_hi || t < row_lo || t >= row_hi) atomicOr(bad, 1);
    else if (s != t) k = ((uint64_t)(s - row_lo) << colbits) | (uint64_t)(t - row_lo);
  } else if (s >= row_lo && s < row_hi && s != t) {
    uint64_t lc;
    if (t >= row_lo && t < row_hi) {
      lc = (uint64_t)(t - row_lo);
    } else {
      uint32_t w = bitmap[t >> 5];
      lc = (uint64_t)(nr + wprefix[t >> 5] + __popc(w & ((1u << (t & 31)) - 1u)));
    }
    k = ((uint64_t)(s - row_lo) << colbits) | lc;
  }
  keys[e] = k;
}

// ---- step 4: duplicate removal ------------------------------------------------------------------
// Two passes over the sorted keys with a scan of the blocks' counts between them: flags and positions of every candidate
// in memory cost 28 bytes a key where this reads 16 (keys twice).  m: a bound on the keys, of which there are *count.
constexpr int kUniqItems = 16;
constexpr int kUniqTile = kThreads * kUniqItems;
static_assert(kThreads / 64 * kUniqItems == 64, "k_compact scans the counts of a block's (round, wavefront) pairs in one wavefront");

__device__ __forceinline__ bool first_of_equal(const uint64_t* __restrict__ keys, int64_t k, int64_t m, uint64_t* v, uint64_t* before) {
  if (k >= m) return false;
  *v = keys[k];
  *before = k ? keys[k - 1] : 0;
  return k == 0 || *before != *v;
}

__global__ __launch_bounds__(kThreads) void k_count_unique(const uint64_t* __restrict__ keys, const int64_t* __restrict__ count,
                                                           int64_t nb, uint32_t* __restrict__ cnt) {
  const int64_t blk = block_id();
  if (blk >= nb) return;
  const int64_t m = *count;
  __shared__ uint32_t wave_cnt[kThreads / 64];
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < kUniqItems; ++i) {
    uint64_t v, before;
    c += (uint32_t)__popcll(__ballot(first_of_equal(keys, blk * kUniqTile + i * kThreads + threadIdx.x, m, &v, &before)));
  }
  if ((threadIdx.x & 63) == 0) wave_cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int i = 0; i < kThreads / 64; ++i) tot += wave_cnt[i];
    cnt[blk] = tot;
  }
}

// Also the row pointers: every row holds its diagonal, so a row starts where the row of the key before is another.
__global__ __launch_bounds__(kThreads) void k_compact(const uint64_t* __restrict__ keys, const int64_t* __restrict__ off,
                                                      const int64_t* __restrict__ count, int64_t nb, int colbits, int64_t nnz,
                                                      uint64_t* __restrict__ ukeys, int32_t* __restrict__ col,
                                                      int64_t* __restrict__ rowptr) {
  const int64_t blk = block_id();
  if (blk >= nb) return;
  const int64_t m = *count;
  if (blk * kUniqTile >= m) return;
  __shared__ uint32_t part[64];            // keys kept by round i, wavefront w at [i * waves + w]; then those before it
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint64_t v[kUniqItems], before[kUniqItems];
  uint64_t kept[kUniqItems];
#pragma unroll
  for (int i = 0; i < kUniqItems; ++i) {
    v[i] = before[i] = 0;
    kept[i] = __ballot(first_of_equal(keys, blk * kUniqTile + i * kThreads + threadIdx.x, m, &v[i], &before[i]));
    if (lane == 0) part[i * (kThreads / 64) + w] = (uint32_t)__popcll(kept[i]);
  }
  __syncthreads();
  if (w == 0) {
    const uint32_t mine = part[lane];
    uint32_t inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t x = __shfl_up(inc, o, 64);
      if (lane >= o) inc += x;
    }
    part[lane] = inc - mine;
  }
  __syncthreads();
  const int64_t base = off[blk];
  const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
  for (int i = 0; i < kUniqItems; ++i) {
    if (!((kept[i] >> lane) & 1ull)) continue;
    const int64_t p = base + part[i * (kThreads / 64) + w] + __popcll(kept[i] & lt);
    ukeys[p] = v[i];
    col[p] = (int32_t)(v[i] & ((1ull << colbits) - 1ull));
    const uint64_t row = v[i] >> colbits;
    if (p == 0 || row != before[i] >> colbits) rowptr[row] = p;
    if (p == nnz - 1) rowptr[row + 1] = nnz;
  }
}

// ptr[q] = first position whose segment id is >= q, for q in [0, n_seg]; seg ids are the bits
// of key[k] from `shift` upwards and are non-decreasing in k.  Requires n >= 1.
__global__ void k_boundaries(const uint64_t* __restrict__ key, int64_t n, int shift, int64_t n_seg, int64_t* __restrict__ ptr) {
  int64_t k = block_id() * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int64_t s = (int64_t)(key[k] >> shift);
  const int64_t sp = k == 0 ? -1 : (int64_t)(key[k - 1] >> shift);
  for (int64_t q = sp + 1; q <= s; ++q) ptr[q] = k;
  if (k == n - 1)
    for (int64_t q = s + 1; q <= n_seg; ++q) ptr[q] = n;
}

// first entry of each row whose (local) column is >= nr: columns are ascending, so the owned columns come first
__global__ void k_row_mid(const int64_t* __restrict__ ptr, const int32_t* __restrict__ col, int64_t nr,
                          int64_t* __restrict__ mid) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i >= nr) return;
  int64_t lo = ptr[i], hi = ptr[i + 1];
  while (lo < hi) {
    const int64_t m = (lo + hi) >> 1;
    if (col[m] < nr) lo = m + 1; else hi = m;
  }
  mid[i] = lo;
}

// ---- step 5: values ---------------------------------------------------------------------------------
// Degrees of the owned rows and fl(1/sqrt(d)) of every local column.  An owned vertex's degree is the entry count of its
// row, which the block holds whole (Sec. 4.1); a halo vertex's row lives elsewhere: its degree comes from the caller's
// global array.
__global__ void k_degrees(const int64_t* __restrict__ ptr, int64_t nr, int64_t nc, const int32_t* __restrict__ deg_global,
                          const int32_t* __restrict__ halo_gid, int32_t* __restrict__ deg, float* __restrict__ dinv) {
  int64_t c = block_id() * blockDim.x + threadIdx.x;
  if (c >= nc) return;
  int32_t d;
  if (c < nr) deg[c] = d = (int32_t)(ptr[c + 1] - ptr[c]);
  else d = deg_global[halo_gid[c - nr]];
  dinv[c] = inv_sqrt_deg(d);
}

// Four entries per thread, whole requests (what bounds the kernels below is the gather of a factor per entry out of L2, 11.8 M
// entries in 51 and 59 us; a launch that found the column pointers alone took 20).
constexpr int kEntriesPerThread = 4;
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));

// entries [p, p + 4) of n in v (the last one again behind the end); their number
__device__ __forceinline__ int load_keys(const uint64_t* __restrict__ keys, int64_t p, int64_t n, uint64_t (&v)[kEntriesPerThread]) {
  if (p + kEntriesPerThread <= n) {
    const u64x2 a = *reinterpret_cast<const u64x2*>(keys + p), b = *reinterpret_cast<const u64x2*>(keys + p + 2);
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    return kEntriesPerThread;
  }
#pragma unroll
  for (int i = 0; i < kEntriesPerThread; ++i) v[i] = keys[p + i < n ? p + i : n - 1];
  return (int)(n - p);
}

__global__ void k_values(const uint64_t* __restrict__ ukeys, int64_t nnz, int colbits, const float* __restrict__ dinv,
                         float* __restrict__ val) {
  const int64_t p = (block_id() * blockDim.x + threadIdx.x) * kEntriesPerThread;
  if (p >= nnz) return;
  const uint64_t colmask = (1ull << colbits) - 1ull;
  uint64_t v[kEntriesPerThread];
  const int n = load_keys(ukeys, p, nnz, v);
  f32x4 o;
#pragma unroll
  for (int i = 0; i < kEntriesPerThread; ++i) o[i] = __fmul_rn(dinv[v[i] >> colbits], dinv[v[i] & colmask]);
  if (n == kEntriesPerThread) *reinterpret_cast<f32x4*>(val + p) = o;
  else
#pragma unroll
    for (int i = 0; i < kEntriesPerThread; ++i)
      if (i < n) val[p + i] = o[i];
}

// ---- step 6: column-major copy ------------------------------------------------------------------------
// The entries sorted by column, those of a column still in row order; a value is computed again, from the same two
// factors, instead of being carried through the sort or fetched from its row-major place (124 us for 11.8 M entries).
// Also the column pointers: colptr[c] = first entry of a column >= c.
__global__ void k_finish_csc(const uint64_t* __restrict__ tkeys, int64_t nnz, int colbits, const float* __restrict__ dinv, int64_t nc,
                             int32_t* __restrict__ rowidx, float* __restrict__ val_t, int64_t* __restrict__ colptr) {
  const int64_t q = (block_id() * blockDim.x + threadIdx.x) * kEntriesPerThread;
  if (q >= nnz) return;
  const uint64_t colmask = (1ull << colbits) - 1ull;
  uint64_t v[kEntriesPerThread];
  const int n = load_keys(tkeys, q, nnz, v);
  int64_t before = q ? (int64_t)(tkeys[q - 1] & colmask) : -1;
  i32x4 r; f32x4 o;
#pragma unroll
  for (int i = 0; i < kEntriesPerThread; ++i) {
    const int64_t c = (int64_t)(v[i] & colmask);
    r[i] = (int32_t)(v[i] >> colbits);
    o[i] = __fmul_rn(dinv[v[i] >> colbits], dinv[c]);
    if (i < n)
      for (; before < c; ++before) colptr[before + 1] = q + i;
  }
  if (q + n == nnz)
    for (; before < nc; ++before) colptr[before + 1] = nnz;
  if (n == kEntriesPerThread) {
    *reinterpret_cast<i32x4*>(rowidx + q) = r;
    *reinterpret_cast<f32x4*>(val_t + q) = o;
  } else {
#pragma unroll
    for (int i = 0; i < kEntriesPerThread; ++i)
      if (i < n) { rowidx[q + i] = r[i]; val_t[q + i] = o[i]; }
  }
}

// ---- schedules ------------------------------------------------------------------------------------------
// A schedule is a stable counting sort of the rows by length class.  Ordinary rows have at most kHubRowNnz entries: 13
// classes, code 0 for [2^11, 2^12) down to 11 for one entry, 12 for none; code 13 are the hub rows, slot 14 counts their
// chunks of entries, slot 15 those of more than kGiantChunks (as a code: no row).  Three launches serve both schedules of a handle: rows of each code per block, one scan, placement.
// What bounds this is the launches, about 5 us each whatever they do, not the 16 bytes a row: against keys, scans, a radix
// pass and list kernels per schedule (28 launches) an R-MAT 2^18 build takes 1170 instead of 1287 us, a training step on a
// mini-batch of 20 K vertices 525 instead of 649.
constexpr int kSchedSlots = 16;
constexpr int kSchedCodes = 13;                      // classes of ordinary rows
constexpr int kHubCode = 13, kChunkSlot = 14, kGiantSlot = 15;
constexpr int kSchedSteps = 2;                       // rows per lane (8: longer code, 13 instead of 5 us for 40 K rows)
constexpr int kSchedTile = kThreads * kSchedSteps;   // rows per block; a wavefront takes 64 kSchedSteps consecutive ones
// What the host keeps: kSchedCodes + 1 class boundaries, then for each row boundary of the launches on row ranges the first
// position of every class, the first hub row and its first chunk at or behind that row, then the number of hub rows, of chunks and of giant rows.
constexpr int kSchedTable = kSchedCodes + 1;
constexpr int kSchedCounts = kSchedTable + (kRowChunks + 1) * (kSchedCodes + 2);
constexpr int kSchedWords = kSchedCounts + 3;
static_assert(kHubRowNnz == 2048 && kGiantSlot == kSchedSlots - 1 && kThreads == 256, "the codes above");
static_assert(2 * kSchedWords * sizeof(int64_t) <= kPinnedBytes, "both schedules of a handle are read back in one page");

struct SchedJob {
  const int64_t* ptr; int64_t n, blocks;
  uint32_t* cnt;            // [kSchedSlots][blocks] rows (chunks) of each slot in a block, then those in the blocks before it
  int32_t* wave_rows; int32_t* hub_rows; int64_t* hub_chunk_ptr; int32_t* chunk_hub;
  int64_t* info;            // [kSchedWords]
  int64_t bound[kRowChunks + 1];     // multiples of 64 rows, or n
};
struct SchedJobs { SchedJob j[2]; int n; };

__device__ __forceinline__ int row_code(int64_t len) {
  return len > kHubRowNnz ? kHubCode : len > 0 ? __clzll((unsigned long long)len) - 52 : kSchedCodes - 1;
}
__device__ __forceinline__ uint32_t row_chunks(int64_t len) {
  return len > kHubRowNnz ? (uint32_t)((len + kHubChunkNnz - 1) / kHubChunkNnz) : 0u;
}

struct SchedRank { uint32_t row, chunk; };     // rows of the lane's code, chunks, in the lanes before it
// 64 rows, one per lane: adds those of code `lane` (the chunks, in lane kChunkSlot, the giant rows, in lane kGiantSlot) to *seen
__device__ __forceinline__ SchedRank sched_step(int code, uint32_t chunks, int lane, uint32_t* seen) {
  const uint64_t lt = (1ull << lane) - 1ull;
  uint64_t peers = ~0ull, mine = ~0ull;    // lanes with this lane's code; lanes of code `lane`
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint64_t bal = __ballot((code >> b) & 1);
    peers &= ((code >> b) & 1) ? bal : ~bal;
    mine &= ((lane >> b) & 1) ? bal : ~bal;
  }
  if (lane < kChunkSlot) *seen += (uint32_t)__popcll(mine);
  SchedRank r{(uint32_t)__popcll(peers & lt), 0u};
  if (__any(chunks != 0)) {
    uint32_t inc = chunks;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t x = __shfl_up(inc, o, 64);
      if (lane >= o) inc += x;
    }
    r.chunk = inc - chunks;
    const uint32_t all = __shfl(inc, 63, 64);
    if (lane == kChunkSlot) *seen += all;
    const uint32_t giants = (uint32_t)__popcll(__ballot(chunks > (uint32_t)kGiantChunks));
    if (lane == kGiantSlot) *seen += giants;
  }
  return r;
}

__global__ __launch_bounds__(kThreads) void k_sched_count(SchedJobs jobs) {
  int64_t blk = block_id();
  const bool second = blk >= jobs.j[0].blocks;
  const SchedJob& a = jobs.j[second ? 1 : 0];
  if (second) blk -= jobs.j[0].blocks;
  if (blk >= a.blocks || (second && jobs.n < 2)) return;
  __shared__ uint32_t wave_cnt[kThreads / 64][kSchedSlots];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t seen = 0;                       // lane c: rows of code c, chunks in slot kChunkSlot
#pragma unroll
  for (int k = 0; k < kSchedSteps; ++k) {
    const int64_t i = blk * kSchedTile + k * kThreads + threadIdx.x;
    const int64_t len = i < a.n ? a.ptr[i + 1] - a.ptr[i] : 0;
    sched_step(i < a.n ? row_code(len) : kGiantSlot, row_chunks(len), lane, &seen);
  }
  if (lane < kSchedSlots) wave_cnt[w][lane] = seen;
  __syncthreads();
  if (threadIdx.x < kSchedSlots) {
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) sum += wave_cnt[i][threadIdx.x];
    a.cnt[threadIdx.x * a.blocks + blk] = sum;
  }
}

// one block per schedule, one wavefront per slot: the counts of the blocks before each block, the totals, and the table's
// rows for boundaries at the end of the matrix
__global__ __launch_bounds__(64 * kSchedSlots) void k_sched_scan(SchedJobs jobs) {
  const SchedJob& a = jobs.j[blockIdx.x];
  __shared__ uint32_t total[kSchedSlots];
  const int lane = threadIdx.x & 63, slot = threadIdx.x >> 6;
  uint32_t* __restrict__ cnt = a.cnt + slot * a.blocks;
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < a.blocks; b0 += 256) {
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t b = b0 + 4 * lane + k;
      v[k] = b < a.blocks ? cnt[b] : 0u;
      sum += v[k];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t x = __shfl_up(inc, o, 64);
      if (lane >= o) inc += x;
    }
    uint32_t run = carry + inc - sum;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int64_t b = b0 + 4 * lane + k;
      if (b < a.blocks) cnt[b] = run;
      run += v[k];
    }
    carry += __shfl(inc, 63, 64);
  }
  if (lane == 0) total[slot] = carry;
  __syncthreads();
  if (threadIdx.x != 0) return;
  int64_t start = 0;
  for (int c = 0; c <= kSchedCodes; ++c) {
    a.info[c] = start;
    if (c < kSchedCodes) start += total[c];
  }
  a.info[kSchedCounts] = total[kHubCode];
  a.info[kSchedCounts + 1] = total[kChunkSlot];
  a.info[kSchedCounts + 2] = total[kGiantSlot];
  a.hub_chunk_ptr[0] = 0;
  for (int j = 0; j <= kRowChunks; ++j) {
    if (a.bound[j] < a.n) continue;
    int64_t* t = a.info + kSchedTable + j * (kSchedCodes + 2);
    int64_t end = 0;
    for (int c = 0; c < kSchedCodes; ++c) t[c] = end += total[c];
    t[kSchedCodes] = total[kHubCode];
    t[kSchedCodes + 1] = total[kChunkSlot];
  }
}

__global__ __launch_bounds__(kThreads) void k_sched_place(SchedJobs jobs) {
  int64_t blk = block_id();
  const bool second = blk >= jobs.j[0].blocks;
  const SchedJob& a = jobs.j[second ? 1 : 0];
  if (second) blk -= jobs.j[0].blocks;
  if (blk >= a.blocks || (second && jobs.n < 2)) return;
  __shared__ uint32_t step_cnt[kThreads / 64][kSchedSteps][kSchedSlots];   // of the wavefront's steps before this one
  __shared__ uint32_t wave_cnt[kThreads / 64][kSchedSlots];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t row0 = blk * kSchedTile + (int64_t)w * 64 * kSchedSteps;
  int code[kSchedSteps];
  uint32_t chunks[kSchedSteps];
  SchedRank rank[kSchedSteps];
#pragma unroll
  for (int k = 0; k < kSchedSteps; ++k) {
    const int64_t i = row0 + 64 * k + lane;
    const int64_t len = i < a.n ? a.ptr[i + 1] - a.ptr[i] : 0;
    code[k] = i < a.n ? row_code(len) : kGiantSlot;
    chunks[k] = row_chunks(len);
  }
  uint32_t seen = 0;
#pragma unroll
  for (int k = 0; k < kSchedSteps; ++k) {
    if (lane < kSchedSlots) step_cnt[w][k][lane] = seen;
    rank[k] = sched_step(code[k], chunks[k], lane, &seen);
  }
  if (lane < kSchedSlots) wave_cnt[w][lane] = seen;
  __syncthreads();
  // position of the wavefront's first row of every code
  if (threadIdx.x < kSchedSlots) {
    const int c = threadIdx.x;
    uint32_t run = a.cnt[c * a.blocks + blk] + (c < kSchedCodes ? (uint32_t)a.info[c] : 0u);
#pragma unroll
    for (int i = 0; i < kThreads / 64; ++i) {
      const uint32_t x = wave_cnt[i][c];
      wave_cnt[i][c] = run;
      run += x;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSchedSteps; ++k) {
    const int64_t first = row0 + 64 * k, i = first + lane;
    if (first >= a.n) break;
    // a boundary of the launches on row ranges: where this step's rows would go is what lies behind it
    if (lane < kSchedCodes + 2) {
      const uint32_t at = wave_cnt[w][lane] + step_cnt[w][k][lane];
#pragma unroll
      for (int j = 0; j <= kRowChunks; ++j)
        if (a.bound[j] == first) a.info[kSchedTable + j * (kSchedCodes + 2) + lane] = at;
    }
    if (i >= a.n) continue;
    const uint32_t at = wave_cnt[w][code[k]] + step_cnt[w][k][code[k]] + rank[k].row;
    if (code[k] != kHubCode) {
      a.wave_rows[at] = (int32_t)i;
    } else {
      const uint32_t c0 = wave_cnt[w][kChunkSlot] + step_cnt[w][k][kChunkSlot] + rank[k].chunk;
      a.hub_rows[at] = (int32_t)i;
      a.hub_chunk_ptr[at + 1] = (int64_t)c0 + chunks[k];
      for (uint32_t c = 0; c < chunks[k]; ++c) a.chunk_hub[c0 + c] = (int32_t)at;
    }
  }
}

void free_schedule(Schedule* sc, bool idle) {
  pool_free(sc->wave_rows, idle);
  pool_free(sc->hub_rows, idle);
  pool_free(sc->hub_chunk_ptr, idle);
  pool_free(sc->chunk_hub, idle);
  *sc = Schedule();
}

// The schedules of a handle in two halves, so that one wait serves all: everything is enqueued against bounds on the numbers
// of long rows and chunks (a row of more than kHubRowNnz entries needs that many), then read back.
struct ScheduleBuild {
  struct Lists { DevBuf cnt, wave_rows, hub_rows, hub_chunk_ptr, chunk_hub; } l[2];
  DevBuf info;
  SchedJobs jobs{};
  const int64_t* host = nullptr;     // kSchedWords words per schedule, valid once the stream has been waited for

  int add(const int64_t* ptr, int64_t n, int64_t nnz, CallScope& sc) {
    Lists& o = l[jobs.n];
    SchedJob& j = jobs.j[jobs.n++];
    const int64_t max_hub = std::min(n, nnz / (kHubRowNnz + 1)), max_chunks = nnz / kHubChunkNnz + max_hub;
    j.ptr = ptr; j.n = n; j.blocks = ceil_div(n, kSchedTile);
    GCN_TRY(o.cnt.alloc(sc, sizeof(uint32_t) * kSchedSlots * (size_t)j.blocks));
    GCN_TRY(o.wave_rows.alloc(sc, sizeof(int32_t) * (size_t)n));
    GCN_TRY(o.hub_rows.alloc(sc, sizeof(int32_t) * (size_t)(max_hub + 1)));
    GCN_TRY(o.hub_chunk_ptr.alloc(sc, sizeof(int64_t) * (size_t)(max_hub + 1)));
    GCN_TRY(o.chunk_hub.alloc(sc, sizeof(int32_t) * (size_t)(max_chunks + 1)));
    j.cnt = o.cnt.as<uint32_t>(); j.wave_rows = o.wave_rows.as<int32_t>(); j.hub_rows = o.hub_rows.as<int32_t>();
    j.hub_chunk_ptr = o.hub_chunk_ptr.as<int64_t>(); j.chunk_hub = o.chunk_hub.as<int32_t>();
    // the class lists and the hub list are cut at kRowChunks row boundaries (multiples of 64 rows)
    for (int k = 0; k <= kRowChunks; ++k) {
      const int64_t r = round_up(ceil_div(n * k, kRowChunks), 64);
      j.bound[k] = k == kRowChunks || r > n ? n : r;
    }
    return GCN_OK;
  }

  int enqueue(CallScope& sc, int64_t* host_words) {
    hipStream_t s = sc.s;
    host = host_words;
    GCN_TRY(info.alloc(sc, sizeof(int64_t) * kSchedWords * (size_t)jobs.n));
    int64_t blocks = 0;
    for (int k = 0; k < jobs.n; ++k) { jobs.j[k].info = info.as<int64_t>() + k * kSchedWords; blocks += jobs.j[k].blocks; }
    k_sched_count<<<fold_grid(blocks), kThreads, 0, s>>>(jobs);
    k_sched_scan<<<jobs.n, 64 * kSchedSlots, 0, s>>>(jobs);
    k_sched_place<<<fold_grid(blocks), kThreads, 0, s>>>(jobs);
    GCN_CHECK_LAUNCH();
    GCN_HIP(hipMemcpyAsync(host_words, info.p, sizeof(int64_t) * kSchedWords * (size_t)jobs.n, hipMemcpyDeviceToHost, s));
    return GCN_OK;
  }

  // schedule k, after the stream has been waited for
  void finish(int k, Schedule* out) {
    const int64_t* h = host + k * kSchedWords;
    constexpr int kFirst = 33 - kSchedCodes;         // longer rows than class kFirst's are hub rows
    *out = Schedule();
    out->n_hub_rows = h[kSchedCounts];
    out->n_chunks = h[kSchedCounts + 1];
    out->n_giant_rows = h[kSchedCounts + 2];
    out->n_wave_rows = jobs.j[k].n - out->n_hub_rows;
    for (int c = 0; c < 34; ++c) out->class_begin[c] = c < kFirst ? 0 : h[c - kFirst];
    for (int j = 0; j <= kRowChunks; ++j) {
      const int64_t* t = h + kSchedTable + j * (kSchedCodes + 2);
      out->chunk_row[j] = jobs.j[k].bound[j];
      for (int c = 0; c < 33; ++c) out->chunk_class_begin[j][c] = c < kFirst ? 0 : t[c - kFirst];
      out->chunk_hub_begin[j] = t[kSchedCodes];
      out->chunk_hubchunk_begin[j] = t[kSchedCodes + 1];
    }
    out->wave_rows = (int32_t*)l[k].wave_rows.release();
    out->hub_rows = (int32_t*)l[k].hub_rows.release();
    out->hub_chunk_ptr = (int64_t*)l[k].hub_chunk_ptr.release();
    out->chunk_hub = (int32_t*)l[k].chunk_hub.release();
  }
};

int key_bits(int64_t n) {              // smallest b >= 1 with 2^b >= n
  int b = 1;
  while ((1LL << b) < n) ++b;
  return b;
}

static int64_t uniq_blocks(int64_t m) { return ceil_div(m, kUniqTile); }
size_t key_words_bytes(int64_t m) { return sizeof(int64_t) * (size_t)(uniq_blocks(m) + 3); }
int64_t* key_verdict(const DevBuf& words, int64_t m) { return words.as<int64_t>() + uniq_blocks(m) + 1; }

static int verdict(int64_t v) {
  if (v & 1) return fail(GCN_EINVAL, "gcn_csr_build: a vertex id lies outside [0, n_global)");
  if (v & 2) return fail(GCN_EINVAL, "gcn_csr_build: d_deg_global holds a degree < 1");
  return GCN_OK;
}

int adopt_arrays(const HandleArrays& h, CallScope& sc, PinnedPage& page, gcn_csr* A) {
  const bool csc = h.colptr->p != nullptr;
  const int64_t nc = h.nr + h.nh;
  ScheduleBuild sched;
  GCN_TRY(sched.add(h.rowptr->as<int64_t>(), h.nr, h.nnz, sc));
  if (csc) GCN_TRY(sched.add(h.colptr->as<int64_t>(), nc, h.nnz, sc));
  GCN_TRY(sched.enqueue(sc, page.words()));
  GCN_HIP(hipStreamSynchronize(sc.s));
  sc.done = true;

  A->n_global = h.n_global; A->row_lo = h.row_lo;
  A->nr = h.nr; A->nh = h.nh; A->nc = nc; A->nnz = h.nnz;
  sched.finish(0, &A->sched);
  if (csc) sched.finish(1, &A->sched_t);
  A->rowptr = (int64_t*)h.rowptr->release(); A->col = (int32_t*)h.col->release();
  A->val = (float*)h.val->release(); A->deg = (int32_t*)h.deg->release();
  A->halo_gid = (int32_t*)h.halo_gid->release();
  A->colptr = (int64_t*)h.colptr->release(); A->rowidx = (int32_t*)h.rowidx->release();
  A->val_t = (float*)h.val_t->release();
  A->mid = h.nh > 0 ? (int64_t*)h.mid->release() : nullptr;
  return GCN_OK;
}

int build_from_keys(const KeyBuild& in, CallScope& sc, PinnedPage& page, gcn_csr* A) {
  hipStream_t s = sc.s;
  const int64_t nr = in.nr, nh = in.nh, nc = nr + nh, m = in.m;
  const int colbits = key_bits(nc), rowbits = key_bits(nr);
  int64_t* read = page.words();
  uint64_t *keys_a = in.keys_a->as<uint64_t>(), *keys_b = in.keys_b->as<uint64_t>();
  const int64_t nb = uniq_blocks(m);
  DevBuf tmp, cnt;
  GCN_TRY(tmp.alloc(sc, std::max(sort_tmp_bytes(m), scan_tmp_bytes(nb))));
  GCN_TRY(cnt.alloc(sc, sizeof(uint32_t) * (size_t)nb));
  // behind the offsets of the blocks: the number of entries, the verdict on the ids, the number of keys sorted
  int64_t* off = in.words->as<int64_t>();
  int64_t* bad = off + nb + 1;
  int64_t* kept = off + nb + 2;
  uint64_t* sorted = nullptr;
  GCN_TRY(radix_sort_u64(keys_a, keys_b, nullptr, nullptr, m, 0, colbits + rowbits, tmp.p, s, &sorted, nullptr, in.count,
                         in.count ? nullptr : kept));
  const int64_t* count = in.count ? in.count : kept;
  uint64_t* ukeys = sorted == keys_a ? keys_b : keys_a;       // unique keys, row-major order
  k_count_unique<<<fold_grid(nb), kThreads, 0, s>>>(sorted, count, nb, cnt.as<uint32_t>());
  GCN_CHECK_LAUNCH();
  GCN_TRY(exclusive_scan_u32(cnt.as<uint32_t>(), off, nb, tmp.p, s));
  GCN_HIP(hipMemcpyAsync(read, off + nb, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
  GCN_HIP(hipStreamSynchronize(s));
  if (!in.count) GCN_TRY(verdict(read[1]));
  const int64_t nnz = read[0];
  if (nnz < nr) return fail(GCN_EHIP, "gcn_csr_build: internal error (nnz %lld < rows %lld)", (long long)nnz, (long long)nr);
  if (nnz >= 0xffffffffLL) return fail(GCN_EINVAL, "gcn_csr_build: more than 2^32-2 stored entries in one block");

  DevBuf rowptr, col, val, deg, dinv;
  GCN_TRY(rowptr.alloc(sc, sizeof(int64_t) * (size_t)(nr + 1)));
  GCN_TRY(col.alloc(sc, sizeof(int32_t) * (size_t)nnz + kEntrySlack));
  GCN_TRY(val.alloc(sc, sizeof(float) * (size_t)nnz + kEntrySlack));
  GCN_TRY(deg.alloc(sc, sizeof(int32_t) * (size_t)nr));
  GCN_TRY(dinv.alloc(sc, sizeof(float) * (size_t)nc));
  k_compact<<<fold_grid(nb), kThreads, 0, s>>>(sorted, off, count, nb, colbits, nnz, ukeys, col.as<int32_t>(), rowptr.as<int64_t>());
  k_degrees<<<grid_for(nc), kThreads, 0, s>>>(rowptr.as<int64_t>(), nr, nc, in.deg_global, in.halo_gid->as<int32_t>(), deg.as<int32_t>(),
                                               dinv.as<float>());
  k_values<<<grid_for(ceil_div(nnz, kEntriesPerThread)), kThreads, 0, s>>>(ukeys, nnz, colbits, dinv.as<float>(), val.as<float>());
  GCN_CHECK_LAUNCH();

  DevBuf mid;
  if (nh > 0) {
    GCN_TRY(mid.alloc(sc, sizeof(int64_t) * (size_t)nr));
    k_row_mid<<<grid_for(nr), kThreads, 0, s>>>(rowptr.as<int64_t>(), col.as<int32_t>(), nr, mid.as<int64_t>());
    GCN_CHECK_LAUNCH();
  }

  // -- column-major copy
  DevBuf colptr, rowidx, val_t;
  if (in.flags & GCN_BUILD_CSC) {
    GCN_TRY(colptr.alloc(sc, sizeof(int64_t) * (size_t)(nc + 1)));
    GCN_TRY(rowidx.alloc(sc, sizeof(int32_t) * (size_t)nnz + kEntrySlack));
    GCN_TRY(val_t.alloc(sc, sizeof(float) * (size_t)nnz + kEntrySlack));
    uint64_t* tsorted = nullptr;           // (the buffer of the keys with duplicates is free again)
    GCN_TRY(radix_sort_u64(ukeys, sorted, nullptr, nullptr, nnz, 0, colbits, tmp.p, s, &tsorted, nullptr));
    k_finish_csc<<<grid_for(ceil_div(nnz, kEntriesPerThread)), kThreads, 0, s>>>(tsorted, nnz, colbits, dinv.as<float>(), nc,
                                                                                 rowidx.as<int32_t>(), val_t.as<float>(), colptr.as<int64_t>());
    GCN_CHECK_LAUNCH();
  }
  HandleArrays h{in.n_global, in.row_lo, nr, nh, nnz, &rowptr, &col, &val, &deg, in.halo_gid, &colptr, &rowidx, &val_t, &mid};
  return adopt_arrays(h, sc, page, A);
}

static int build_impl(const int32_t* d_src, const int32_t* d_dst, int64_t n_edges, int64_t n_global,
                      int64_t row_lo, int64_t row_hi, const int32_t* d_deg_global, int flags,
                      hipStream_t s, gcn_csr* A) {
  const int64_t nr = row_hi - row_lo;
  const bool whole = (row_lo == 0 && row_hi == n_global);
  const int64_t m = n_edges + nr;          // candidate entries: edges + diagonal

  CallScope sc(s);
  PinnedPage page;
  GCN_TRY(page.take(sc));
  int64_t* read = page.words();
  // -- validation and halo bitmap.  A whole graph has no halo, and its ids are checked while its keys are made: the
  // verdict is read with the number of entries, and what is enqueued until then uses no id as an index.
  const int64_t words = ceil_div(n_global, 32);
  DevBuf off, bitmap, wcnt, wprefix, tmp;
  GCN_TRY(off.alloc(sc, key_words_bytes(m)));
  int64_t* bad = key_verdict(off, m);
  GCN_HIP(hipMemsetAsync(bad, 0, sizeof(int64_t), s));
  if (d_deg_global) k_validate_deg<<<grid_for(n_global), kThreads, 0, s>>>(d_deg_global, n_global, (int*)bad);
  int64_t nh = 0;
  if (!whole) {
    GCN_TRY(tmp.alloc(sc, scan_tmp_bytes(words)));
    GCN_TRY(bitmap.alloc(sc, sizeof(uint32_t) * (size_t)words));
    GCN_TRY(wcnt.alloc(sc, sizeof(uint32_t) * (size_t)words));
    GCN_TRY(wprefix.alloc(sc, sizeof(int64_t) * (size_t)(words + 1)));
    GCN_HIP(hipMemsetAsync(bitmap.p, 0, sizeof(uint32_t) * (size_t)words, s));
    if (n_edges > 0) k_validate<<<grid_for(n_edges), kThreads, 0, s>>>(d_src, d_dst, n_edges, n_global, (int*)bad);
    GCN_CHECK_LAUNCH();
    GCN_HIP(hipMemcpyAsync(read, bad, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    GCN_HIP(hipStreamSynchronize(s));
    GCN_TRY(verdict(read[0]));
    if (n_edges > 0) k_mark_halo<<<grid_for(n_edges), kThreads, 0, s>>>(d_src, d_dst, n_edges, row_lo, row_hi, bitmap.as<uint32_t>());
    k_popc<<<grid_for(words), kThreads, 0, s>>>(bitmap.as<uint32_t>(), words, wcnt.as<uint32_t>());
    GCN_CHECK_LAUNCH();
    GCN_TRY(exclusive_scan_u32(wcnt.as<uint32_t>(), wprefix.as<int64_t>(), words, tmp.p, s));
    GCN_HIP(hipMemcpyAsync(read, wprefix.as<int64_t>() + words, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    GCN_HIP(hipStreamSynchronize(s));
    nh = read[0];
  }
  const int64_t nc = nr + nh;
  if (nc >= 0x7fffffffLL) return fail(GCN_EINVAL, "gcn_csr_build: more than 2^31-1 local columns");
  DevBuf halo_gid;
  GCN_TRY(halo_gid.alloc(sc, sizeof(int32_t) * (size_t)(nh > 0 ? nh : 1)));
  if (nh > 0) k_halo_list<<<grid_for(words), kThreads, 0, s>>>(bitmap.as<uint32_t>(), wprefix.as<int64_t>(), words, halo_gid.as<int32_t>());
  GCN_CHECK_LAUNCH();

  // -- keys
  const int colbits = key_bits(nc);
  if (colbits + key_bits(nr) > 62) return fail(GCN_EINVAL, "gcn_csr_build: block too large for 64-bit sort keys");
  DevBuf keys_a, keys_b;
  GCN_TRY(keys_a.alloc(sc, sizeof(uint64_t) * (size_t)m));
  GCN_TRY(keys_b.alloc(sc, sizeof(uint64_t) * (size_t)m));
  k_make_keys<<<grid_for(m), kThreads, 0, s>>>(d_src, d_dst, n_edges, row_lo, row_hi, nr, colbits,
                                                bitmap.as<uint32_t>(), wprefix.as<int64_t>(), keys_a.as<uint64_t>(), (int*)bad);
  GCN_CHECK_LAUNCH();
  KeyBuild in;
  in.n_global = n_global; in.row_lo = row_lo; in.nr = nr; in.nh = nh;
  in.keys_a = &keys_a; in.keys_b = &keys_b; in.words = &off; in.m = m;
  in.halo_gid = &halo_gid; in.deg_global = d_deg_global; in.flags = flags;
  return build_from_keys(in, sc, page, A);
}

int segment_boundaries(const uint64_t* keys, int64_t n, int shift, int64_t n_seg, int64_t* ptr, hipStream_t s) {
  if (n < 1) return fail(GCN_EINVAL, "segment_boundaries: empty input");
  k_boundaries<<<grid_for(n), kThreads, 0, s>>>(keys, n, shift, n_seg, ptr);
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

int ensure_workspace(gcn_csr* A, size_t bytes) {
  if (bytes <= A->ws_bytes) return GCN_OK;
  if (A->ws) {
    int device = -1;
    GCN_HIP(hipGetDevice(&device));
    GCN_HIP(hipDeviceSynchronize());
    pool_free(A->ws, device == A->device);      // (another device than the handle's was waited for: hipFree waits for the right one)
    A->ws = nullptr; A->ws_bytes = 0;
  }
  size_t want = (size_t)round_up((int64_t)bytes, 1 << 20);
  GCN_TRY(pool_alloc(&A->ws, want));
  A->ws_bytes = want;
  return GCN_OK;
}

}  // namespace gcn

using namespace gcn;

extern "C" int gcn_csr_build(const int32_t* d_src, const int32_t* d_dst, int64_t n_edges, int64_t n_global,
                             int64_t row_lo, int64_t row_hi, const int32_t* d_deg_global, int flags,
                             void* stream, gcn_csr_t** out) {
  clear_error();
  if (!out) return fail(GCN_EINVAL, "gcn_csr_build: out is NULL");
  *out = nullptr;
  if (n_edges < 0 || (n_edges > 0 && (!d_src || !d_dst))) return fail(GCN_EINVAL, "gcn_csr_build: bad edge list");
  if (n_global < 1 || n_global > 0x7fffffffLL) return fail(GCN_EINVAL, "gcn_csr_build: n_global must be in [1, 2^31)");
  // stored entries then stay below 2^32: the column sweep's plan sorts entry positions as 32-bit payloads, and partition
  // figures count entries in 32 bits
  if (n_edges + n_global >= 0xffffffffLL) return fail(GCN_EINVAL, "gcn_csr_build: more than 2^32 - 1 edges and rows");
  if (row_lo < 0 || row_hi <= row_lo || row_hi > n_global) return fail(GCN_EINVAL, "gcn_csr_build: need 0 <= row_lo < row_hi <= n_global");
  if (!(row_lo == 0 && row_hi == n_global) && !d_deg_global)
    return fail(GCN_EINVAL, "gcn_csr_build: a block that is not the whole graph needs d_deg_global");
  if (flags & ~GCN_BUILD_CSC) return fail(GCN_EINVAL, "gcn_csr_build: unknown flag");
  gcn_csr* A = new (std::nothrow) gcn_csr();
  if (!A) return fail(GCN_ENOMEM, "gcn_csr_build: host allocation failed");
  if (hipGetDevice(&A->device) != hipSuccess) { delete A; return fail(GCN_EHIP, "hipGetDevice failed"); }
  int rc = build_impl(d_src, d_dst, n_edges, n_global, row_lo, row_hi, d_deg_global, flags, (hipStream_t)stream, A);
  if (rc != GCN_OK) { gcn_csr_free(A); return rc; }
  *out = A;
  return GCN_OK;
}

extern "C" int gcn_csr_info(const gcn_csr_t* A, int64_t* nr, int64_t* nh, int64_t* nnz) {
  clear_error();
  if (!A) return fail(GCN_EINVAL, "gcn_csr_info: NULL handle");
  if (nr) *nr = A->nr;
  if (nh) *nh = A->nh;
  if (nnz) *nnz = A->nnz;
  return GCN_OK;
}

extern "C" int gcn_csr_arrays(const gcn_csr_t* A, const int64_t** rowptr, const int32_t** col, const float** val,
                              const int32_t** deg, const int32_t** halo_gid, const int64_t** colptr,
                              const int32_t** rowidx, const float** val_t) {
  clear_error();
  if (!A) return fail(GCN_EINVAL, "gcn_csr_arrays: NULL handle");
  if (rowptr) *rowptr = A->rowptr;
  if (col) *col = A->col;
  if (val) *val = A->val;
  if (deg) *deg = A->deg;
  if (halo_gid) *halo_gid = A->halo_gid;
  if (colptr) *colptr = A->colptr;
  if (rowidx) *rowidx = A->rowidx;
  if (val_t) *val_t = A->val_t;
  return GCN_OK;
}

extern "C" int gcn_csr_free(gcn_csr_t* A) {
  if (!A) return GCN_OK;
  int device = A->device;
  (void)hipGetDevice(&device);
  if (device != A->device) (void)hipSetDevice(A->device);
  const bool idle = hipDeviceSynchronize() == hipSuccess;
  void* ptrs[] = {A->rowptr, A->col, A->val, A->deg, A->halo_gid, A->colptr, A->rowidx, A->val_t, A->mid, A->ws};
  for (void* p : ptrs) pool_free(p, idle);
  free_schedule(&A->sched, idle);
  free_schedule(&A->sched_t, idle);
  free_panel_plans(A, idle);
  for (hipEvent_t e : A->side_events) if (e) (void)hipEventDestroy(e);
  if (A->side_stream) (void)hipStreamDestroy(A->side_stream);
  if (device != A->device) (void)hipSetDevice(device);
  delete A;
  return GCN_OK;
}
