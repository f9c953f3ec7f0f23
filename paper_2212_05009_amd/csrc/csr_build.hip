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
// in memory cost 28 bytes a key where this reads 16 (keys twice).
constexpr int kUniqItems = 16;
constexpr int kUniqTile = kThreads * kUniqItems;
static_assert(kThreads / 64 * kUniqItems == 64, "k_compact scans the counts of a block's (round, wavefront) pairs in one wavefront");

__device__ __forceinline__ bool first_of_equal(const uint64_t* __restrict__ keys, int64_t k, int64_t m, uint64_t* v) {
  if (k >= m) return false;
  *v = keys[k];
  return *v != kInvalidKey && (k == 0 || keys[k - 1] != *v);
}

__global__ __launch_bounds__(kThreads) void k_count_unique(const uint64_t* __restrict__ keys, int64_t m, int64_t nb,
                                                           uint32_t* __restrict__ cnt) {
  const int64_t blk = block_id();
  if (blk >= nb) return;
  __shared__ uint32_t wave_cnt[kThreads / 64];
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < kUniqItems; ++i) {
    uint64_t v = 0;
    c += (uint32_t)__popcll(__ballot(first_of_equal(keys, blk * kUniqTile + i * kThreads + threadIdx.x, m, &v)));
  }
  if ((threadIdx.x & 63) == 0) wave_cnt[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int i = 0; i < kThreads / 64; ++i) tot += wave_cnt[i];
    cnt[blk] = tot;
  }
}

__global__ __launch_bounds__(kThreads) void k_compact(const uint64_t* __restrict__ keys, const int64_t* __restrict__ off,
                                                      int64_t m, int64_t nb, int colbits, uint64_t* __restrict__ ukeys,
                                                      int32_t* __restrict__ col) {
  const int64_t blk = block_id();
  if (blk >= nb) return;
  __shared__ uint32_t part[64];            // keys kept by round i, wavefront w at [i * waves + w]; then those before it
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint64_t v[kUniqItems];
  uint64_t kept[kUniqItems];
#pragma unroll
  for (int i = 0; i < kUniqItems; ++i) {
    v[i] = 0;
    kept[i] = __ballot(first_of_equal(keys, blk * kUniqTile + i * kThreads + threadIdx.x, m, &v[i]));
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
  }
}

// ptr[q] = first position whose segment id is >= q, for q in [0, n_seg]; seg ids are the bits
// of key[k] from `shift` upwards that are set in `mask` and are non-decreasing in k.  Requires n >= 1.
__global__ void k_boundaries(const uint64_t* __restrict__ key, int64_t n, int shift, uint64_t mask, int64_t n_seg,
                             int64_t* __restrict__ ptr) {
  int64_t k = block_id() * blockDim.x + threadIdx.x;
  if (k >= n) return;
  int64_t s = (int64_t)((key[k] >> shift) & mask);
  int64_t sp = k == 0 ? -1 : (int64_t)((key[k - 1] >> shift) & mask);
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
// val(i,j) = fl(1/sqrt(d_i)) * fl(1/sqrt(d_j)), each operation correctly rounded in fp32.
// Both steps go through fp64: an fp64 square root or quotient rounded once more to fp32 equals the
// correctly rounded fp32 result (53 >= 2*24 + 2 bits), whatever the fp32 code generation options are.
__device__ __forceinline__ float inv_sqrt_deg(int32_t d) {
  const float r = (float)sqrt((double)(float)d);
  return (float)(1.0 / (double)r);
}

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

__global__ void k_values(const uint64_t* __restrict__ ukeys, int64_t nnz, int colbits, const float* __restrict__ dinv,
                         float* __restrict__ val) {
  int64_t p = block_id() * blockDim.x + threadIdx.x;
  if (p >= nnz) return;
  const uint64_t v = ukeys[p];
  val[p] = __fmul_rn(dinv[v >> colbits], dinv[v & ((1ull << colbits) - 1ull)]);
}

// ---- step 6: column-major copy ------------------------------------------------------------------------
// The entries sorted by column, those of a column still in row order; a value is computed again, from the same two
// factors, instead of being carried through the sort or fetched from its row-major place (124 us for 11.8 M entries).
__global__ void k_finish_csc(const uint64_t* __restrict__ tkeys, int64_t nnz, int colbits, const float* __restrict__ dinv,
                             int32_t* __restrict__ rowidx, float* __restrict__ val_t) {
  int64_t q = block_id() * blockDim.x + threadIdx.x;
  if (q >= nnz) return;
  const uint64_t v = tkeys[q];
  rowidx[q] = (int32_t)(v >> colbits);
  val_t[q] = __fmul_rn(dinv[v >> colbits], dinv[v & ((1ull << colbits) - 1ull)]);
}

// ---- schedules ------------------------------------------------------------------------------------------
__global__ void k_sched_keys(const int64_t* __restrict__ ptr, int64_t n, uint64_t* __restrict__ keys,
                             uint32_t* __restrict__ hub_flag, uint32_t* __restrict__ hub_chunks) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int64_t len = ptr[i + 1] - ptr[i];
  bool hub = len > kHubRowNnz;
  hub_flag[i] = hub ? 1u : 0u;
  hub_chunks[i] = hub ? (uint32_t)((len + kHubChunkNnz - 1) / kHubChunkNnz) : 0u;
  // longest rows first: class 0 holds lengths in [2^31, ..), class 31 length 1, class 32 empty rows
  uint32_t cls = len > 0 ? (uint32_t)__clzll((unsigned long long)len) - 32u : 32u;
  keys[i] = hub ? kInvalidKey : (((uint64_t)cls << 32) | (uint64_t)i);
}

__global__ void k_take_low32(const uint64_t* __restrict__ keys, int64_t n, int32_t* __restrict__ out) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < n) out[i] = (int32_t)(keys[i] & 0xffffffffull);
}

__global__ void k_hub_lists(const uint32_t* __restrict__ hub_flag, const int64_t* __restrict__ hub_pos,
                            const uint32_t* __restrict__ hub_chunks, const int64_t* __restrict__ chunk_pos,
                            int64_t n, int32_t* __restrict__ hub_rows,
                            int64_t* __restrict__ hub_chunk_ptr, int32_t* __restrict__ chunk_hub) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i == 0) hub_chunk_ptr[0] = 0;
  if (i >= n || !hub_flag[i]) return;
  int64_t h = hub_pos[i];
  hub_rows[h] = (int32_t)i;
  int64_t c0 = chunk_pos[i];
  hub_chunk_ptr[h + 1] = c0 + hub_chunks[i];
  for (uint32_t c = 0; c < hub_chunks[i]; ++c) chunk_hub[c0 + c] = (int32_t)h;
}

// What the host keeps of a schedule: class boundaries (kClassSegs + 1 words, of which the hub rows' class is the last that
// counts), the table of k_chunk_bounds, the numbers of hub rows and of their chunks.
constexpr int kClassSegs = 64;
constexpr int kChunkTable = (kRowChunks + 1) * 35;
constexpr int kSchedWords = kClassSegs + 1 + kChunkTable + 2;
static_assert(2 * kSchedWords * sizeof(int64_t) <= kPinnedBytes, "both schedules of a handle are read back in one page");
struct RowBounds { int64_t row[kRowChunks + 1]; };

// Row boundaries in the schedule's lists.  For boundary j (row bounds.row[j]): out[j * 35 + c], c < 33, = first position
// of class c (list positions cb[c] .. cb[c + 1], rows ascending) whose row is >= bound[j]; out[j * 35 + 33] = first
// hub row (ascending list of n_hub rows) >= bound[j]; out[j * 35 + 34] = that hub row's first chunk of entries.
__global__ void k_chunk_bounds(const int32_t* __restrict__ wave_rows, const int64_t* __restrict__ cb,
                               const int32_t* __restrict__ hub_rows, const int64_t* __restrict__ n_hub,
                               const int64_t* __restrict__ n_chunks, const int64_t* __restrict__ hub_chunk_ptr, RowBounds bounds,
                               int64_t* __restrict__ out, int64_t* __restrict__ counts) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t == 0) { counts[0] = *n_hub; counts[1] = *n_chunks; }
  if (t >= (kRowChunks + 1) * 34) return;
  const int j = t / 34, c = t % 34;
  const int32_t* list = c < 33 ? wave_rows : hub_rows;
  int64_t lo = c < 33 ? cb[c] : 0, hi = c < 33 ? cb[c + 1] : *n_hub;
  const int64_t r = bounds.row[j];
  while (lo < hi) {
    const int64_t mid = lo + (hi - lo) / 2;
    if ((int64_t)list[mid] < r) lo = mid + 1; else hi = mid;
  }
  out[j * 35 + c] = lo;
  if (c == 33) out[j * 35 + 34] = hub_chunk_ptr[lo];
}

void free_schedule(Schedule* sc, bool idle) {
  pool_free(sc->wave_rows, idle);
  pool_free(sc->hub_rows, idle);
  pool_free(sc->hub_chunk_ptr, idle);
  pool_free(sc->chunk_hub, idle);
  *sc = Schedule();
}

// A schedule in two halves, so that one wait serves both of a handle: everything is enqueued against bounds on the numbers
// of long rows and chunks (a row of more than kHubRowNnz entries needs that many), then read back.
struct ScheduleBuild {
  DevBuf keys_a, keys_b, hub_flag, hub_chunks, hub_pos, chunk_pos, tmp, info;
  DevBuf wave_rows, hub_rows, hub_chunk_ptr, chunk_hub;
  RowBounds bounds;
  const int64_t* host = nullptr;     // kSchedWords words, valid once the stream has been waited for

  int enqueue(const int64_t* ptr, int64_t n, int64_t nnz, CallScope& sc, int64_t* host_words) {
    hipStream_t s = sc.s;
    host = host_words;
    const int64_t max_hub = std::min(n, nnz / (kHubRowNnz + 1)), max_chunks = nnz / kHubChunkNnz + max_hub;
    GCN_TRY(keys_a.alloc(sc, sizeof(uint64_t) * (size_t)n));
    GCN_TRY(keys_b.alloc(sc, sizeof(uint64_t) * (size_t)n));
    GCN_TRY(hub_flag.alloc(sc, sizeof(uint32_t) * (size_t)n));
    GCN_TRY(hub_chunks.alloc(sc, sizeof(uint32_t) * (size_t)n));
    GCN_TRY(hub_pos.alloc(sc, sizeof(int64_t) * (size_t)(n + 1)));
    GCN_TRY(chunk_pos.alloc(sc, sizeof(int64_t) * (size_t)(n + 1)));
    GCN_TRY(tmp.alloc(sc, std::max(sort_tmp_bytes(n), scan_tmp_bytes(n))));
    GCN_TRY(info.alloc(sc, sizeof(int64_t) * kSchedWords));
    GCN_TRY(wave_rows.alloc(sc, sizeof(int32_t) * (size_t)n));
    GCN_TRY(hub_rows.alloc(sc, sizeof(int32_t) * (size_t)(max_hub + 1)));
    GCN_TRY(hub_chunk_ptr.alloc(sc, sizeof(int64_t) * (size_t)(max_hub + 1)));
    GCN_TRY(chunk_hub.alloc(sc, sizeof(int32_t) * (size_t)(max_chunks + 1)));
    int64_t* class_begin = info.as<int64_t>();
    int64_t* table = class_begin + kClassSegs + 1;

    k_sched_keys<<<grid_for(n), kThreads, 0, s>>>(ptr, n, keys_a.as<uint64_t>(), hub_flag.as<uint32_t>(), hub_chunks.as<uint32_t>());
    GCN_CHECK_LAUNCH();
    GCN_TRY(exclusive_scan_u32(hub_flag.as<uint32_t>(), hub_pos.as<int64_t>(), n, tmp.p, s));
    GCN_TRY(exclusive_scan_u32(hub_chunks.as<uint32_t>(), chunk_pos.as<int64_t>(), n, tmp.p, s));
    uint64_t* sorted = nullptr;
    GCN_TRY(radix_sort_u64(keys_a.as<uint64_t>(), keys_b.as<uint64_t>(), nullptr, nullptr, n, 32, 40, tmp.p, s, &sorted, nullptr));
    // hub rows carry the key ~0: they follow the ordinary rows, as segment 63
    k_take_low32<<<grid_for(n), kThreads, 0, s>>>(sorted, n, wave_rows.as<int32_t>());
    k_boundaries<<<grid_for(n), kThreads, 0, s>>>(sorted, n, 32, kClassSegs - 1, kClassSegs, class_begin);
    k_hub_lists<<<grid_for(n), kThreads, 0, s>>>(hub_flag.as<uint32_t>(), hub_pos.as<int64_t>(), hub_chunks.as<uint32_t>(),
                                                  chunk_pos.as<int64_t>(), n, hub_rows.as<int32_t>(), hub_chunk_ptr.as<int64_t>(),
                                                  chunk_hub.as<int32_t>());
    // the class lists and the hub list cut at kRowChunks row boundaries (multiples of 64 rows)
    for (int j = 0; j <= kRowChunks; ++j) {
      const int64_t r = round_up(ceil_div(n * j, kRowChunks), 64);
      bounds.row[j] = j == kRowChunks || r > n ? n : r;
    }
    k_chunk_bounds<<<(unsigned)ceil_div((kRowChunks + 1) * 34, 256), 256, 0, s>>>(
        wave_rows.as<int32_t>(), class_begin, hub_rows.as<int32_t>(), hub_pos.as<int64_t>() + n, chunk_pos.as<int64_t>() + n,
        hub_chunk_ptr.as<int64_t>(), bounds, table, table + kChunkTable);
    GCN_CHECK_LAUNCH();
    GCN_HIP(hipMemcpyAsync(host_words, info.p, sizeof(int64_t) * kSchedWords, hipMemcpyDeviceToHost, s));
    return GCN_OK;
  }

  // after the stream has been waited for
  void finish(int64_t n, Schedule* out) {
    const int64_t* table = host + kClassSegs + 1;
    *out = Schedule();
    out->n_hub_rows = table[kChunkTable];
    out->n_chunks = table[kChunkTable + 1];
    out->n_wave_rows = n - out->n_hub_rows;
    for (int c = 0; c < 34; ++c) out->class_begin[c] = host[c];
    for (int j = 0; j <= kRowChunks; ++j) {
      out->chunk_row[j] = bounds.row[j];
      for (int c = 0; c < 33; ++c) out->chunk_class_begin[j][c] = table[j * 35 + c];
      out->chunk_hub_begin[j] = table[j * 35 + 33];
      out->chunk_hubchunk_begin[j] = table[j * 35 + 34];
    }
    out->wave_rows = (int32_t*)wave_rows.release();
    out->hub_rows = (int32_t*)hub_rows.release();
    out->hub_chunk_ptr = (int64_t*)hub_chunk_ptr.release();
    out->chunk_hub = (int32_t*)chunk_hub.release();
  }
};

static int bits_for(int64_t max_value_exclusive) {   // smallest b with 2^b - 1 > max_value_exclusive - 1 ... i.e. 2^b > max_value_exclusive
  int b = 1;
  while ((1LL << b) <= max_value_exclusive) ++b;
  return b;
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
  DevBuf bad, bitmap, wcnt, wprefix, tmp;
  GCN_TRY(bad.alloc(sc, sizeof(int64_t)));
  size_t tb = sort_tmp_bytes(m);
  if (scan_tmp_bytes(m) > tb) tb = scan_tmp_bytes(m);
  if (scan_tmp_bytes(words) > tb) tb = scan_tmp_bytes(words);
  GCN_TRY(tmp.alloc(sc, tb));
  GCN_HIP(hipMemsetAsync(bad.p, 0, sizeof(int64_t), s));
  if (d_deg_global) k_validate_deg<<<grid_for(n_global), kThreads, 0, s>>>(d_deg_global, n_global, bad.as<int>());
  auto verdict = [&](int64_t v) {
    if (v & 1) return fail(GCN_EINVAL, "gcn_csr_build: a vertex id lies outside [0, n_global)");
    if (v & 2) return fail(GCN_EINVAL, "gcn_csr_build: d_deg_global holds a degree < 1");
    return (int)GCN_OK;
  };
  int64_t nh = 0;
  if (!whole) {
    GCN_TRY(bitmap.alloc(sc, sizeof(uint32_t) * (size_t)words));
    GCN_TRY(wcnt.alloc(sc, sizeof(uint32_t) * (size_t)words));
    GCN_TRY(wprefix.alloc(sc, sizeof(int64_t) * (size_t)(words + 1)));
    GCN_HIP(hipMemsetAsync(bitmap.p, 0, sizeof(uint32_t) * (size_t)words, s));
    if (n_edges > 0) k_validate<<<grid_for(n_edges), kThreads, 0, s>>>(d_src, d_dst, n_edges, n_global, bad.as<int>());
    GCN_CHECK_LAUNCH();
    GCN_HIP(hipMemcpyAsync(read, bad.p, sizeof(int64_t), hipMemcpyDeviceToHost, s));
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

  // -- keys, sort, unique
  const int colbits = bits_for(nc);
  const int rowbits = bits_for(nr);
  if (colbits + rowbits > 62) return fail(GCN_EINVAL, "gcn_csr_build: block too large for 64-bit sort keys");
  DevBuf keys_a, keys_b, cnt, off;
  GCN_TRY(keys_a.alloc(sc, sizeof(uint64_t) * (size_t)m));
  GCN_TRY(keys_b.alloc(sc, sizeof(uint64_t) * (size_t)m));
  k_make_keys<<<grid_for(m), kThreads, 0, s>>>(d_src, d_dst, n_edges, row_lo, row_hi, nr, colbits,
                                                bitmap.as<uint32_t>(), wprefix.as<int64_t>(), keys_a.as<uint64_t>(), bad.as<int>());
  GCN_CHECK_LAUNCH();
  uint64_t* sorted = nullptr;
  GCN_TRY(radix_sort_u64(keys_a.as<uint64_t>(), keys_b.as<uint64_t>(), nullptr, nullptr, m, 0, colbits + rowbits,
                         tmp.p, s, &sorted, nullptr));
  uint64_t* other = (sorted == keys_a.as<uint64_t>()) ? keys_b.as<uint64_t>() : keys_a.as<uint64_t>();
  const int64_t nb = ceil_div(m, kUniqTile);
  GCN_TRY(cnt.alloc(sc, sizeof(uint32_t) * (size_t)nb));
  GCN_TRY(off.alloc(sc, sizeof(int64_t) * (size_t)(nb + 1)));
  k_count_unique<<<fold_grid(nb), kThreads, 0, s>>>(sorted, m, nb, cnt.as<uint32_t>());
  GCN_CHECK_LAUNCH();
  GCN_TRY(exclusive_scan_u32(cnt.as<uint32_t>(), off.as<int64_t>(), nb, tmp.p, s));
  GCN_HIP(hipMemcpyAsync(read, bad.p, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  GCN_HIP(hipMemcpyAsync(read + 1, off.as<int64_t>() + nb, sizeof(int64_t), hipMemcpyDeviceToHost, s));
  GCN_HIP(hipStreamSynchronize(s));
  GCN_TRY(verdict(read[0]));
  const int64_t nnz = read[1];
  if (nnz < nr) return fail(GCN_EHIP, "gcn_csr_build: internal error (nnz %lld < rows %lld)", (long long)nnz, (long long)nr);
  if (nnz >= 0xffffffffLL) return fail(GCN_EINVAL, "gcn_csr_build: more than 2^32-2 stored entries in one block");

  DevBuf rowptr, col, val, deg, dinv;
  GCN_TRY(rowptr.alloc(sc, sizeof(int64_t) * (size_t)(nr + 1)));
  GCN_TRY(col.alloc(sc, sizeof(int32_t) * (size_t)nnz + kEntrySlack));
  GCN_TRY(val.alloc(sc, sizeof(float) * (size_t)nnz + kEntrySlack));
  GCN_TRY(deg.alloc(sc, sizeof(int32_t) * (size_t)nr));
  uint64_t* ukeys = other;                  // unique keys, row-major order
  GCN_TRY(dinv.alloc(sc, sizeof(float) * (size_t)nc));
  k_compact<<<fold_grid(nb), kThreads, 0, s>>>(sorted, off.as<int64_t>(), m, nb, colbits, ukeys, col.as<int32_t>());
  k_boundaries<<<grid_for(nnz), kThreads, 0, s>>>(ukeys, nnz, colbits, ~0ull, nr, rowptr.as<int64_t>());
  k_degrees<<<grid_for(nc), kThreads, 0, s>>>(rowptr.as<int64_t>(), nr, nc, d_deg_global, halo_gid.as<int32_t>(), deg.as<int32_t>(),
                                               dinv.as<float>());
  k_values<<<grid_for(nnz), kThreads, 0, s>>>(ukeys, nnz, colbits, dinv.as<float>(), val.as<float>());
  GCN_CHECK_LAUNCH();

  DevBuf mid;
  if (nh > 0) {
    GCN_TRY(mid.alloc(sc, sizeof(int64_t) * (size_t)nr));
    k_row_mid<<<grid_for(nr), kThreads, 0, s>>>(rowptr.as<int64_t>(), col.as<int32_t>(), nr, mid.as<int64_t>());
    GCN_CHECK_LAUNCH();
  }

  // -- column-major copy
  DevBuf colptr, rowidx, val_t;
  if (flags & GCN_BUILD_CSC) {
    GCN_TRY(colptr.alloc(sc, sizeof(int64_t) * (size_t)(nc + 1)));
    GCN_TRY(rowidx.alloc(sc, sizeof(int32_t) * (size_t)nnz + kEntrySlack));
    GCN_TRY(val_t.alloc(sc, sizeof(float) * (size_t)nnz + kEntrySlack));
    uint64_t* tsorted = nullptr;           // (the buffer of the keys with duplicates is free again)
    GCN_TRY(radix_sort_u64(ukeys, sorted, nullptr, nullptr, nnz, 0, colbits, tmp.p, s, &tsorted, nullptr));
    k_boundaries<<<grid_for(nnz), kThreads, 0, s>>>(tsorted, nnz, 0, (1ull << colbits) - 1ull, nc, colptr.as<int64_t>());
    k_finish_csc<<<grid_for(nnz), kThreads, 0, s>>>(tsorted, nnz, colbits, dinv.as<float>(), rowidx.as<int32_t>(), val_t.as<float>());
    GCN_CHECK_LAUNCH();
  }
  ScheduleBuild by_row, by_col;
  GCN_TRY(by_row.enqueue(rowptr.as<int64_t>(), nr, nnz, sc, read));
  if (flags & GCN_BUILD_CSC) GCN_TRY(by_col.enqueue(colptr.as<int64_t>(), nc, nnz, sc, read + kSchedWords));
  GCN_HIP(hipStreamSynchronize(s));
  sc.done = true;

  A->n_global = n_global; A->row_lo = row_lo;
  A->nr = nr; A->nh = nh; A->nc = nc; A->nnz = nnz;
  by_row.finish(nr, &A->sched);
  if (flags & GCN_BUILD_CSC) by_col.finish(nc, &A->sched_t);
  A->rowptr = (int64_t*)rowptr.release(); A->col = (int32_t*)col.release();
  A->val = (float*)val.release(); A->deg = (int32_t*)deg.release();
  A->halo_gid = (int32_t*)halo_gid.release();
  A->colptr = (int64_t*)colptr.release(); A->rowidx = (int32_t*)rowidx.release();
  A->val_t = (float*)val_t.release();
  A->mid = nh > 0 ? (int64_t*)mid.release() : nullptr;
  return GCN_OK;
}

int segment_boundaries(const uint64_t* keys, int64_t n, int shift, int64_t n_seg, int64_t* ptr, hipStream_t s) {
  if (n < 1) return fail(GCN_EINVAL, "segment_boundaries: empty input");
  k_boundaries<<<grid_for(n), kThreads, 0, s>>>(keys, n, shift, ~0ull, n_seg, ptr);
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
