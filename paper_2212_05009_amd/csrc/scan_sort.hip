// Device-wide exclusive scan and stable LSD radix sort for gfx950 (64-wide wavefronts).
// These are the integer building blocks of the CSR / CSC / halo-list construction; all of
// their results are order-deterministic (no floating point, no order-dependent atomics).
#include <algorithm>

#include "common.h"

namespace gcn {

// ------------------------------------------------------------------------------------------
// Exclusive scan, uint32 in -> int64 out, reduce-then-scan: block sums, then every block adds up the sums before its own
// (up to kScanFewBlocks blocks) or finds them scanned by a launch of their own.  The scans of a graph build are short (a
// few hundred blocks) and there are a dozen of them: what counts is the launch, about 5 us.
// ------------------------------------------------------------------------------------------
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ __forceinline__ int64_t wave_inclusive_scan(int64_t v, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    int64_t o = __shfl_up(v, off, 64);
    if (lane >= off) v += o;
  }
  return v;
}

// exclusive prefix of `v` over the THREADS threads of the block; *total = block sum
template <int THREADS = kScanThreads>
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* total) {
  __shared__ int64_t wave_tot[THREADS / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t inc = wave_inclusive_scan(v, lane);
  if (lane == 63) wave_tot[w] = inc;
  __syncthreads();
  int64_t base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) {
    int64_t t = wave_tot[i];
    if (i < w) base += t;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const uint32_t* __restrict__ in,
                                                              int64_t n, int64_t* __restrict__ sums) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x;
  int64_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i)
    if (base + i * kScanThreads < n) s += in[base + i * kScanThreads];
  int64_t tot;
  block_exclusive_scan(s, &tot);
  if (threadIdx.x == 0) sums[blockIdx.x] = tot;
}

// one block: in-place exclusive scan of sums[0..m); writes the grand total to *total_out
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(int64_t* __restrict__ sums, int64_t m,
                                                            int64_t* __restrict__ total_out) {
  int64_t carry = 0;
  for (int64_t c0 = 0; c0 < m; c0 += kScanThreads) {
    int64_t i = c0 + threadIdx.x;
    int64_t v = i < m ? sums[i] : 0;
    int64_t tot;
    int64_t ex = block_exclusive_scan(v, &tot);
    if (i < m) sums[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) *total_out = carry;
}

// SCANNED: sums[b] is the sum of all blocks before b; else it is block b's own, and the last block writes the total
template <bool SCANNED>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const uint32_t* __restrict__ in,
                                                             int64_t n, const int64_t* __restrict__ sums,
                                                             int64_t* __restrict__ out) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  int64_t s = 0;
  // a thread's items are 64 bytes of the input and 128 of the output: whole requests where the arrays start on 16 bytes
  const bool wide = base + kScanItems <= n && (((uintptr_t)in | (uintptr_t)out) & 15) == 0;
  if (wide) {
#pragma unroll
    for (int i = 0; i < kScanItems; i += 4) {
      const uint4 x = *reinterpret_cast<const uint4*>(in + base + i);
      v[i] = x.x; v[i + 1] = x.y; v[i + 2] = x.z; v[i + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) v[i] = (base + i < n) ? in[base + i] : 0u;
  }
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) s += v[i];
  int64_t before;
  if constexpr (SCANNED) {
    before = sums[blockIdx.x];
  } else {
    int64_t p = 0;
    for (int64_t i = threadIdx.x; i < blockIdx.x; i += kScanThreads) p += sums[i];
    block_exclusive_scan(p, &before);
  }
  int64_t tot;
  int64_t run = before + block_exclusive_scan(s, &tot);
  if (!SCANNED && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = before + tot;
  if (wide) {
#pragma unroll
    for (int i = 0; i < kScanItems; i += 2) {
      longlong2 y;
      y.x = run;
      y.y = run + v[i];
      run = y.y + v[i + 1];
      *reinterpret_cast<longlong2*>(out + base + i) = y;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      if (base + i < n) out[base + i] = run;
      run += v[i];
    }
  }
}

// One block for all of a short input: one launch instead of two.  A wavefront takes consecutive runs of 256 items (64 requests
// of 16 bytes) and asks for all of them before it adds up the first: what bounds this is one round trip to memory.
constexpr int kScanOneThreads = 1024;
constexpr int kScanOneRuns = 8;
constexpr int64_t kScanOneMax = kScanOneThreads / 64 * kScanOneRuns * 256;
__global__ __launch_bounds__(kScanOneThreads) void k_scan_one(const uint32_t* __restrict__ in, int64_t n, int runs, int64_t* __restrict__ out) {
  __shared__ int64_t wave_tot[kScanOneThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t base = (int64_t)w * runs * 256 + 4 * lane;
  uint4 v[kScanOneRuns];
  int64_t before[kScanOneRuns], sum = 0;
#pragma unroll
  for (int i = 0; i < kScanOneRuns; ++i) {
    const int64_t p = base + 256 * i;
    v[i] = make_uint4(0, 0, 0, 0);
    if (i >= runs) continue;
    if (p + 4 <= n && ((uintptr_t)in & 15) == 0) v[i] = *reinterpret_cast<const uint4*>(in + p);
    else {
      if (p < n) v[i].x = in[p];
      if (p + 1 < n) v[i].y = in[p + 1];
      if (p + 2 < n) v[i].z = in[p + 2];
      if (p + 3 < n) v[i].w = in[p + 3];
    }
  }
#pragma unroll
  for (int i = 0; i < kScanOneRuns; ++i) {
    if (i >= runs) continue;
    const int64_t mine = (int64_t)v[i].x + v[i].y + v[i].z + v[i].w;
    const int64_t inc = wave_inclusive_scan(mine, lane);
    before[i] = sum + inc - mine;
    sum += __shfl(inc, 63, 64);
  }
  if (lane == 0) wave_tot[w] = sum;
  __syncthreads();
  int64_t first = 0, total = 0;
#pragma unroll
  for (int i = 0; i < kScanOneThreads / 64; ++i) {
    if (i < w) first += wave_tot[i];
    total += wave_tot[i];
  }
#pragma unroll
  for (int i = 0; i < kScanOneRuns; ++i) {
    const int64_t p = base + 256 * i;
    if (i >= runs) continue;
    int64_t run = first + before[i];
    const uint32_t x[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (p + k < n) out[p + k] = run;
      run += x[k];
    }
  }
  if (threadIdx.x == 0) out[n] = total;
}

constexpr int64_t kScanFewBlocks = 1024;         // (a block then reads at most 8 KB of sums)

size_t scan_tmp_bytes(int64_t n) { return sizeof(int64_t) * (size_t)(ceil_div(n > 0 ? n : 1, kScanTile) + 1); }

int exclusive_scan_u32(const uint32_t* in, int64_t* out, int64_t n, void* tmp, hipStream_t s) {
  if (n < 0) return fail(GCN_EINVAL, "scan: negative size");
  if (n == 0) {
    GCN_HIP(hipMemsetAsync(out, 0, sizeof(int64_t), s));
    return GCN_OK;
  }
  const int64_t nb = ceil_div(n, kScanTile);
  if (nb * kScanThreads >= ((int64_t)1 << 32)) return fail(GCN_EINVAL, "scan: input too large for one launch");
  if (n <= kScanOneMax) {
    k_scan_one<<<dim3(1), dim3(kScanOneThreads), 0, s>>>(in, n, (int)ceil_div(n, kScanOneThreads / 64 * 256), out);
    GCN_CHECK_LAUNCH();
    return GCN_OK;
  }
  int64_t* sums = (int64_t*)tmp;
  k_scan_reduce<<<dim3((unsigned)nb), dim3(kScanThreads), 0, s>>>(in, n, sums);
  if (nb <= kScanFewBlocks) {
    k_scan_apply<false><<<dim3((unsigned)nb), dim3(kScanThreads), 0, s>>>(in, n, sums, out);
  } else {
    k_scan_sums<<<dim3(1), dim3(kScanThreads), 0, s>>>(sums, nb, out + n);
    k_scan_apply<true><<<dim3((unsigned)nb), dim3(kScanThreads), 0, s>>>(in, n, sums, out);
  }
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

// ------------------------------------------------------------------------------------------
// Stable LSD radix sort.
// Per pass: (1) per-block digit histogram, (2) the output offset of each (digit, block), (3) every block ranks its keys
// stably, orders them in LDS and writes them out digit by digit.  Stability inside a block: a wavefront owns a contiguous run
// of keys and walks it 64 keys at a time; keys with equal digits inside one step are ordered by lane
// (ballot match + popcount of lower lanes), steps are ordered by a running per-wave counter,
// waves are ordered by a prefix over the per-wave counters.
// A pass is bound by its writes: without the LDS step a wavefront's 64 keys go to up to 64 places, 8 bytes each; with it
// the keys of a block leave in runs of 12 on the average, 96 bytes (long inputs).
// Three launch shapes by the number of keys:
//   from 2^21 on    digits of up to 9 bits, 6144 keys per block (12 keys a digit; LDS for two blocks a compute unit): 18 and
//                   36 bits, R-MAT 2^18, take 2 and 4 passes for the 3 and 5 of 8 bits.  Scatter of 13.2 M keys: 8 bits, 4096
//                   keys 58 us; 9 bits, 4096 / 6144 / 8192 keys 72 / 71 / 121; histogram and scan are another 35 us either
//                   way.  The offsets are a scan of the digit-major table, two launches of their own.
//   below           digits of up to 8 bits, 2048 keys per block, so that compute units are not left without one;
//   up to 512 such blocks  no scan: a block adds up the block-major table itself (at most 512 KB out of L2 per block, less
//                   than the two launches it saves).
// With a device-side count (`count`) the host's n is a bound: blocks behind the count have nothing to do.  DROP leaves out
// keys of all ones and writes how many are left to `kept`.
// ------------------------------------------------------------------------------------------
constexpr int kSortThreads = 256, kSortItems = 8, kSortBits = 8;
constexpr int kSortBigThreads = 512, kSortBigItems = 12, kSortBigBits = 9;
constexpr int64_t kSortBigFrom = (int64_t)1 << 21;
constexpr int64_t kSortOwnBlocks = 512;
static_assert(kSortThreads == 1 << kSortBits && kSortBigThreads == 1 << kSortBigBits, "a thread of a block keeps one digit");

struct SortPass {
  const uint64_t* keys_in; uint64_t* keys_out;
  const uint32_t* pay_in; uint32_t* pay_out;
  int64_t n; const int64_t* count;       // keys: n, or *count <= n where given
  int64_t* kept;                         // DROP: number of keys that are not all ones
  int shift; uint32_t mask;
  int64_t nblocks;
  uint32_t* hist;                        // [nblocks][digits] where a block finds its offsets itself, else [digits][nblocks]
  const int64_t* offsets;                // scanned digit-major table, or null
};

template <int THREADS, int ITEMS, bool DROP>
__global__ __launch_bounds__(THREADS) void k_sort_hist(SortPass a) {
  __shared__ uint32_t h[THREADS];
  const int64_t n = a.count ? *a.count : a.n;
  const int64_t base = (int64_t)blockIdx.x * THREADS * ITEMS;
  if (!a.offsets && base >= n) return;
  h[threadIdx.x] = 0;
  __syncthreads();
  uint64_t key[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int64_t idx = base + (int64_t)i * THREADS + threadIdx.x;
    key[i] = idx < n ? a.keys_in[idx] : 0ull;
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int64_t idx = base + (int64_t)i * THREADS + threadIdx.x;
    if (idx < n && !(DROP && key[i] == ~0ull)) atomicAdd(&h[(uint32_t)(key[i] >> a.shift) & a.mask], 1u);
  }
  __syncthreads();
  a.hist[a.offsets ? (int64_t)threadIdx.x * a.nblocks + blockIdx.x : (int64_t)blockIdx.x * THREADS + threadIdx.x] = h[threadIdx.x];
}

template <int THREADS, int ITEMS, bool PAY, bool DROP>
__global__ __launch_bounds__(THREADS) void k_sort_scatter(SortPass a) {
  constexpr int WAVES = THREADS / 64, TILE = THREADS * ITEMS;
  constexpr int kBits = THREADS == 512 ? 9 : 8;
  __shared__ uint32_t wave_cnt[WAVES][THREADS];
  __shared__ uint32_t digit_base[THREADS];         // output position of the digit's first key, less its position in the block
  __shared__ uint64_t stage[TILE];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
  const int64_t n = a.count ? *a.count : a.n;
  const int64_t tile_base = (int64_t)blockIdx.x * TILE;
  if (tile_base >= n && !(DROP && blockIdx.x == 0)) return;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) wave_cnt[i][t] = 0;

  const int64_t wave_base = tile_base + (int64_t)w * 64 * ITEMS;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint64_t key[ITEMS];
  uint32_t pay[ITEMS];
  uint32_t rank[ITEMS];
  auto valid = [&](int it) { return wave_base + (int64_t)it * 64 + lane < n && !(DROP && key[it] == ~0ull); };
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int64_t idx = wave_base + (int64_t)it * 64 + lane;
    key[it] = idx < n ? a.keys_in[idx] : 0ull;
    if constexpr (PAY) pay[it] = idx < n ? a.pay_in[idx] : 0u;
  }
  // the offset of this thread's digit
  int64_t before;
  if (a.offsets) {
    before = a.offsets[(int64_t)t * a.nblocks + blockIdx.x];
  } else {
    // a wavefront adds up every WAVES-th block's row of the table, four digits a lane, then the wavefronts meet in LDS
    constexpr int PART = THREADS / 64 / 4;         // wavefronts side by side on a row
    static_assert(PART * 4 * 64 == THREADS && WAVES * THREADS * 8 <= TILE * 8, "a lane has four digits; the sums fit the staging area");
    uint2* sums = reinterpret_cast<uint2*>(stage);
    const int nb = (int)((n + TILE - 1) / TILE), mine = (int)blockIdx.x;
    const int dq = (w % PART) * 64 + lane;
    uint32_t lo[4] = {0, 0, 0, 0}, all[4] = {0, 0, 0, 0};
#pragma unroll 8
    for (int b = w / PART; b < nb; b += WAVES / PART) {
      const uint4 v = *reinterpret_cast<const uint4*>(a.hist + (int64_t)b * THREADS + 4 * dq);
      const uint32_t x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) { all[k] += x[k]; lo[k] += b < mine ? x[k] : 0u; }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sums[(w / PART) * THREADS + 4 * dq + k] = make_uint2(lo[k], all[k]);
    __syncthreads();
    uint32_t own_lo = 0, own_all = 0;
#pragma unroll
    for (int i = 0; i < WAVES / PART; ++i) { own_lo += sums[i * THREADS + t].x; own_all += sums[i * THREADS + t].y; }
    int64_t total;
    before = (int64_t)own_lo + block_exclusive_scan<THREADS>((int64_t)own_all, &total);
    if (DROP && blockIdx.x == 0 && t == 0) *a.kept = total;
  }
  if (DROP && a.offsets && blockIdx.x == 0 && t == 0) *a.kept = a.offsets[(int64_t)THREADS * a.nblocks];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const bool ok = valid(it);
    const uint32_t dg = (uint32_t)(key[it] >> a.shift) & a.mask;
    uint64_t peers = __ballot(ok);
#pragma unroll
    for (int b = 0; b < kBits; ++b) {
      const bool bit = (dg >> b) & 1u;
      const uint64_t bal = __ballot(ok && bit);
      peers &= bit ? bal : ~bal;
    }
    // peers: valid lanes of this step with the same digit (includes this lane when valid)
    const int leader = ok ? (__ffsll((unsigned long long)peers) - 1) : 0;
    uint32_t base = 0;
    if (ok && lane == leader) {
      base = wave_cnt[w][dg];
      wave_cnt[w][dg] = base + (uint32_t)__popcll(peers);
    }
    base = __shfl(base, leader, 64);
    rank[it] = base + (uint32_t)__popcll(peers & lt_mask);
  }
  __syncthreads();
  int here;                                        // valid keys of the block: they take the places 0 .. here - 1
  {
    uint32_t run = 0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) run += wave_cnt[i][t];
    int64_t total;
    const uint32_t first = (uint32_t)block_exclusive_scan<THREADS>((int64_t)run, &total);
    here = (int)total;
    digit_base[t] = (uint32_t)before - first;      // (positions are below 2^32; the difference may wrap)
    run = first;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const uint32_t c = wave_cnt[i][t];
      wave_cnt[i][t] = run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    rank[it] += wave_cnt[w][(uint32_t)(key[it] >> a.shift) & a.mask];
    if (valid(it)) stage[rank[it]] = key[it];
  }
  __syncthreads();
  uint32_t dst[ITEMS];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int pos = it * THREADS + t;
    if (pos < here) {
      const uint64_t k = stage[pos];
      dst[it] = digit_base[(uint32_t)(k >> a.shift) & a.mask] + (uint32_t)pos;
      a.keys_out[dst[it]] = k;
    }
  }
  if constexpr (PAY) {
    uint32_t* pstage = reinterpret_cast<uint32_t*>(stage);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
      if (valid(it)) pstage[rank[it]] = pay[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int pos = it * THREADS + t;
      if (pos < here) a.pay_out[dst[it]] = pstage[pos];
    }
  }
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// entries of the offset table of the sort of n keys
static int64_t sort_table(int64_t n) {
  const bool big = n >= kSortBigFrom;
  return big ? kSortBigThreads * ceil_div(n, kSortBigThreads * kSortBigItems) : kSortThreads * ceil_div(n > 0 ? n : 1, kSortThreads * kSortItems);
}

// (a sort of fewer keys may need the larger table of the short blocks)
size_t sort_tmp_bytes(int64_t n) {
  const int64_t m = std::max(sort_table(n), sort_table(std::min<int64_t>(n, kSortBigFrom - 1)));
  return align256(sizeof(uint32_t) * (size_t)m) + align256(sizeof(int64_t) * (size_t)(m + 1)) +
         align256(scan_tmp_bytes(m));
}

template <int THREADS, int ITEMS>
static int sort_pass(SortPass a, bool drop, int64_t* offsets, void* scan_tmp, hipStream_t s) {
  const dim3 grid((unsigned)a.nblocks), block(THREADS);
  a.offsets = offsets;
  if (drop) k_sort_hist<THREADS, ITEMS, true><<<grid, block, 0, s>>>(a);
  else k_sort_hist<THREADS, ITEMS, false><<<grid, block, 0, s>>>(a);
  if (offsets) GCN_TRY(exclusive_scan_u32(a.hist, offsets, THREADS * a.nblocks, scan_tmp, s));
  if (a.pay_in) k_sort_scatter<THREADS, ITEMS, true, false><<<grid, block, 0, s>>>(a);
  else if (drop) k_sort_scatter<THREADS, ITEMS, false, true><<<grid, block, 0, s>>>(a);
  else k_sort_scatter<THREADS, ITEMS, false, false><<<grid, block, 0, s>>>(a);
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

int radix_sort_u64(uint64_t* keys_a, uint64_t* keys_b, uint32_t* pay_a, uint32_t* pay_b, int64_t n,
                   int bit_lo, int bit_hi, void* tmp, hipStream_t s, uint64_t** keys_out,
                   uint32_t** pay_out, const int64_t* count, int64_t* kept) {
  if (n < 0 || bit_lo < 0 || bit_hi > 64 || bit_hi < bit_lo || n >= ((int64_t)1 << 32)) return fail(GCN_EINVAL, "sort: bad arguments");
  if (kept && (pay_a || bit_hi == bit_lo || n == 0)) return fail(GCN_EINVAL, "sort: keys are only left out in a pass over plain keys");
  SortPass a{};
  a.keys_in = keys_a; a.keys_out = keys_b;
  a.pay_in = pay_a; a.pay_out = pay_a ? pay_b : nullptr;
  if (n > 0) {
    const bool big = n >= kSortBigFrom;
    a.n = n; a.count = count; a.kept = kept;
    a.nblocks = ceil_div(n, big ? kSortBigThreads * kSortBigItems : kSortThreads * kSortItems);
    const int64_t m = sort_table(n);
    a.hist = (uint32_t*)tmp;
    int64_t* offsets = (int64_t*)((char*)tmp + align256(sizeof(uint32_t) * (size_t)m));
    void* scan_tmp = (char*)offsets + align256(sizeof(int64_t) * (size_t)(m + 1));
    if (!big && a.nblocks <= kSortOwnBlocks) offsets = nullptr;
    int passes = (int)ceil_div(bit_hi - bit_lo, big ? kSortBigBits : kSortBits);
    for (int shift = bit_lo; shift < bit_hi; --passes) {
      const int bits = (int)ceil_div(bit_hi - shift, passes);
      const bool drop = kept && shift == bit_lo;
      a.shift = shift; a.mask = (1u << bits) - 1u;
      if (big) GCN_TRY((sort_pass<kSortBigThreads, kSortBigItems>(a, drop, offsets, scan_tmp, s)));
      else GCN_TRY((sort_pass<kSortThreads, kSortItems>(a, drop, offsets, scan_tmp, s)));
      if (drop) a.count = kept;            // the rest of the passes see the keys that are left
      shift += bits;
      uint64_t* tk = a.keys_out; a.keys_out = const_cast<uint64_t*>(a.keys_in); a.keys_in = tk;
      uint32_t* tp = a.pay_out; a.pay_out = const_cast<uint32_t*>(a.pay_in); a.pay_in = tp;
    }
  }
  *keys_out = const_cast<uint64_t*>(a.keys_in);
  if (pay_out) *pay_out = const_cast<uint32_t*>(a.pay_in);
  return GCN_OK;
}

}  // namespace gcn
