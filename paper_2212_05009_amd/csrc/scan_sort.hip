// Device-wide exclusive scan and stable LSD radix sort for gfx950 (64-wide wavefronts).
// These are the integer building blocks of the CSR / CSC / halo-list construction; all of
// their results are order-deterministic (no floating point, no order-dependent atomics).
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

// exclusive prefix of `v` over the 256 threads of the block; *total = block sum
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* total) {
  __shared__ int64_t wave_tot[kScanThreads / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t inc = wave_inclusive_scan(v, lane);
  if (lane == 63) wave_tot[w] = inc;
  __syncthreads();
  int64_t base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kScanThreads / 64; ++i) {
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
// Stable LSD radix sort, 8 bits per pass.
// Per pass: (1) per-block digit histogram, (2) exclusive scan of the digit-major histogram
// table gives each (digit, block) its output offset, (3) every block ranks its keys stably,
// orders them in LDS and writes them out digit by digit.  Stability inside a block: a wavefront owns a contiguous run
// of keys and walks it 64 keys at a time; keys with equal digits inside one step are ordered by lane
// (ballot match + popcount of lower lanes), steps are ordered by a running per-wave counter,
// waves are ordered by a prefix over the per-wave counters.
// A pass is bound by its writes: without the LDS step a wavefront's 64 keys go to up to 64 places, 8 bytes each; with it
// the 4096 keys of a block leave in runs of 16 on the average, 128 bytes.
// ------------------------------------------------------------------------------------------
constexpr int kSortThreads = 256;
static_assert(kSortThreads == kScanThreads, "k_sort_scatter scans one value per digit with block_exclusive_scan");
// Keys per thread: 16, or 8 where that would leave compute units without a block (fewer than two each).
static inline int sort_items(int64_t n) { return n >= (int64_t)2 * 256 * kSortThreads * 16 ? 16 : 8; }
static inline int64_t sort_blocks(int64_t n) { return ceil_div(n > 0 ? n : 1, (int64_t)kSortThreads * sort_items(n)); }

template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const uint64_t* __restrict__ keys,
                                                            int64_t n, int shift, uint32_t mask, int64_t nblocks,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortThreads * ITEMS;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    int64_t idx = base + (int64_t)i * kSortThreads + threadIdx.x;
    if (idx < n) atomicAdd(&h[(uint32_t)(keys[idx] >> shift) & mask], 1u);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

template <int ITEMS, bool PAY>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(
    const uint64_t* __restrict__ keys_in, uint64_t* __restrict__ keys_out,
    const uint32_t* __restrict__ pay_in, uint32_t* __restrict__ pay_out, int64_t n, int shift, uint32_t mask,
    int64_t nblocks, const int64_t* __restrict__ offsets) {
  __shared__ uint32_t wave_cnt[kSortThreads / 64][256];
  __shared__ int64_t digit_base[256];              // output position of the digit's first key, less its position in the block
  __shared__ uint64_t stage[kSortThreads * ITEMS];
  const int t = threadIdx.x, w = t >> 6, lane = t & 63;
#pragma unroll
  for (int i = 0; i < kSortThreads / 64; ++i) wave_cnt[i][t] = 0;
  __syncthreads();

  const int64_t tile_base = (int64_t)blockIdx.x * kSortThreads * ITEMS;
  const int64_t wave_base = tile_base + (int64_t)w * 64 * ITEMS;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint64_t key[ITEMS];
  uint32_t pay[ITEMS];
  uint32_t rank[ITEMS];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int64_t idx = wave_base + (int64_t)it * 64 + lane;
    key[it] = idx < n ? keys_in[idx] : 0ull;
    if constexpr (PAY) pay[it] = idx < n ? pay_in[idx] : 0u;
  }
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const bool valid = wave_base + (int64_t)it * 64 + lane < n;
    const uint32_t dg = (uint32_t)(key[it] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (dg >> b) & 1u;
      const uint64_t bal = __ballot(valid && bit);
      peers &= bit ? bal : ~bal;
    }
    // peers: valid lanes of this step with the same digit (includes this lane when valid)
    const int leader = valid ? (__ffsll((unsigned long long)peers) - 1) : 0;
    uint32_t base = 0;
    if (valid && lane == leader) {
      base = wave_cnt[w][dg];
      wave_cnt[w][dg] = base + (uint32_t)__popcll(peers);
    }
    base = __shfl(base, leader, 64);
    rank[it] = base + (uint32_t)__popcll(peers & lt_mask);
  }
  __syncthreads();
  {
    uint32_t run = 0;
#pragma unroll
    for (int i = 0; i < kSortThreads / 64; ++i) run += wave_cnt[i][t];
    int64_t total;
    const uint32_t first = (uint32_t)block_exclusive_scan((int64_t)run, &total);
    digit_base[t] = offsets[(int64_t)t * nblocks + blockIdx.x] - (int64_t)first;
    run = first;
#pragma unroll
    for (int i = 0; i < kSortThreads / 64; ++i) {
      uint32_t c = wave_cnt[i][t];
      wave_cnt[i][t] = run;
      run += c;
    }
  }
  __syncthreads();
  // the valid keys of the block take the places 0 .. here - 1
  const int here = (int)(n - tile_base < kSortThreads * ITEMS ? n - tile_base : kSortThreads * ITEMS);
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    rank[it] += wave_cnt[w][(uint32_t)(key[it] >> shift) & mask];
    if (wave_base + (int64_t)it * 64 + lane < n) stage[rank[it]] = key[it];
  }
  __syncthreads();
  int64_t dst[ITEMS];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int pos = it * kSortThreads + t;
    if (pos < here) {
      const uint64_t k = stage[pos];
      dst[it] = digit_base[(uint32_t)(k >> shift) & mask] + pos;
      keys_out[dst[it]] = k;
    }
  }
  if constexpr (PAY) {
    uint32_t* pstage = reinterpret_cast<uint32_t*>(stage);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it)
      if (wave_base + (int64_t)it * 64 + lane < n) pstage[rank[it]] = pay[it];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITEMS; ++it) {
      const int pos = it * kSortThreads + t;
      if (pos < here) pay_out[dst[it]] = pstage[pos];
    }
  }
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// (for 8 keys per thread: enough for any sort of at most n keys)
size_t sort_tmp_bytes(int64_t n) {
  const int64_t m = 256 * ceil_div(n > 0 ? n : 1, (int64_t)kSortThreads * 8);
  return align256(sizeof(uint32_t) * (size_t)m) + align256(sizeof(int64_t) * (size_t)(m + 1)) +
         align256(scan_tmp_bytes(m));
}

template <int ITEMS>
static void sort_pass(const uint64_t* kin, uint64_t* kout, const uint32_t* pin, uint32_t* pout, int64_t n, int shift,
                      uint32_t mask, int64_t nb, const int64_t* offsets, hipStream_t s) {
  if (pin) k_sort_scatter<ITEMS, true><<<dim3((unsigned)nb), dim3(kSortThreads), 0, s>>>(kin, kout, pin, pout, n, shift, mask, nb, offsets);
  else k_sort_scatter<ITEMS, false><<<dim3((unsigned)nb), dim3(kSortThreads), 0, s>>>(kin, kout, nullptr, nullptr, n, shift, mask, nb, offsets);
}

int radix_sort_u64(uint64_t* keys_a, uint64_t* keys_b, uint32_t* pay_a, uint32_t* pay_b, int64_t n,
                   int bit_lo, int bit_hi, void* tmp, hipStream_t s, uint64_t** keys_out,
                   uint32_t** pay_out) {
  if (n < 0 || bit_lo < 0 || bit_hi > 64 || bit_hi < bit_lo) return fail(GCN_EINVAL, "sort: bad arguments");
  uint64_t* kin = keys_a; uint64_t* kout = keys_b;
  uint32_t* pin = pay_a;  uint32_t* pout = pay_a ? pay_b : nullptr;
  if (n > 0) {
    const int64_t nb = sort_blocks(n);
    if (nb * kSortThreads >= ((int64_t)1 << 32)) return fail(GCN_EINVAL, "sort: input too large for one launch");
    const int64_t m = 256 * nb;
    const bool big = sort_items(n) == 16;
    char* p = (char*)tmp;
    uint32_t* hist = (uint32_t*)p;          p += align256(sizeof(uint32_t) * (size_t)m);
    int64_t* offsets = (int64_t*)p;         p += align256(sizeof(int64_t) * (size_t)(m + 1));
    void* scan_tmp = p;
    for (int shift = bit_lo; shift < bit_hi; shift += 8) {
      const uint32_t mask = bit_hi - shift >= 8 ? 255u : (1u << (bit_hi - shift)) - 1u;     // no bit from bit_hi on counts
      if (big) k_sort_hist<16><<<dim3((unsigned)nb), dim3(kSortThreads), 0, s>>>(kin, n, shift, mask, nb, hist);
      else k_sort_hist<8><<<dim3((unsigned)nb), dim3(kSortThreads), 0, s>>>(kin, n, shift, mask, nb, hist);
      GCN_TRY(exclusive_scan_u32(hist, offsets, m, scan_tmp, s));
      if (big) sort_pass<16>(kin, kout, pin, pout, n, shift, mask, nb, offsets, s);
      else sort_pass<8>(kin, kout, pin, pout, n, shift, mask, nb, offsets, s);
      GCN_CHECK_LAUNCH();
      uint64_t* tk = kin; kin = kout; kout = tk;
      uint32_t* tp = pin; pin = pout; pout = tp;
    }
  }
  *keys_out = kin;
  if (pay_out) *pay_out = pin;
  return GCN_OK;
}

}  // namespace gcn
