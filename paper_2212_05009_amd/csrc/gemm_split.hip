// C[M x N] = A[M x K] W^T and dW = A^T B of fp32 operands on the bf16 matrix pipe (Sec. 3.2: the gradient handed down and that of W^k), for
// products whose arithmetic takes longer than their bytes on the fp32 pipe.  Not the forward pass's H W: what it rounds otherwise changes
// the sign of hidden values next to zero, and each such sign switches an element of the gradient on or off (neighbourhoods of 490: 3.5e-4 of
// dW's norm, next to nothing of it error), so that a training step would not repeat what it gave.
//
// An fp32 value from 2^-108 on is the exact sum of three bf16 values: its rounding, the rounding of what is left (2^-8 of it at most), and of
// what is then left (2^-17; 24 bits of significand are 3 x 8).  Products with smaller operands are formed on the fp32 pipe.  A product of two values is nine products, of which the six of weight 2^-18 and
// more are formed, each exact in fp32, and added by the matrix pipe in fp32: what is left out is up to 2^-24 of the product, 2^-27 as a
// rule (a rounding: up to 2^-24, 2^-25 as a rule).  Six bf16 operations at sixteen times the fp32 rate: the products are then bound by memory.
#include <algorithm>
#include <type_traits>

#include "rows_buf.h"

namespace gcn {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4w __attribute__((ext_vector_type(4), aligned(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct SplitArgs {
  const float* A; int64_t lda; const float* W; int64_t ldw; float* C; int64_t ldc;
  int64_t M; int N; int K;
  const float* mask; int64_t ldmask; int64_t mask_rows;
  int endC;                // nothing beyond column N of C may be written
};

// The six products of parts, the smallest first.  The matrix pipe aligns what it adds to the largest term and cuts off the rest, downwards: each
// step's sum starts from zero and is added to the result by a rounded fp32 addition.  (Sums carried through the pipe over all steps: error of a
// 256 x 256 gradient over 2.45 M rows 7.8e-6, 1.7e-6 on the fp32 pipe.)  The first parts' products are added by themselves, and to the others by
// another rounded addition, or the pipe would cut the last bits of sums of few terms: one nonzero term of K 3.5e-8, this way 2.6e-8, as on the
// fp32 pipe (2.5e-8); two to eight of 602 3.7e-8 .. 5.7e-8 for 3.1e-8 .. 5.4e-8, more terms less than there.  What is cut has the same sign everywhere, which no sum over
// rows averages out: operands are taken with the other sign in every other step, and in rows of every other number of bits.  The product of 602
// terms, summed over 512 rows as a sparse product sums it: 6.2e-7 off with one sign for all, 9.3e-8 with both, 4.4e-7 on the fp32 pipe; results
// of a two-layer forward pass over neighbourhoods of 490: 7.4e-7, 6.5e-8 and 9e-8.
__device__ constexpr int kTerm[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;
constexpr int kRT = 2;                                 // tiles of 16 rows of a wavefront

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  const bf16x2 h = __builtin_convertvector(floatx2{lo, hi}, bf16x2);
  uint32_t u;
  __builtin_memcpy(&u, &h, 4);
  return u;
}
// {lo, hi} = the values of p[0] + p[1] + p[2]
__device__ __forceinline__ void split2(float lo, float hi, uint32_t (&p)[3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    p[k] = pack_bf16(lo, hi);
    lo -= __uint_as_float(p[k] << 16);
    hi -= __uint_as_float(p[k] & 0xffff0000u);
  }
}
// What the parts of v lack
__device__ __forceinline__ float left_over(float v) {
#pragma unroll
  for (int k = 0; k < 3; ++k) v -= __uint_as_float(pack_bf16(v, 0.f) << 16);
  return v;
}
// Sums that are no finite number (a value beyond the bf16 range, an infinity, a NaN: inf = inf + NaN in parts), or below 2^-90 and not zero: products of
// parts may lie under the smallest fp32 number.
struct RangeCheck {
  uint32_t most = 0u, least = 0xffffffffu;             // least: of the sums that are not zero, less one
  __device__ __forceinline__ void add(float v) {
    const uint32_t b = __float_as_uint(v) & 0x7fffffffu;
    most = b > most ? b : most;
    least = b - 1u < least ? b - 1u : least;
  }
  __device__ __forceinline__ bool out() const { return most >= 0x7f800000u || least < ((127u - 90u) << 23) - 1u; }
};
// The least magnitude of operands that are not zero.  The last part of one below 2^-108 may have bits under the smallest bf16 number (2^-133); what a
// sum looks like says nothing about it, the other operand may be large.  Three integer operations for two values: 602 -> 128 on 233 K rows 256 ->
// 278 us, 256 -> 256 on 2.45 M 2.03 -> 2.10 ms (both with W stored [K x N]), A^T B 602 x 128 344 -> 350 us.
struct LeastOperand {
  uint32_t least = 0xffffffffu;                        // twice the bits, less one: zero is the largest
  __device__ __forceinline__ void add(float lo, float hi) {
    const uint32_t a = 2u * __float_as_uint(lo) - 1u, b = 2u * __float_as_uint(hi) - 1u;
    const uint32_t c = a < b ? a : b;
    least = c < least ? c : least;
  }
  __device__ __forceinline__ bool out() const { return least < 2u * ((127u - 108u) << 23) - 1u; }
};
__device__ __forceinline__ floatx4 mfma(const u32x4& w, const u32x4& x, floatx4 acc) {
  bf16x8 a, b;
  __builtin_memcpy(&a, &w, 16); __builtin_memcpy(&b, &x, 16);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}
// meets the workgroup for LDS alone: global requests stay in flight
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// What bounds it: a wavefront's own instructions, of the matrix and the vector pipe in turn (two wavefronts a SIMD), and the clock.  2.45 M rows x
// 256 x 256: 2.28 ms, the matrix pipe busy for 34 % of what the nominal clock has (at 1.8 GHz; 2.2 in kernels that wait for memory).  While a
// step is multiplied (192 operations a wavefront at 256 columns) the next one is split, in their shadow, and the one after asked for, its
// own registers' places as they fall free.  Bare sums took 1.68 ms (1.96 with splitting first and multiplying then; 2.42 with W in plain loads, their
// addresses in registers, spilled); 1.80 with the sums of each step added by vector operations, without which the error grows to that of the fp32 pipe
// and beyond (terms of one sign); 2.28 with the other sign in every other step and row, the first parts' products by themselves, and small operands
// found.
// Lane (c, q) = (lane % 16, lane / 16) supplies row c of a tile of 16 rows, k = 8 q .. 8 q + 7 of a step of 32, as the second
// MFMA operand and column 16 t + c of W as the first: register r of its accumulator t is column 16 t + 4 q + r of row c.
// LDS holds W as operands, [step][tile][part][lane], 16 bytes each: all of it (RES), or two steps in turn, which the workgroup reads
// from L2 and splits again for every pass over its rows.
template <int NT, bool RES, bool MASK>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_nn_split(SplitArgs a) {
  extern __shared__ u32x4 split_lds[];
  constexpr int kStep = NT * 3 * 64;                   // u32x4 of a step of W
  constexpr int kPieces = (NT * 64 + kThreads - 1) / kThreads;
  const int steps = (a.K + 31) / 32;
  const int n0 = (int)blockIdx.y * (NT * 16);
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, q = lane >> 4;

  // piece p of a step: the eight k of one lane's operand of one tile; what lies behind K or N is answered with zeros
  const RowsBuf wb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.W), 0, (int)(((a.N - 1) * a.ldw + a.K) * 4), 0x00020000);
  const int ldw = (int)a.ldw;
  int w_at[kPieces];
#pragma unroll
  for (int i = 0; i < kPieces; ++i) {
    const int p = ((int)threadIdx.x + i * kThreads) % (NT * 64);      // (threads left over do another's work over again)
    const int n = n0 + 16 * (p >> 6) + (p & 15), pq = (p >> 4) & 3;
    w_at[i] = n < a.N ? (n * ldw + 8 * pq) * 4 : (int)0x80000000u;
  }
  auto load_w = [&](int s, int i, float (&v)[8]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const auto x = __builtin_amdgcn_raw_buffer_load_b128(wb, w_at[i] + 128 * s + 16 * h, 0, 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[4 * h + j] = __uint_as_float(x[j]);
    }
  };
  // pair j of its values (behind K lies the row after it)
  auto pair_w = [&](int s, int i, int j, const float (&v)[8], float& lo, float& hi) {
    const int in = a.K - 32 * s - 8 * (((((int)threadIdx.x + i * kThreads) % (NT * 64)) >> 4) & 3) - 2 * j;
    lo = in > 0 ? v[2 * j] : 0.f;
    hi = in > 1 ? v[2 * j + 1] : 0.f;
  };
  // in three parts
  auto split_w = [&](int s, int i, int j, const float (&v)[8], u32x4 (&o)[3]) {
    float lo, hi;
    pair_w(s, i, j, v, lo, hi);
    uint32_t u[3];
    split2(lo, hi, u);
#pragma unroll
    for (int k = 0; k < 3; ++k) o[k][j] = u[k];
  };
  auto place_w = [&](u32x4* __restrict__ at, int i, const u32x4 (&o)[3]) {
    const int p = ((int)threadIdx.x + i * kThreads) % (NT * 64);
#pragma unroll
    for (int k = 0; k < 3; ++k) at[((p >> 6) * 3 + k) * 64 + (p & 63)] = o[k];
  };
  // All of W is looked at, also where only its first step is placed; four steps at a time (one after the other: 11 us at K = 602).
  LeastOperand least_w;
  constexpr int kAhead = 4;
  for (int s0 = 0; s0 < steps; s0 += kAhead) {
    float v[kAhead][kPieces][8];
#pragma unroll
    for (int h = 0; h < kAhead; ++h)
#pragma unroll
      for (int i = 0; i < kPieces; ++i) load_w(s0 + h < steps ? s0 + h : steps - 1, i, v[h][i]);
#pragma unroll
    for (int h = 0; h < kAhead; ++h)
#pragma unroll
      for (int i = 0; i < kPieces; ++i) {
        const int s = s0 + h;
        if (s >= steps) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float lo, hi;
          pair_w(s, i, j, v[h][i], lo, hi);
          least_w.add(lo, hi);
        }
        if (!RES && s > 0) continue;
        u32x4 o[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) split_w(s, i, j, v[h][i], o);
        place_w(split_lds + s * kStep, i, o);
      }
  }
  const bool w_out = __syncthreads_or(least_w.out());

  const int64_t ntiles = (a.M + 16 * kRT - 1) / (16 * kRT);
  const int64_t stride = (int64_t)gridDim.x * kWaves;
  // rows past M are answered with zeros, what a row is asked for past K is cleared
  auto rows_left = [&](int64_t tile) { return (int)(a.M - tile * (16 * kRT) < 16 * kRT ? a.M - tile * (16 * kRT) : 16 * kRT); };
  auto a_buf = [&](int64_t tile) {
    const int left = rows_left(tile);
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.A + tile * (16 * kRT) * a.lda), 0,
                                             left > 0 ? (int)(((left - 1) * (int)a.lda + a.K) * 4) : 0, 0x00020000);
  };
  auto load_a = [&](RowsBuf b, int s, int rt, floatx4 (&x)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(b, ((16 * rt + c) * (int)a.lda + 32 * s + 8 * q + 4 * h) * 4, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) x[h][i] = __uint_as_float(v[i]);
    }
  };
  const int tail = a.K - (32 * (steps - 1) + 8 * q);   // elements of the lane's part of the last step
  // pair j of the values of row tile rt, of which `in` count, times `sign` in the first tile and -`sign` in the second
  auto split_a = [&](const floatx4 (&v)[kRT][2], int rt, int j, int in, float sign, u32x4 (&x)[kRT][3], LeastOperand& least) {
    const float by = rt & 1 ? -sign : sign;
    float lo = v[rt][j >> 1][2 * (j & 1)], hi = v[rt][j >> 1][2 * (j & 1) + 1];
    lo = 2 * j < in ? lo : 0.f;
    hi = 2 * j + 1 < in ? hi : 0.f;
    least.add(lo, hi);
    uint32_t u[3];
    split2(lo * by, hi * by, u);
#pragma unroll
    for (int k = 0; k < 3; ++k) x[rt][k][j] = u[k];
  };

  // Every wavefront of the workgroup makes the same number of passes (they meet at the steps of W).  While a step is multiplied, the next
  // one is split and the one after it asked for.
  // Rows go to the workgroups 128 at a time, as in the other streaming kernels: what one of them wrote last is read from the L2 of the same
  // compute units.
  constexpr int kGroup = 128 / (16 * kRT);             // tiles of 128 rows
  int64_t tile = gridDim.x % 8 == 0 ? (int64_t)(blockIdx.x / 8) * (8 * kWaves) + (w / kGroup) * (8 * kGroup) + (blockIdx.x % 8) * kGroup + w % kGroup
                                    : (int64_t)blockIdx.x * kWaves + w;
  const int64_t passes = (ntiles + stride - 1) / stride;
  // The sign of a row in its first step: of an even number of bits of the row below 64.  The lane's tiles are all odd or all even (stride is a multiple of eight).
  const float sign0 = (__popc(c) + (int)(tile & 1)) & 1 ? -1.f : 1.f;
  int64_t tile_l = tile;                               // of the step asked for last
  int step_l = 0;
  auto advance = [&] { if (++step_l == steps) { step_l = 0; tile_l += stride; } };
  floatx4 raw[kRT][2];
  u32x4 x[kRT][3];
  LeastOperand first;                                  // of the first step of a pass
#pragma unroll
  for (int rt = 0; rt < kRT; ++rt) load_a(a_buf(tile), 0, rt, raw[rt]);
#pragma unroll
  for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
    for (int j = 0; j < 4; ++j) split_a(raw, rt, j, steps == 1 ? tail : 8, sign0, x, first);
  advance();
#pragma unroll
  for (int rt = 0; rt < kRT; ++rt) load_a(a_buf(tile_l), step_l, rt, raw[rt]);
  int cur = 0;
  bool first_out = __any(first.out());
  for (int64_t pass = 0; pass < passes; ++pass, tile += stride) {
    floatx4 acc[kRT][NT];
#pragma unroll
    for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[rt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    bool again = w_out || first_out;
    float sign = sign0;
    for (int s = 0; s < steps; ++s) {
      const int sn = s + 1 == steps ? 0 : s + 1;
      const float sign_n = sn == 0 ? sign0 : -sign;
      const int in = sn == steps - 1 ? tail : 8;
      advance();
      const RowsBuf nb = a_buf(tile_l);
      float wv[8];
      if constexpr (!RES) load_w(sn, 0, wv);
      u32x4 xn[kRT][3], wo[3];
      LeastOperand least;
      const u32x4* __restrict__ wl = split_lds + (RES ? s : cur) * kStep + lane;
      constexpr int TB = NT > 8 ? 1 : 2;
      constexpr int kGroups = NT / TB;
      // units of work beside the products: pairs of A (each row tile's next part is asked for behind its last pair), then of W
      constexpr int kUnitsA = kRT * 4, kUnits = kUnitsA + (RES ? 0 : kPieces * 4);
      u32x4 wn[TB][3];
#pragma unroll
      for (int t = 0; t < TB; ++t)
#pragma unroll
        for (int k = 0; k < 3; ++k) wn[t][k] = wl[(t * 3 + k) * 64];
#pragma unroll
      for (int g = 0; g < kGroups; ++g) {
        u32x4 wf[TB][3];
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int k = 0; k < 3; ++k) wf[t][k] = wn[t][k];
        if (g + 1 < kGroups) {
#pragma unroll
          for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int k = 0; k < 3; ++k) wn[t][k] = wl[(((g + 1) * TB + t) * 3 + k) * 64];
        }
        __builtin_amdgcn_sched_barrier(0);
        floatx4 low[kRT][TB], high[kRT][TB];
#pragma unroll
        for (int m = 0; m < 6; ++m)
#pragma unroll
          for (int t = 0; t < TB; ++t)
#pragma unroll
            for (int rt = 0; rt < kRT; ++rt) {
              const floatx4 none{0.f, 0.f, 0.f, 0.f};
              if (m < 5) low[rt][t] = mfma(wf[t][kTerm[m][0]], x[rt][kTerm[m][1]], m ? low[rt][t] : none);
              else high[rt][t] = mfma(wf[t][0], x[rt][0], none);
            }
#pragma unroll
        for (int u = g * kUnits / kGroups; u < (g + 1) * kUnits / kGroups; ++u) {
          if (u < kUnitsA) {
            split_a(raw, u >> 2, u & 3, in, sign_n, xn, least);
            if ((u & 3) == 3) load_a(nb, step_l, u >> 2, raw[u >> 2]);
          } else {
            const int i = (u - kUnitsA) >> 2;
            split_w(sn, i, u & 3, wv, wo);
            if ((u & 3) == 3) {
              place_w(split_lds + (cur ^ 1) * kStep, i, wo);
              if (i + 1 < kPieces) load_w(sn, i + 1, wv);
            }
          }
        }
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int rt = 0; rt < kRT; ++rt) {
            const floatx4 sum = high[rt][t] + low[rt][t];
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rt][g * TB + t][r] = __builtin_fmaf(sum[r], rt & 1 ? -sign : sign, acc[rt][g * TB + t][r]);
            asm volatile("" : "+v"(acc[rt][g * TB + t]));      // (here, not behind the loop)
          }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
        for (int k = 0; k < 3; ++k) x[rt][k] = xn[rt][k];
      sign = sign_n;
      const bool out = __any(least.out());
      if (sn != 0) again = again || out;
      else first_out = out;
      if constexpr (!RES) {
        lds_barrier();
        cur ^= 1;
      }
    }
    const int left = rows_left(tile);
    // An operand or a sum out of the range in which the parts stand for their values: those rows are multiplied again on the fp32 pipe.  602 terms to 128
    // columns on 233 K rows, such an operand in no row 314 us, one of 50 K 376, one of 1000 449, one of 32 660 (1027 with requests of one k), in W 745
    // (1179); 419 on the fp32 pipe.  256 to 256 on 2.45 M rows 2.44 ms, 2.67, 3.41, 5.7 (9.1), 6.5 (11.9); 2.60.
    RangeCheck range;
#pragma unroll
    for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) range.add(acc[rt][t][r]);
    const bool sums_out = __any(range.out());
    if (__builtin_expect((int)again | (int)sums_out, 0)) {       // (one branch: two ways into it cost 50 registers)
      const RowsBuf ab = a_buf(tile);
      int ce = c, qe = q;
      asm volatile("" : "+v"(ce), "+v"(qe));
#pragma unroll
      for (int rt = 0; rt < kRT; ++rt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[rt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
      // sixteen k at a time, four in a row a lane: step i of them takes k = k0 + 4 q + i of both operands
      constexpr int kAtOnce = NT > 8 ? NT / 2 : NT;    // (tiles of W asked for together)
      for (int k0 = 0; k0 < a.K; k0 += 16) {
        const int k = k0 + 4 * qe, in = a.K - k;
        float xs[kRT][4];
#pragma unroll
        for (int rt = 0; rt < kRT; ++rt) {
          const auto v = __builtin_amdgcn_raw_buffer_load_b128(ab, ((16 * rt + ce) * (int)a.lda + k) * 4, 0, 0);
#pragma unroll
          for (int i = 0; i < 4; ++i) xs[rt][i] = i < in ? __uint_as_float(v[i]) : 0.f;
        }
#pragma unroll
        for (int t0 = 0; t0 < NT; t0 += kAtOnce) {
          float ws[kAtOnce][4];
#pragma unroll
          for (int t = 0; t < kAtOnce; ++t) {
            const int n = n0 + 16 * (t0 + t) + ce;
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(wb, (int)(n < a.N ? (uint32_t)(n * ldw + k) * 4u : kNoPlace), 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) ws[t][i] = i < in ? __uint_as_float(v[i]) : 0.f;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < kAtOnce; ++t)
#pragma unroll
              for (int rt = 0; rt < kRT; ++rt)
                acc[rt][t0 + t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ws[t][i], xs[rt][i], acc[rt][t0 + t], 0, 0, 0);
        }
      }
    }
    if (left <= 0) continue;
#pragma unroll
    for (int rt = 0; rt < kRT; ++rt) {
      const int64_t row0 = tile * (16 * kRT) + 16 * rt;
      const int here = left - 16 * rt < 16 ? left - 16 * rt : 16;
      if (here <= 0) continue;
      // (the places of the results are not worth registers over the products)
      int ce = c, qe = q;
      asm volatile("" : "+v"(ce), "+v"(qe) : : "memory");
      const int cend = a.endC ? a.N : (a.N + 3) & ~3;  // where the last row may be written to
      const RowsBuf cb = rows_part<float>(a.C, row0, a.ldc, here, n0, cend);
      floatx4 keep[MASK ? NT : 1];
      const bool free_row = MASK && row0 + ce >= a.mask_rows;
      if constexpr (MASK) {
        const int64_t masked = a.mask_rows - row0;
        const int mrows = masked < here ? (masked > 0 ? (int)masked : 0) : here;
        const RowsBuf mb = rows_part<float>(a.mask, row0, a.ldmask, mrows, n0, a.N);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const auto v = __builtin_amdgcn_raw_buffer_load_b128(mb, (ce * (int)a.ldmask + 16 * t + 4 * qe) * 4, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r) keep[t][r] = __uint_as_float(v[r]);
        }
      }
      auto finish = [&](auto cut) {                    // cut: a row may end inside a group of four, behind which nothing may be written
        constexpr bool CUT = decltype(cut)::value;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int n = 16 * t + 4 * qe;
          u32x4 v;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = __float_as_uint(acc[rt][t][r]);
            if constexpr (MASK) v[r] = keep[t][r] > 0.f || free_row ? v[r] : 0u;
          }
          const int left_n = a.N - n0 - n;
          const uint32_t off = (uint32_t)(ce * (int)a.ldc + n) * 4u;
          __builtin_amdgcn_raw_buffer_store_b128(v, cb, (int)(left_n > (CUT ? 3 : 0) ? off : kNoPlace), 0, 0);
          if constexpr (CUT)
#pragma unroll
            for (int r = 0; r < 3; ++r)
              __builtin_amdgcn_raw_buffer_store_b32(v[r], cb, (int)(left_n < 4 && r < left_n ? off + 4u * r : kNoPlace), 0, 0);
        }
      };
      if (a.endC) finish(std::true_type());
      else finish(std::false_type());
    }
  }
}

// ---- dW = A^T B ---------------------------------------------------------------------------------------------
// Partial products of C[M x N] = A[Kd x M]^T B[Kd x N] (Sec. 3.2: the weight gradient, a sum over all rows of the block).  A workgroup
// owns MB x NB elements of C for one range of rows.  16 G rows of both operands at a time are asked for, split into their three parts
// once for the whole workgroup and placed in LDS as operands of v_mfma_f32_32x32x16_bf16 (lane (c, h) = (lane % 32, lane / 32): column c,
// rows 8 h .. 8 h + 7), in the other half of a double buffer, while the WA x WB wavefronts of each of the G groups multiply the
// 16 rows that are theirs, TA x TB tiles of 32 x 32 each.
//
// A thread asks for two neighbouring columns of eight rows: component i is for tile i of a pair, so tile 2 P + i holds the columns
// {64 P + 2 c + i}, and both the requests and the places in LDS of neighbouring lanes are neighbours.
struct SplitTnArgs {
  const float* A; int64_t lda; const float* B; int64_t ldb;
  int64_t Kd; int M; int N; int64_t rows_per_split; int mblocks; int nsplit;
  float* partial;      // [nsplit][M * N]
};
typedef float floatx16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ floatx16 mfma32(const u32x4& x, const u32x4& y, floatx16 acc) {
  bf16x8 a, b;
  __builtin_memcpy(&a, &x, 16); __builtin_memcpy(&b, &y, 16);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}

template <int TA, int TB, int WA, int WB, int G>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_tn_split(SplitTnArgs a) {
  static_assert(WA * WB * G == kWaves && (TA * WA) % 2 == 0 && (TB * WB) % 2 == 0, "eight wavefronts, tiles in pairs");
  constexpr int kTilesA = TA * WA, kTiles = TA * WA + TB * WB;          // of a group
  constexpr int kRows = 16 * G, kBuf = G * kTiles * 3 * 64;              // u32x4 of a buffer
  constexpr int kUnitsAll = kTiles / 2 * 64 * G;                         // (pair of tiles, lane of an operand, group)
  constexpr int kUnits = (kUnitsAll + kThreads - 1) / kThreads;
  constexpr int D = TA * TB <= 4 ? 2 : 1;                                // chunks asked for ahead of the one that is split (registers)
  extern __shared__ u32x4 split_lds[];
  constexpr int kSmall = 256;
  __shared__ int small[kSmall], n_small;                 // chunks with small operands, in order, each up to once a wavefront
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int g = w / (WA * WB), wa = (w / WB) % WA, wb = w % WB;
  const int m0 = (int)blockIdx.y % a.mblocks * (32 * kTilesA), n0 = (int)blockIdx.y / a.mblocks * (32 * (kTiles - kTilesA));

  // this thread's units: its columns in its operand (behind the last one nothing is asked for, or counted), its rows, its place
  bool of_b[kUnits];
  int off[kUnits], put[kUnits];
  uint32_t second[kUnits];
#pragma unroll
  for (int i = 0; i < kUnits; ++i) {
    const int u = ((int)threadIdx.x + i * kThreads) % kUnitsAll;       // (threads left over do another's work over again)
    const int slot = u & 63, pair = (u >> 6) % (kTiles / 2), gr = (u >> 6) / (kTiles / 2);      // (uniform over a wavefront but for slot)
    of_b[i] = 2 * pair >= kTilesA;
    const int col = (of_b[i] ? n0 + 64 * (pair - kTilesA / 2) : m0 + 64 * pair) + 2 * (slot & 31);
    const int width = of_b[i] ? a.N : a.M;
    const int ld = (int)(of_b[i] ? a.ldb : a.lda);
    off[i] = col < width ? ((16 * gr + 8 * (slot >> 5)) * ld + col) * 4 : (int)0x80000000u;
    second[i] = col + 1 < width ? 0xffffffffu : 0u;
    put[i] = (gr * kTiles + 2 * pair) * 3 * 64 + slot;
  }
  typedef float floatx2w __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  floatx2w raw[D][kUnits][8];

  for (int split = (int)blockIdx.x; split < a.nsplit; split += (int)gridDim.x) {
    const int64_t k_lo = (int64_t)split * a.rows_per_split;
    const int64_t k_hi = k_lo + a.rows_per_split < a.Kd ? k_lo + a.rows_per_split : a.Kd;
    auto rows_of = [&](const float* p, int64_t ld, int width, int64_t k) {
      const int64_t left = k_hi - k < kRows ? k_hi - k : kRows;
      return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p + k * ld), 0, left > 0 ? (int)(((left - 1) * (int)ld + width) * 4) : 0, 0x00020000);
    };
    auto load = [&](int64_t k, int i, floatx2w (&raw)[kUnits][8]) {
      const bool ob = __builtin_amdgcn_readfirstlane((int)of_b[i]);
      const RowsBuf b = ob ? rows_of(a.B, a.ldb, a.N, k) : rows_of(a.A, a.lda, a.M, k);
      const int ld = (int)(ob ? a.ldb : a.lda);
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, off[i] + 4 * r * ld, 0, 0);
        raw[i][r] = floatx2w{__uint_as_float(v[0]), __uint_as_float(v[1] & second[i])};
      }
    };
    // rows 2 j, 2 j + 1 of component e of unit i, those of A times `sign`, in three parts
    LeastOperand least;                                  // of the chunk that is split
    auto note = [&](int64_t k) {
      if (__any(least.out()) && lane == 0) {
        const int at = atomicAdd(&n_small, 1);
        if (at < kSmall) small[at] = (int)((k - k_lo) / kRows);
      }
      least = LeastOperand();
    };
    u32x4 part[3];
    auto convert = [&](const floatx2w (&raw)[kUnits][8], int i, int e, int j, float sign) {
      uint32_t o[3];
      const float by = of_b[i] ? 1.f : sign;
      least.add(raw[i][2 * j][e], raw[i][2 * j + 1][e]);
      split2(raw[i][2 * j][e] * by, raw[i][2 * j + 1][e] * by, o);
#pragma unroll
      for (int k = 0; k < 3; ++k) part[k][j] = o[k];
    };
    auto place = [&](u32x4* __restrict__ buf, int i, int e) {
#pragma unroll
      for (int k = 0; k < 3; ++k) buf[put[i] + (e * 3 + k) * 64] = part[k];
    };

    floatx16 acc[TA][TB];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int i = 0; i < kUnits; ++i) load(k_lo + d * kRows, i, raw[d]);
    if (threadIdx.x == 0) n_small = 0;
    lds_barrier();
#pragma unroll
    for (int i = 0; i < kUnits; ++i) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
#pragma unroll
        for (int j = 0; j < 4; ++j) convert(raw[0], i, e, j, 1.f);
        place(split_lds, i, e);
      }
      load(k_lo + D * kRows, i, raw[0]);
    }
    note(k_lo);                                            // (before the barrier: those of a chunk lie side by side in the list)
    __syncthreads();
    // Chunk k, whose operands are in half P of the buffer, is multiplied; the next one is split and placed in the other half, and the one
    // D + 1 chunks on is asked for.  Every other chunk of A is taken with the other sign: what the pipe cuts off is cut downwards, in every
    // chunk the same way.
    auto step = [&](int64_t k, auto half, float sign) {
      const int P = half;
      const u32x4* __restrict__ la = split_lds + P * kBuf + (g * kTiles + wa * TA) * 3 * 64 + lane;
      const u32x4* __restrict__ lb = split_lds + P * kBuf + (g * kTiles + kTilesA + wb * TB) * 3 * 64 + lane;
      u32x4* __restrict__ other = split_lds + (P ^ 1) * kBuf;
      u32x4 bf[TB][3], an[3];
#pragma unroll
      for (int p = 0; p < 3; ++p) an[p] = la[p * 64];
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int p = 0; p < 3; ++p) bf[j][p] = lb[(j * 3 + p) * 64];
      constexpr int kWork = kUnits * 8;               // pairs of rows to split
#pragma unroll
      for (int i = 0; i < TA; ++i) {
        u32x4 af[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) af[p] = an[p];
        if (i + 1 < TA) {
#pragma unroll
          for (int p = 0; p < 3; ++p) an[p] = la[((i + 1) * 3 + p) * 64];
        }
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          __builtin_amdgcn_sched_barrier(0);
          floatx16 low, high;
#pragma unroll
          for (int r = 0; r < 16; ++r) low[r] = high[r] = 0.f;
#pragma unroll
          for (int m = 0; m < 5; ++m) {
            if (m == 1) high = mfma32(af[0], bf[j][0], high);
            low = mfma32(af[kTerm[m][0]], bf[j][kTerm[m][1]], low);
          }
#pragma unroll
          for (int u = (i * TB + j) * kWork / (TA * TB); u < (i * TB + j + 1) * kWork / (TA * TB); ++u) {
            const int un = u >> 3, e = (u >> 2) & 1;
            convert(raw[D == 1 ? 0 : P ^ 1], un, e, u & 3, -sign);
            if ((u & 3) == 3) place(other, un, e);
            if ((u & 7) == 7) load(k + (D + 1) * kRows, un, raw[D == 1 ? 0 : P ^ 1]);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = __builtin_fmaf(high[r] + low[r], sign, acc[i][j][r]);
          asm volatile("" : "+v"(acc[i][j]));          // (here, not behind the loop)
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      note(k + kRows);
      lds_barrier();
    };
    if constexpr (D == 1) {
      int half = 0;
      float sign = 1.f;
      for (int64_t k = k_lo; k < k_hi; k += kRows, half ^= 1, sign = -sign) step(k, half, sign);
    } else {                                             // (the registers of a chunk are told apart by the code)
      for (int64_t k = k_lo; k < k_hi; k += 2 * kRows) {
        step(k, std::integral_constant<int, 0>(), 1.f);
        if (k + kRows >= k_hi) break;
        step(k + kRows, std::integral_constant<int, 1>(), -1.f);
      }
    }

    // The group's rows of chunk k on the fp32 pipe, eight asked for at a time (all of 2.45 M rows 3.2 ms, with two at a time 5.2): whole, or what the
    // parts of their operands lack.
    auto fp32_rows = [&](int64_t k, auto lacking) {
      const RowsBuf ra = rows_of(a.A, a.lda, a.M, k), rb = rows_of(a.B, a.ldb, a.N, k);
#pragma unroll 1
      for (int k8 = 16 * g; k8 < 16 * g + 16; k8 += 8) {
        float av[4][TA], bv[4][TB];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int row = k8 + 2 * kk + h;
#pragma unroll
          for (int i = 0; i < TA; ++i) {
            const int t = wa * TA + i, m = m0 + 64 * (t >> 1) + 2 * c + (t & 1);
            av[kk][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ra, (int)(m < a.M ? (uint32_t)(row * (int)a.lda + m) * 4u : kNoPlace), 0, 0));
          }
#pragma unroll
          for (int j = 0; j < TB; ++j) {
            const int t = wb * TB + j, n = n0 + 64 * (t >> 1) + 2 * c + (t & 1);
            bv[kk][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (int)(n < a.N ? (uint32_t)(row * (int)a.ldb + n) * 4u : kNoPlace), 0, 0));
          }
        }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
          for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j) {
              if constexpr (decltype(lacking)::value) {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(left_over(av[kk][i]), bv[kk][j], acc[i][j], 0, 0, 0);
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[kk][i], left_over(bv[kk][j]), acc[i][j], 0, 0, 0);
              } else {
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[kk][i], bv[kk][j], acc[i][j], 0, 0, 0);
              }
            }
      }
    };
    // Sums out of range (as above), or many chunks with small operands: the rows of the split once more.  Few such chunks: the products of what the
    // parts of their operands lack are added.  Hidden gradients of networks trained to max |Z| 75 .. 700 hold operands below 2^-108 in 0 to 5 rows of
    // 50 K to 100 K, and the last workgroup holds up the launch.  256 x 256 over 2.45 M rows, such an operand in no row 2.09 ms, one of 50 K 2.10 (its
    // whole range of rows again: 7.3), one of 1000 2.18, one of 32 5.3; 2.44 on the fp32 pipe.
    RangeCheck range;
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) range.add(acc[i][j][r]);
    const bool sums_out = __syncthreads_or(range.out());
    const int noted = __builtin_amdgcn_readfirstlane(n_small);
    if (__builtin_expect((int)sums_out | (int)(noted > 0), 0)) {
      if (sums_out || noted > kSmall) {
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
          for (int j = 0; j < TB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
        for (int64_t k = k_lo; k < k_hi; k += kRows) fp32_rows(k, std::false_type());
      } else {
        int before = -1;
        for (int e = 0; e < noted; ++e) {
          const int at = __builtin_amdgcn_readfirstlane(small[e]);
          if (at != before) fp32_rows(k_lo + (int64_t)at * kRows, std::true_type());
          before = at;
        }
      }
      __syncthreads();                                   // (the list may be begun anew)
    }
    // the groups' sums
    if constexpr (G > 1) {
      float* red = reinterpret_cast<float*>(split_lds);
      constexpr int kOne = TA * TB * 16 * 64;
#pragma unroll
      for (int from = 1; from < G; ++from) {
        if (g == from) {
#pragma unroll
          for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r) red[(wa * WB + wb) * kOne + ((i * TB + j) * 16 + r) * 64 + lane] = acc[i][j][r];
        }
        __syncthreads();
        if (g == 0) {
#pragma unroll
          for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int j = 0; j < TB; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r) acc[i][j][r] += red[(wa * WB + wb) * kOne + ((i * TB + j) * 16 + r) * 64 + lane];
        }
        __syncthreads();
      }
    }
    if (g == 0) {
      // register r of lane (c, h) holds row 8 (r / 4) + 4 h + r % 4 of A's tile, column c of B's
      int ce = c, he = h;
      asm volatile("" : "+v"(ce), "+v"(he));
      float* __restrict__ P = a.partial + (int64_t)split * a.M * a.N;
#pragma unroll
      for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int j = 0; j < TB; ++j) {
          const int ta = wa * TA + i, tb = wb * TB + j;
          const int n = n0 + 64 * (tb >> 1) + 2 * ce + (tb & 1);
          if (n >= a.N) continue;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int m = m0 + 64 * (ta >> 1) + 2 * (8 * (r / 4) + 4 * he + (r % 4)) + (ta & 1);
            if (m < a.M) P[(int64_t)m * a.N + n] = acc[i][j][r];
          }
        }
    }
  }
}

constexpr size_t kSplitLds = 160 * 1024;

template <int NT>
int split_launch(const SplitArgs& a, hipStream_t s) {
  constexpr int64_t lim = 256;                         // (a workgroup has a compute unit to itself)
  const size_t step = (size_t)NT * 3 * 1024;
  const int steps = (a.K + 31) / 32;
  const bool res = steps * step <= kSplitLds;
  const size_t lds = (res ? steps : 2) * step;
  const int64_t wgs = ceil_div(a.M, 16 * kRT * kWaves);
  const int panels = (int)ceil_div(a.N, NT * 16);
  const unsigned blocks = (unsigned)std::min<int64_t>(wgs, std::max<int64_t>(1, lim / panels));
  auto go = [&](auto kern) -> int {
    GCN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    kern<<<dim3(blocks, (unsigned)panels), dim3(kThreads), lds, s>>>(a);
    GCN_CHECK_LAUNCH();
    return GCN_OK;
  };
  if (res) return a.mask ? go(k_gemm_nn_split<NT, true, true>) : go(k_gemm_nn_split<NT, true, false>);
  return a.mask ? go(k_gemm_nn_split<NT, false, true>) : go(k_gemm_nn_split<NT, false, false>);
}

// tiles per wavefront, wavefronts, groups; blocks of MB x NB elements of C
struct TnShape { int ta, tb, wa, wb, g; int mb() const { return 32 * ta * wa; } int nb() const { return 32 * tb * wb; } };
constexpr TnShape kTnShapes[] = {{2, 2, 2, 2, 2}, {2, 2, 4, 2, 1}, {2, 2, 2, 4, 1}, {4, 2, 2, 4, 1}, {3, 2, 4, 2, 1}};

// the shape that reads least, then the one that multiplies least
TnShape tn_shape(int M, int N) {
  TnShape best = kTnShapes[0];
  int64_t least = INT64_MAX;
  for (const TnShape& t : kTnShapes) {
    const int64_t bm = ceil_div(M, t.mb()), bn = ceil_div(N, t.nb());
    const int64_t cost = (bm * N + bn * M) * 4 + bm * t.mb() * bn * t.nb() / 64;
    if (cost < least) { least = cost; best = t; }
  }
  return best;
}

int tn_blocks(int M, int N) { const TnShape t = tn_shape(M, N); return (int)(ceil_div(M, t.mb()) * ceil_div(N, t.nb())); }

int tn_splits(int64_t Kd, int M, int N) {
  const int64_t want = 256 / tn_blocks(M, N), most = ceil_div(Kd, 128);
  return (int)std::max<int64_t>(1, std::min(want, most));
}

}  // namespace

// Where the fp32 kernels take longer.  Measured, their time over this kernel's for W^T without / with a mask, on 4 K to 512 K rows of K elements to N
// columns:
//   W in registers (N = 192, 256; gemm_nn_limits_blocks)   128 -> 192 on 32 K rows 0.98 / 1.00, from 64 K 1.5-1.7 / 1.4-1.6; 256 -> 256 on 32 K
//                   0.75 / 0.73, from 64 K 1.16-1.23 / 1.09-1.13; 128 -> 256 from 64 K 1.09-1.16 / 1.02-1.05, 100 -> 256 1.06 / 1.01, 104 -> 256
//                   0.95-0.99 / 0.92-0.97: from 2^16 rows on, to 256 columns from K = 128 on;
//   W in LDS, whole k steps (K <= 128 or a multiple of it)  N <= 64 0.5-1.0, N = 72 .. 128 0.9-1.4, but nothing is gained in a training step
//                   (the pipe's clock: 2^18 x 128 x 128 83 -> 69 us, what follows 14 us longer); N = 129 .. 192 on 32 K 0.9-1.0 / 0.8-1.0, from 64 K
//                   1.1-1.4 / 0.95-1.3 (the least at K = 48); N = 193 .. 256 on 64 K 1.02-1.16 / 0.88-1.04, on 512 K 1.01-1.11 / 0.96-1.06 up to
//                   K = 96, beyond (W's parts do not fit LDS) 0.9 / 0.8: from 2^16 rows on, no masks with many columns or few terms;
//   others (K = 160, 237, 300, 602, or W too large for LDS) N <= 48 on up to 32 K 0.7-1.0 / 0.7-1.0, from 64 K 1.15-1.7 / 1.12-1.7;
//                   N = 64 .. 128 with W in LDS on up to 64 rows 0.80-0.95, from 128 1.05-1.17, but N = 50, 64 and rows of whole quads up to 3 K 0.94-1.0;
//                   else on any number 1.0-2.3 / 1.05-2.5; N = 129 .. 192 on 4 K 0.84-1.02 / 1.2-1.3, from 8 K 0.97-2.3 / 1.2-2.8;
//                   N = 193 .. 400 on 4 K 0.66-0.75 / 0.86-0.94, on 32 K 1.04-1.5 / 1.3-1.6, from 64 K 1.3-1.8 / 1.6-2.0.
// Its error against 64 bits is a third of theirs: 128 columns of K = 128 / 602 terms of either sign 5.7e-8 / 9.6e-8 (2.0e-7 / 4.4e-7), positive
// ones 4.2e-8 / 6.9e-8 (1.2e-7 / 2.6e-7).
bool gemm_nn_split_ok(const void* A, int64_t lda, int64_t ldw, int64_t ldc, int64_t M, int N, int K, int dtype, const GemmEpilogue& epi) {
  const Tuning& t = tune();
  if (t.gemm_split == 0 || dtype != GCN_F32 || !epi.b_trans || epi.bias || epi.relu || epi.C2) return false;
  // (tiles of rows, and W, are buffers with 32-bit offsets)
  if (lda >= 1 << 23 || ldc >= 1 << 23 || epi.ldmask >= 1 << 23 || K >= 1 << 23 || ldw >= 1 << 23) return false;
  if ((double)N * (double)ldw * 4 >= 1 << 30) return false;
  if (t.gemm_split == 2) return true;
  if (t.gemm_fast != 1 || t.gemm_regw != 1) return false;      // (an override is a choice between the fp32 kernels)
  if (gemm_nn_limits_blocks(A, lda, M, N, K, dtype)) return M >= 1 << 16 && (N <= 192 || K >= 128);
  if (gemm_nn_direct_ok(N, K) && (K <= 128 || K % 128 == 0))
    return M >= 1 << 16 && N > 128 && (N <= 192 ? K >= (epi.mask ? 60 : 48) : !epi.mask && K >= 48 && K <= 96);
  if (N <= 48) return M >= 1 << 16;
  if (gemm_nn_direct_ok(N, K) && M < (N <= 64 && K % 4 == 0 ? 1 << 13 : 65)) return false;
  return N <= 128 || (N <= 192 ? M >= 1 << 13 : M * ceil_div(N, 256) >= 1 << 15);
}

int gemm_nn_split(const void* A, int64_t lda, const float* W, int64_t ldw, void* C, int64_t ldc, int64_t M, int N, int K,
                  const GemmEpilogue& epi, hipStream_t s) {
  SplitArgs a{(const float*)A, lda, W, ldw, (float*)C, ldc, M, N, K, (const float*)epi.mask, epi.ldmask, epi.mask_rows,
              N % 4 != 0 && (!epi.c_rows_padded || ((uintptr_t)C % 16) != 0 || ldc % 4 != 0)};
  if (N <= 64) return split_launch<4>(a, s);
  if (N <= 128) return split_launch<8>(a, s);
  if (N <= 192) return split_launch<12>(a, s);
  return split_launch<16>(a, s);
}

// More than 64 columns on both sides (300 K rows x 128 x 64 78 / 89 us, x 602 x 16 243 / 323: there the product waits for memory, and 32 rows in flight
// are too few); a workgroup's block is 128 x 128 at least.  fp32 kernels / this one with the final sum, us, by the kernel that it takes the place of:
//   operands through LDS  both sides above 128, or one above 128 and up to 256: 2 K rows x 256 x 256 47 / 39, x 80 x 200 25.7 / 22.6, 20 K x 256 x 80 35 / 32,
//                         100 K x 300 x 256 245 / 164, 2.45 M x 256 x 256 2440 / 2110, x 100 x 256 1306 / 1299: from 2 K rows on;
//                         else 20 K x 72 x 72 19.6 / 20.0, 64 K 29.8 / 27.8, 300 K 105 / 88; 64 K x 128 x 128 36.0 / 36.4, 300 K 117 / 106; 16 K x 384 x 128 38.5 / 41.8,
//                         32 K 58.5 / 57.3, 64 K 95 / 80;
//   vector requests       2 K x 128 x 66 37 / 17, 8 K x 300 x 66 54 / 33, 300 K x 100 x 66 120 / 91: from 2 K rows on;
//   single requests       (rows of A of no whole quads, of B of no whole pairs) 20 K x 65 x 65 17.4 / 20.3, 64 K 30.4 / 27.7, 300 K 141 / 87; 64 K x 173 x 128 51 / 55, 128 K
//                         101 / 86; 16 K x 505 x 100 34 / 40, 32 K 63 / 58; 8 K x 602 x 128 33 / 40, 20 K 62 / 56; 8 K x 602 x 256 48 / 51, 16 K 83 / 72:
//                         there, as with narrow outputs through LDS, from 1.5e9 products or 2^17 rows on.
// Error against 64 bits 4.4e-7 for 1.7e-6 (256 x 256 over 2.45 M rows), 1.2e-7 for 5.8e-7 (128 x 128 over 2^18).
bool gemm_tn_split_ok(const void* A, int64_t lda, const void* B, int64_t ldb, int64_t Kd, int M, int N, int dtype) {
  const Tuning& t = tune();
  if (t.gemm_split == 0 || dtype != GCN_F32 || Kd < 1 || M < 1 || N < 1) return false;
  if (lda >= 1 << 23 || ldb >= 1 << 23) return false;
  if (t.gemm_split == 2) return true;
  if (t.gemm_tn_wide != 1 || t.gemm_tn_lds != 1 || M <= 64 || N <= 64 || Kd < 2048) return false;
  const int less = std::min(M, N), more = std::max(M, N);
  const bool always = gemm_tn_lds_ok(A, lda, B, ldb, Kd, M, N, dtype) ? less > 128 || (more > 128 && more <= 256) : gemm_tn_wide_ok(A, lda, B, ldb, N, dtype);
  return always || Kd >= 1 << 17 || (double)Kd * M * N >= 1.5e9;
}

size_t gemm_tn_split_ws_bytes(int64_t Kd, int M, int N) { return sizeof(float) * (size_t)tn_splits(Kd, M, N) * (size_t)M * (size_t)N; }

int gemm_tn_split_partials(const void* A, int64_t lda, const void* B, int64_t ldb, int64_t Kd, int M, int N, float* partial, int* nsplit_out,
                           hipStream_t s, int max_blocks) {
  const TnShape t = tn_shape(M, N);
  const int per_split = tn_blocks(M, N);
  const int64_t rps = round_up(ceil_div(Kd, tn_splits(Kd, M, N)), 32);
  const int nsplit = (int)ceil_div(Kd, rps);            // every split holds at least one row
  *nsplit_out = nsplit;
  SplitTnArgs a{(const float*)A, lda, (const float*)B, ldb, Kd, M, N, rps, (int)ceil_div(M, t.mb()), nsplit, partial};
  const int at_once = max_blocks > 0 ? std::min(nsplit, std::max(1, max_blocks / per_split)) : nsplit;
  const size_t lds = (size_t)2 * t.g * (t.ta * t.wa + t.tb * t.wb) * 3 * 1024;
#define GCN_TNS(TA, TB, WA, WB, G)                                                                              \
  if (t.ta == TA && t.tb == TB && t.wa == WA && t.wb == WB && t.g == G) {                                         \
    auto kern = k_gemm_tn_split<TA, TB, WA, WB, G>;                                                              \
    GCN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds)); \
    kern<<<dim3((unsigned)at_once, (unsigned)per_split), kThreads, lds, s>>>(a);                                 \
  }
  GCN_TNS(2, 2, 2, 2, 2) GCN_TNS(2, 2, 4, 2, 1) GCN_TNS(2, 2, 2, 4, 1) GCN_TNS(4, 2, 2, 4, 1) GCN_TNS(3, 2, 4, 2, 1)
#undef GCN_TNS
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

}  // namespace gcn
