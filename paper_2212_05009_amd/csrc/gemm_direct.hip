// Streaming forms of the two tall-and-skinny dense products of a GCN layer (Sec. 3.1: the product
// with W^k after the sparse aggregation, and the weight gradient), for gfx950.  The long operand
// (one row per vertex) goes from global memory straight into the MFMA operand registers: no LDS
// staging and no barrier in the main loop, so a wavefront keeps many independent loads in flight,
// which is what a product bound by HBM bandwidth needs.
//
//   nn_direct : C[M x N] = A[M x K] W[K x N], W small enough to sit in LDS for the whole kernel.
//               MFMA 16x16x4: lane (c = l%16, q = l/16) loads A[row c][k0 + 4q .. k0 + 4q + 3] with one
//               16-byte load and feeds element i of it to the i-th of four MFMAs, whose W operand is
//               W[k0 + 4q + i][col c]: every k of the 16-wide step is used exactly once, only in a
//               permuted order, which a sum does not care about.
//   tn_direct : C[M x N] = A[Kd x M]^T B[Kd x N], Kd = number of vertices.  MFMA 32x32x2: lane
//               (c = l%32, h = l/32) loads A[k + h][m0 + c] and B[k + h][n0 + c]: 128-byte coalesced
//               rows.  The four wavefronts of a block take interleaved row chunks of one output tile,
//               add their tiles through LDS and write one partial tile per block.
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "rows_buf.h"

namespace gcn {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// 4 consecutive elements starting at column k (multiple of 4) of a row, zero beyond `limit`
template <typename T>
__device__ __forceinline__ void load_quad(const T* __restrict__ row, int k, int limit, bool vec_ok, float (&o)[4]) {
  if (vec_ok && k + 3 < limit) {
    if constexpr (sizeof(T) == 4) {
      float4 v = *reinterpret_cast<const float4*>(row + k);
      o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
    } else {
      uint2 v = *reinterpret_cast<const uint2*>(row + k);
      o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xffff0000u);
      o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xffff0000u);
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (k + i < limit) ? load_one<T>(row + k + i) : 0.f;
}

// 4 consecutive elements starting at column n (multiple of 4) of a row, none beyond `limit`
template <typename T>
__device__ __forceinline__ void store_quad(T* __restrict__ row, int n, int limit, bool vec_ok, const float (&v)[4]) {
  if (vec_ok && n + 3 < limit) {
    if constexpr (sizeof(T) == 4) {
      *reinterpret_cast<float4*>(row + n) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
      bf16_t h[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) store_one<T>(&h[i], v[i]);
      uint2 pk;
      pk.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
      pk.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
      *reinterpret_cast<uint2*>(row + n) = pk;
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (n + i < limit) store_one<T>(row + n + i, v[i]);
}

// ------------------------------------------------------------------------------------------
struct NnDirectArgs {
  const void* A; int64_t lda; const float* W; int64_t ldw; void* C; int64_t ldc;
  int64_t M; int N; int K; int vecA; int vecC; int vecC2; int vecM;
  const float* bias; int relu; const void* mask; int64_t ldmask; int64_t mask_rows; void* C2; int64_t ldc2;
  int trans;               // W is stored [N x K]
  // k_gemm_nn_fast: a row of A / of the outputs ends with its last element, nothing beyond may be touched
  int endA = 0, endC = 0;
};

typedef float floatx4w __attribute__((ext_vector_type(4), aligned(4)));

// put(k, n, W[k][n]) for every element of the LDS copy of W (Kp x NP elements, Kp a multiple of 16, zero beyond K and N).
// W stored [N x K]: a lane takes four k of a row with one request, four lanes 64 bytes of it and the next four the row
// after, whose places in LDS are other banks (lanes along one row alone meet on few banks, in the layout of whole quads on
// one: 128 x 128, 4 K rows 22 us that way, 16 us this way).
// The requests do not depend on the places behind them: a lane asks for several elements before it writes the first.  Places past
// the edge are asked for at the edge (and written again, with the same value) or cleared at the end.  Measured, one tile of
// rows with everything around it, us one element at a time / this way: 128 x 128 12.2 / 10.6,
// 256 x 47 12.7 / 10.7, 50 x 50 6.8 / 6.2 (16 x 16, which is one element a thread, 6.1).
template <int NP, typename F>
__device__ __forceinline__ void walk_w(const float* __restrict__ W, int64_t ldw, int trans, int K, int N, int Kp, int threads, F put) {
  if (__builtin_expect(trans, 0) && K >= 4) {
    constexpr int kBatch = 4;
    const int total = Kp / 4 * NP;
    for (int e0 = threadIdx.x; e0 < total; e0 += kBatch * threads) {
      floatx4w v[kBatch];
      int kk[kBatch], nn[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int e = e0 + u * threads < total ? e0 + u * threads : e0;
        const int n = (e >> 2) % NP, k = 4 * ((e & 3) + 4 * ((e >> 2) / NP));
        kk[u] = k < K - 4 ? k : K - 4;
        nn[u] = n < N ? n : N - 1;
        v[u] = *reinterpret_cast<const floatx4w*>(W + (int64_t)nn[u] * ldw + kk[u]);
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) put(kk[u] + i, nn[u], v[u][i]);
    }
    for (int e = threadIdx.x; e < (Kp - K) * NP; e += threads) put(K + e / NP, e % NP, 0.f);
    for (int e = threadIdx.x; e < K * (NP - N); e += threads) put(e / (NP - N), N + e % (NP - N), 0.f);
  } else {
    constexpr int kBatch = 8;
    const int total = Kp * NP;
    const int64_t sk = trans ? 1 : ldw, sn = trans ? ldw : 1;
    for (int e0 = threadIdx.x; e0 < total; e0 += kBatch * threads) {
      float v[kBatch];
      int at[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        at[u] = e0 + u * threads < total ? e0 + u * threads : e0;
        const int k = at[u] / NP, n = at[u] % NP;
        const float x = W[(k < K ? k : K - 1) * sk + (n < N ? n : N - 1) * sn];
        v[u] = __uint_as_float(__float_as_uint(x) & (k < K && n < N ? 0xffffffffu : 0u));
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) put(at[u] / NP, at[u] % NP, v[u]);
    }
  }
}

constexpr int kNnThreads = 512;
constexpr int kNnKU = 8;          // 16-wide k steps whose loads are issued together

// At most 128 registers for up to 8 column tiles, so that two 8-wave blocks share a compute unit
// (four wavefronts per SIMD): measured 161 -> 137 us for 2^18 x 128 x 128.
template <typename T, int NT>
__global__ __launch_bounds__(kNnThreads) __attribute__((amdgpu_waves_per_eu(NT <= 8 ? 4 : 2, 8))) void k_gemm_nn_direct(NnDirectArgs a) {
  extern __shared__ float Ws[];                      // [Kp][LDW], zero beyond K and N
  constexpr int LDW = NT * 16 + 4;                    // 4 k-rows apart land 16 banks apart
  const int Kp = (a.K + 15) & ~15;
  walk_w<NT * 16>(a.W, a.ldw, a.trans, a.K, a.N, Kp, kNnThreads, [&](int k, int n, float v) { Ws[k * LDW + n] = v; });
  __syncthreads();

  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = lane & 15, q = lane >> 4;
  const T* __restrict__ A = reinterpret_cast<const T*>(a.A);
  T* __restrict__ C = reinterpret_cast<T*>(a.C);
  T* __restrict__ C2 = reinterpret_cast<T*>(a.C2);
  const T* __restrict__ Mk = reinterpret_cast<const T*>(a.mask);
  const bool vec_ok = a.vecA == 4;
  const int64_t ntiles = (a.M + 15) / 16;
  constexpr int WPB = kNnThreads / 64;

  // Software pipeline over the tiles of this wavefront: the operand rows (first 128 k) and the mask
  // values of the NEXT tile are requested before the current tile's MFMAs and stores, so that a
  // wavefront always has a tile's worth of loads in flight.
  constexpr int TC = NT < 8 ? NT : 8;                 // column tiles finished together (bounds registers)
  constexpr bool kPrefetchMask = NT <= 4;
  const int64_t stride = (int64_t)gridDim.x * WPB;
  auto load_a = [&](int64_t tile, int k0, float (&av)[kNnKU][4]) {
    const int64_t row = tile * 16 + c;
    const T* __restrict__ arow = A + (row < a.M ? row : a.M - 1) * a.lda;
#pragma unroll
    for (int u = 0; u < kNnKU; ++u) {
      if (k0 + 16 * u < Kp) load_quad<T>(arow, k0 + 16 * u + 4 * q, a.K, vec_ok, av[u]);
      else { av[u][0] = av[u][1] = av[u][2] = av[u][3] = 0.f; }
    }
  };
  auto load_m = [&](int64_t tile, int t0, float (&keep)[TC][4]) {
    const int64_t m = tile * 16 + c;
    const bool masked = Mk != nullptr && m < a.mask_rows && m < a.M;
#pragma unroll
    for (int t = 0; t < TC; ++t) {
      keep[t][0] = keep[t][1] = keep[t][2] = keep[t][3] = 1.f;
      if (masked && t0 + t < NT) load_quad<T>(Mk + m * a.ldmask, (t0 + t) * 16 + 4 * q, a.N, a.vecM == 4, keep[t]);
    }
  };

  int64_t tile = (int64_t)blockIdx.x * WPB + w;
  float a_nxt[kNnKU][4], m_nxt[TC][4];
  if (tile < ntiles) {
    load_a(tile, 0, a_nxt);
    if (kPrefetchMask) load_m(tile, 0, m_nxt);
  }
  for (; tile < ntiles; tile += stride) {
    float av[kNnKU][4], keep[TC][4];
#pragma unroll
    for (int u = 0; u < kNnKU; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) av[u][i] = a_nxt[u][i];
    if (kPrefetchMask) {
#pragma unroll
      for (int t = 0; t < TC; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) keep[t][i] = m_nxt[t][i];
    }
    if (tile + stride < ntiles) {
      load_a(tile + stride, 0, a_nxt);
      if (kPrefetchMask) load_m(tile + stride, 0, m_nxt);
    }

    floatx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < Kp; k0 += 16 * kNnKU) {
      if (k0 > 0) load_a(tile, k0, av);
#pragma unroll
      for (int u = 0; u < kNnKU; ++u) {
        if (k0 + 16 * u < Kp) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float* wrow = Ws + (k0 + 16 * u + 4 * q + i) * LDW + c;
#pragma unroll
            for (int t = 0; t < NT; ++t)
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wrow[t * 16], av[u][i], acc[t], 0, 0, 0);
          }
        }
      }
    }

    // W is the first MFMA operand, so the 16 x 16 result tile is transposed: register r of lane (c, q)
    // holds output column 16t + 4q + r of row c.  A lane owns 4 consecutive columns of its row:
    // one 16-byte store (and one 16-byte mask load) per column tile.
    const int64_t m = tile * 16 + c;
    if (m < a.M) {
      const bool masked = Mk != nullptr && m < a.mask_rows;
#pragma unroll
      for (int t0 = 0; t0 < NT; t0 += TC) {
        if (!kPrefetchMask) load_m(tile, t0, keep);
#pragma unroll
        for (int t = 0; t < TC; ++t) {
          if (t0 + t >= NT) continue;
          const int n = (t0 + t) * 16 + 4 * q;
          if (n >= a.N) continue;
          float v[4], pre[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            pre[r] = acc[t0 + t][r] + ((a.bias && n + r < a.N) ? a.bias[n + r] : 0.f);
            v[r] = a.relu ? (pre[r] > 0.f ? pre[r] : 0.f) : pre[r];
            if (masked) v[r] = keep[t][r] > 0.f ? v[r] : 0.f;
          }
          if (C2) store_quad<T>(C2 + m * a.ldc2, n, a.N, a.vecC2 == 4, pre);
          store_quad<T>(C + m * a.ldc, n, a.N, a.vecC == 4, v);
        }
      }
    }
  }
}

// ---- the same product without a single data-dependent branch ----------------------------------------
// For operands whose rows start on a 4-byte word, K up to 128 (KU = ceil(K / 16) k steps, the
// whole row in one request batch, a tail of the row cleared by bit masks) or a multiple of 128 (KU = 8), N up to 256 and a
// mask that covers every row.  Rows on 16 bytes (bf16: 8) may be read up to the next multiple of 4 elements, and written
// that far where their owner allows it (GemmEpilogue::c_rows_padded); in other rows the request that would pass the end is
// moved back to end with the row and its elements are shifted into place, and the last columns of the result are stored
// one by one.  Measured, 500 K x 50 x 50 in contiguous rows (200
// bytes): general kernel 128 us, this one 69 us.  Every load is an
// unconditional 16-byte (bf16: 8-byte) request - rows beyond M are clamped to the last row and dropped at
// the store - so the compiler can keep the next step's operand loads in flight across the MFMAs of the
// current one instead of waiting at every join of the general kernel's bounds checks.
// (the global memory path takes 8- and 16-byte requests at any word address)
template <typename T> __device__ __forceinline__ void vload4(const T* __restrict__ p, float (&o)[4]) {
  if constexpr (sizeof(T) == 4) {
    const floatx4w v = *reinterpret_cast<const floatx4w*>(p);
    o[0] = v[0]; o[1] = v[1]; o[2] = v[2]; o[3] = v[3];
  } else {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2), aligned(4)));
    const u32x2 v = *reinterpret_cast<const u32x2*>(p);
    o[0] = __uint_as_float(v[0] << 16); o[1] = __uint_as_float(v[0] & 0xffff0000u);
    o[2] = __uint_as_float(v[1] << 16); o[3] = __uint_as_float(v[1] & 0xffff0000u);
  }
}
template <typename T> __device__ __forceinline__ void buf_load4(RowsBuf b, uint32_t off, float (&o)[4]) {
  if constexpr (sizeof(T) == 4) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b128(b, (int)off, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(q[i]);
  } else {
    const auto q = __builtin_amdgcn_raw_buffer_load_b64(b, (int)off, 0, 0);
    o[0] = __uint_as_float(q[0] << 16); o[1] = __uint_as_float(q[0] & 0xffff0000u);
    o[2] = __uint_as_float(q[1] << 16); o[3] = __uint_as_float(q[1] & 0xffff0000u);
  }
}
template <typename T> __device__ __forceinline__ void buf_store4(RowsBuf b, uint32_t off, const float (&v)[4]) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  if constexpr (sizeof(T) == 4) {
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])}, b,
                                           (int)off, 0, 0);
  } else {
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{(uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16),
                                                (uint32_t)f32_to_bf16(v[2]) | ((uint32_t)f32_to_bf16(v[3]) << 16)}, b, (int)off, 0, 0);
  }
}
template <typename T> __device__ __forceinline__ void buf_store1(RowsBuf b, uint32_t off, float v) {
  if constexpr (sizeof(T) == 4) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), b, (int)off, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(v), b, (int)off, 0, 0);
}

// whether the registers of an instance leave room for two blocks a compute unit
constexpr bool nn_two_blocks(int NT, int KU, bool MASK) { return NT <= 8 && !(MASK && NT == 8 && KU > 4); }

// FULL: K is a multiple of 16 and N = 16 NT, so there is no tail to clear and no column group to skip.  CH: k chunks per tile (0: by
// the arguments).
//
// Nothing between the requests of a tile and their use may branch, stores included: loads and stores share one counter of
// requests in flight, and behind a join at which some stores may not have been issued the only safe wait for the next tile's
// operand is a wait for all, stores too - one round trip of the stores per tile, and the matrix pipe idle meanwhile.  So rows past M
// and columns past N are dropped by the stores' range check, the mask of a tile is requested before its first MFMA, and
// the chunks of a tile are unrolled.  (Asked for a tile ahead instead, with this tile's stores behind it, the mask costs up to 20 %:
// 40 K rows 16 -> 128 17.4 us against 14.0, 100 K 47 -> 256 68 / 60, 2.45 M 1107 / 1086.)  Measured on rows of whole lines, us with
// conditional stores and bias loads between them / this way: 300 K rows 50 -> 50 41 / 33, 64 -> 64 36.5 / 31.0, 32 -> 128 42 / 38,
// 47 -> 256 144 / 124, 128 -> 128 114 / 98 (100 TFLOP/s: the matrix pipe); with the mask 50 -> 50 40 / 35, 41 -> 128 95 / 73, 47 -> 256
// 179 / 136, on 2.45 M rows 1389 / 1086; but 64 -> 64 and 50 -> 50 with the mask on 1 M rows and more 107 / 114 and 126 / 136.
template <typename T, int NT, int KU, int CH, bool MASK, bool SAVE, bool FULL>
__global__ __launch_bounds__(kNnThreads) __attribute__((amdgpu_waves_per_eu(nn_two_blocks(NT, KU, MASK) ? 4 : 2, 8))) void k_gemm_nn_fast(NnDirectArgs a) {
  // W in LDS.  NT a multiple of 4: [k][t / 4][c][t % 4], so that the four column tiles 4 tq .. 4 tq + 3 of a
  // lane's (k, c) are one 16-byte read and the 16 lanes of a k row read 256 contiguous bytes.  Else [k][LDW].
  extern __shared__ float Ws[];
  constexpr int LDW = NT * 16 + 4;
  constexpr bool kQuad = NT % 4 == 0;
  constexpr int TQ = kQuad ? NT / 4 : 1;
  const int chunks = CH > 0 ? CH : (a.K + 16 * KU - 1) / (16 * KU);   // k chunks per tile
  walk_w<NT * 16>(a.W, a.ldw, a.trans, a.K, a.N, chunks * 16 * KU, kNnThreads, [&](int k, int n, float v) {
    const int t = n >> 4, cc = n & 15;
    Ws[kQuad ? ((k * TQ + (t >> 2)) * 16 + cc) * 4 + (t & 3) : k * LDW + n] = v;
  });
  float* bias = Ws + chunks * 16 * KU * (kQuad ? NT * 16 : LDW);      // behind W; zeros where there is none
  for (int n = threadIdx.x; n < NT * 16; n += kNnThreads) bias[n] = a.bias && n < a.N ? a.bias[n] : 0.f;
  const uint32_t neg = a.relu ? 0u : 0xffffffffu;                     // what stays of a value that is not positive
  __syncthreads();

  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, q = lane >> 4;
  const T* __restrict__ A = reinterpret_cast<const T*>(a.A);
  constexpr int WPB = kNnThreads / 64;
  const int64_t ntiles = (a.M + 15) / 16;
  const int64_t stride = (int64_t)gridDim.x * WPB;
  // K that is no multiple of 16: the lane's request of the very last k step may start past K (moved to column 0)
  // or reach past it (the row is padded to 4 elements); `tail` clears what is not part of the product
  const int k_last = 16 * KU * chunks - 16 + 4 * q;
  const int n_ok = a.K - k_last;
  // (endA: moved back to column K - 4, `shift` elements too early)
  const int shift = !FULL && a.endA && n_ok > 0 && n_ok < 4 ? 4 - n_ok : 0;
  const int last_off = n_ok > 0 ? k_last - shift : 0;
  uint32_t tail[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) tail[i] = i < n_ok ? 0xffffffffu : 0u;
  const int n_up = FULL ? NT * 16 : (a.N + 3) & ~3;     // columns come in groups of 4; the rows are that long
  // part u of chunk `chunk` of the lane's row of a tile
  auto a_row = [&](int64_t tile) -> const T* {
    const int64_t row = tile * 16 + c;
    return A + (row < a.M ? row : a.M - 1) * a.lda + (FULL ? 4 * q : 0);
  };
  auto load_a = [&](const T* __restrict__ arow, int chunk, int u, float (&x)[4]) {
    if constexpr (FULL) vload4<T>(arow + chunk * (16 * KU) + 16 * u, x);
    else vload4<T>(arow + ((u == KU - 1 && chunk == chunks - 1) ? last_off : chunk * (16 * KU) + 16 * u + 4 * q), x);
  };
  auto rows_left = [&](int64_t tile) { return (int)(a.M - tile * 16 < 16 ? a.M - tile * 16 : 16); };
  // place of column n of the lane's row in a buffer of 16 rows
  auto place = [&](int64_t ld, int n) -> uint32_t {
    const uint32_t off = (uint32_t)(c * (int)ld + n) * (uint32_t)sizeof(T);
    return FULL || n < n_up ? off : kNoPlace;
  };

  int64_t tile = (int64_t)blockIdx.x * WPB + w;
  if (tile >= ntiles) return;
  // Registers hold one operand row part of each kind: as soon as its MFMAs are issued, the same part of the next chunk or tile is
  // asked for.
  float av[KU][4];
  float keep[MASK ? NT : 1][4];
  {
    const T* __restrict__ arow = a_row(tile);
#pragma unroll
    for (int u = 0; u < KU; ++u) load_a(arow, 0, u, av[u]);
    // The loop is entered with as many requests behind the operand's as it is repeated with, so that its waits need not tell
    // the two apart: stores that the range check drops stand for those of a tile before.
    const RowsBuf cb = rows_buf<T>(a.C, tile * 16, a.ldc, rows_left(tile));
    const float none[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if constexpr (SAVE) buf_store4<T>(cb, kNoPlace - 32 * t - 16, none);
      buf_store4<T>(cb, kNoPlace - 32 * t, none);
    }
  }
  for (; tile < ntiles; tile += stride) {
    asm volatile("" ::: "memory");         // (the bias stays in LDS)
    const int64_t after = tile + stride < ntiles ? tile + stride : tile;      // (at the end the same tile again, unused)
    if constexpr (MASK) {
      const RowsBuf mb = rows_buf<T>(a.mask, tile * 16, a.ldmask, rows_left(tile));
#pragma unroll
      for (int t = 0; t < NT; ++t) buf_load4<T>(mb, place(a.ldmask, 16 * t + 4 * q), keep[t]);
      __builtin_amdgcn_sched_barrier(0);
    }
    floatx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto do_chunk = [&](int chunk) {
      const bool same = chunk + 1 < chunks;
      const T* __restrict__ next = a_row(same ? tile : after);
      const int next_chunk = same ? chunk + 1 : 0;
      // kQuad: the W operands of step (u, i + 1) are read from LDS before the MFMAs of step (u, i) are issued
      const floatx4* wq = reinterpret_cast<const floatx4*>(Ws) + ((chunk * (16 * KU) + 4 * q) * TQ) * 16 + c;
      const float* wbase = Ws + (chunk * (16 * KU) + 4 * q) * LDW + c;
      floatx4 wc[TQ], wn[TQ];
      if constexpr (kQuad) {
#pragma unroll
        for (int tq = 0; tq < TQ; ++tq) wc[tq] = wq[tq * 16];
      }
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        float x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = av[u][i];
        if constexpr (!FULL) {
          if (u == KU - 1 && chunk == chunks - 1) {
            if (a.endA) {
              if (shift & 1) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; }
              if (shift & 2) { x[0] = x[2]; x[1] = x[3]; }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = __uint_as_float(__float_as_uint(x[i]) & tail[i]);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (kQuad) {
            const int st = 4 * u + i, kn = 16 * ((st + 1) >> 2) + ((st + 1) & 3);
            if (st + 1 < KU * 4) {
#pragma unroll
              for (int tq = 0; tq < TQ; ++tq) wn[tq] = wq[(kn * TQ + tq) * 16];
            }
#pragma unroll
            for (int tq = 0; tq < TQ; ++tq)
#pragma unroll
              for (int r = 0; r < 4; ++r)
                acc[tq * 4 + r] = __builtin_amdgcn_mfma_f32_16x16x4f32(wc[tq][r], x[i], acc[tq * 4 + r], 0, 0, 0);
#pragma unroll
            for (int tq = 0; tq < TQ; ++tq) wc[tq] = wn[tq];
          } else {
            const float* wrow = wbase + (16 * u + i) * LDW;
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(wrow[t * 16], x[i], acc[t], 0, 0, 0);
          }
          if (NT >= 8 || i == 3) __builtin_amdgcn_sched_barrier(0);      // (else all of W is read ahead, and spilled)
        }
        load_a(next, next_chunk, u, av[u]);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    if constexpr (CH > 0) {
#pragma unroll
      for (int chunk = 0; chunk < CH; ++chunk) do_chunk(chunk);
    } else {
      for (int chunk = 0; chunk < chunks; ++chunk) do_chunk(chunk);
    }
    // register r of lane (c, q) holds output column 16t + 4q + r of row c
    float last[4] = {0.f, 0.f, 0.f, 0.f}, last2[4] = {0.f, 0.f, 0.f, 0.f};      // the quad that column N cuts, and where it starts
    int at = a.N;
    const RowsBuf cb = rows_buf<T>(a.C, tile * 16, a.ldc, rows_left(tile));
    RowsBuf cb2 = cb;
    if constexpr (SAVE) cb2 = rows_buf<T>(a.C2, tile * 16, a.ldc2, rows_left(tile));
    float v[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const floatx4 bv = *reinterpret_cast<const floatx4*>(bias + t * 16 + 4 * q);
      acc[t] += bv;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v[t][r] = acc[t][r] > 0.f ? acc[t][r] : __uint_as_float(__float_as_uint(acc[t][r]) & neg);
        if constexpr (MASK) v[t][r] = keep[t][r] > 0.f ? v[t][r] : 0.f;
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int n = t * 16 + 4 * q;
      float pre[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) pre[r] = acc[t][r];
      const bool part = !FULL && a.endC && n < a.N && n + 4 > a.N;
      const uint32_t off = part ? kNoPlace : place(a.ldc, n), off2 = !SAVE || part ? kNoPlace : place(a.ldc2, n);
      if constexpr (!FULL) {
        if (2 * t + 2 > NT || NT <= 4) {
#pragma unroll
          for (int r = 0; r < 4; ++r) { last[r] = part ? v[t][r] : last[r]; last2[r] = SAVE && part ? pre[r] : last2[r]; }
          at = part ? n : at;
        }
      }
      if constexpr (SAVE) buf_store4<T>(cb2, off2, pre);
      buf_store4<T>(cb, off, v[t]);
    }
    if constexpr (!FULL) {
      if (a.endC) {        // the columns that a row ends in, one after the other
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool in = at + r < a.N;
          if constexpr (SAVE) buf_store1<T>(cb2, in ? (uint32_t)(c * (int)a.ldc2 + at + r) * (uint32_t)sizeof(T) : kNoPlace, last2[r]);
          buf_store1<T>(cb, in ? (uint32_t)(c * (int)a.ldc + at + r) * (uint32_t)sizeof(T) : kNoPlace, last[r]);
        }
      }
    }
  }
}

static int nn_tiles(int N) { return N <= 16 ? 1 : N <= 32 ? 2 : N <= 48 ? 3 : N <= 64 ? 4 : N <= 128 ? 8 : 16; }

size_t gemm_nn_direct_lds_bytes(int N, int K) {
  return sizeof(float) * (size_t)((K + 15) & ~15) * (size_t)(nn_tiles(N) * 16 + 4);
}

bool gemm_nn_direct_ok(int N, int K) { return N <= 256 && gemm_nn_direct_lds_bytes(N, K) <= 128 * 1024; }

template <typename T, int NT>
static int nn_launch(const NnDirectArgs& a, hipStream_t s) {
  const size_t lds = gemm_nn_direct_lds_bytes(a.N, a.K);
  auto kern = k_gemm_nn_direct<T, NT>;
  GCN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  const int64_t ntiles = ceil_div(a.M, 16);
  const int per_cu = lds > 80 * 1024 ? 1 : 2;         // blocks that fit one compute unit's LDS
  int64_t blocks = ceil_div(ntiles, kNnThreads / 64);
  if (blocks > 256 * per_cu) blocks = 256 * per_cu;
  kern<<<dim3((unsigned)blocks), dim3(kNnThreads), lds, s>>>(a);
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

template <typename T, int NT, int KU>
static int nn_launch_fast(const NnDirectArgs& a, hipStream_t s) {
  const size_t lds = gemm_nn_direct_lds_bytes(a.N, a.K) + sizeof(float) * 16 * NT;      // (and the bias)
  const int64_t ntiles = ceil_div(a.M, 16);
  const int per_cu = lds > 80 * 1024 || !nn_two_blocks(NT, KU, a.mask != nullptr) ? 1 : 2;
  int64_t blocks = ceil_div(ntiles, kNnThreads / 64);
  if (blocks > 256 * per_cu) blocks = 256 * per_cu;
  auto go = [&](auto kern) -> int {
    GCN_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    kern<<<dim3((unsigned)blocks), dim3(kNnThreads), lds, s>>>(a);
    GCN_CHECK_LAUNCH();
    return GCN_OK;
  };
  auto pick = [&](auto ch) -> int {
    constexpr int CH = decltype(ch)::value;
    if constexpr (KU == 1 || KU == 2 || KU == 4 || KU == 8) {
      if ((a.K % 16) == 0 && a.N == NT * 16) {
        if (a.mask) return go(k_gemm_nn_fast<T, NT, KU, CH, true, false, true>);
        return a.C2 ? go(k_gemm_nn_fast<T, NT, KU, CH, false, true, true>) : go(k_gemm_nn_fast<T, NT, KU, CH, false, false, true>);
      }
    }
    if (a.mask) return go(k_gemm_nn_fast<T, NT, KU, CH, true, false, false>);
    return a.C2 ? go(k_gemm_nn_fast<T, NT, KU, CH, false, true, false>) : go(k_gemm_nn_fast<T, NT, KU, CH, false, false, false>);
  };
  if constexpr (KU == 8) {
    if (a.K > 256) return pick(std::integral_constant<int, 0>());
    if (a.K > 128) return pick(std::integral_constant<int, 2>());
  }
  return pick(std::integral_constant<int, 1>());
}

// the branch-free kernel serves rows on word boundaries with K up to 128 or a multiple of 128
template <typename T>
static bool nn_fast(NnDirectArgs a, hipStream_t s, int* rc) {
  const bool off = tune().gemm_fast == 0;
  const int NT = nn_tiles(a.N);
  if (off) return false;
  auto words = [](const void* p, int64_t ld) { return ((uintptr_t)p % 4) == 0 && (ld * (int64_t)sizeof(T)) % 4 == 0; };
  a.endA = a.vecA != 4;
  if (a.endA && (a.K < 4 || !words(a.A, a.lda) || (a.K * sizeof(T)) % 4 != 0)) return false;
  a.endC |= a.vecC != 4 || (a.C2 && a.vecC2 != 4);
  if (a.endC && (!words(a.C, a.ldc) || (a.C2 && !words(a.C2, a.ldc2)))) return false;
  if (a.mask && (a.vecM != 4 || a.mask_rows < a.M || a.C2)) return false;
  if (a.ldc >= 1 << 24 || a.ldc2 >= 1 << 24 || a.ldmask >= 1 << 24) return false;      // (16 rows are one buffer, with 32-bit offsets)
  const int ku = a.K % 128 == 0 ? 8 : a.K < 128 ? (a.K + 15) / 16 : 0;
  if (ku == 0) return false;
#define GCN_NN_FAST(NTV)                                              \
  {                                                                   \
    switch (ku) {                                                     \
      case 1: *rc = nn_launch_fast<T, NTV, 1>(a, s); break;           \
      case 2: *rc = nn_launch_fast<T, NTV, 2>(a, s); break;           \
      case 3: *rc = nn_launch_fast<T, NTV, 3>(a, s); break;           \
      case 4: *rc = nn_launch_fast<T, NTV, 4>(a, s); break;           \
      case 5: *rc = nn_launch_fast<T, NTV, 5>(a, s); break;           \
      case 6: *rc = nn_launch_fast<T, NTV, 6>(a, s); break;           \
      case 7: *rc = nn_launch_fast<T, NTV, 7>(a, s); break;           \
      default: *rc = nn_launch_fast<T, NTV, 8>(a, s); break;          \
    }                                                                 \
    return true;                                                      \
  }
  switch (NT) {
    case 1: GCN_NN_FAST(1)
    case 2: GCN_NN_FAST(2)
    case 3: GCN_NN_FAST(3)
    case 4: GCN_NN_FAST(4)
    case 8: GCN_NN_FAST(8)
    default: GCN_NN_FAST(16)
  }
#undef GCN_NN_FAST
}

template <typename T>
static int nn_dispatch(const NnDirectArgs& a, hipStream_t s) {
  int rc = GCN_OK;
  if (nn_fast<T>(a, s, &rc)) return rc;
  switch (nn_tiles(a.N)) {
    case 1: return nn_launch<T, 1>(a, s);
    case 2: return nn_launch<T, 2>(a, s);
    case 3: return nn_launch<T, 3>(a, s);
    case 4: return nn_launch<T, 4>(a, s);
    case 8: return nn_launch<T, 8>(a, s);
    default: return nn_launch<T, 16>(a, s);
  }
}

int gemm_nn_direct(const void* A, int64_t lda, const float* W, int64_t ldw, void* C, int64_t ldc, int64_t M, int N,
                   int K, int dtype, const GemmEpilogue& epi, hipStream_t s) {
  if (M == 0) return GCN_OK;
  const size_t es = dtype == GCN_BF16 ? 2 : 4;
  auto vec_of = [&](const void* p, int64_t ld) { return (p && (ld % 4) == 0 && ((uintptr_t)p % (4 * es)) == 0) ? 4 : 1; };
  NnDirectArgs a{A, lda, W, ldw, C, ldc, M, N, K, vec_of(A, lda), vec_of(C, ldc), vec_of(epi.C2, epi.ldc2),
                 vec_of(epi.mask, epi.ldmask),
                 epi.bias, epi.relu, epi.mask, epi.ldmask, epi.mask_rows, epi.C2, epi.ldc2, epi.b_trans ? 1 : 0,
                 0, N % 4 != 0 && !epi.c_rows_padded};
  return dtype == GCN_BF16 ? nn_dispatch<bf16_t>(a, s) : nn_dispatch<float>(a, s);
}

// ------------------------------------------------------------------------------------------
struct TnDirectArgs {
  const void* A; int64_t lda; const void* B; int64_t ldb;
  int64_t Kd; int M; int N; int64_t rows_per_split; int nsplit;
  float* partial;   // [nsplit][M*N]
};

constexpr int kTnMaxUK = 8;       // most row pairs whose loads are issued together

template <typename T, int TM, int TN, int kTnUK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_gemm_tn_direct(TnDirectArgs a) {
  __shared__ float red[2][TM * TN * 16 * 64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * (32 * TM), n0 = blockIdx.z * (32 * TN);
  const int64_t k_lo = (int64_t)blockIdx.x * a.rows_per_split;
  const int64_t k_hi = k_lo + a.rows_per_split < a.Kd ? k_lo + a.rows_per_split : a.Kd;
  const T* __restrict__ A = reinterpret_cast<const T*>(a.A);
  const T* __restrict__ B = reinterpret_cast<const T*>(a.B);

  // per-lane column offsets (clamped into the row so that every address is valid) and validity
  int64_t aoff[TM], boff[TN];
  bool aok[TM], bok[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) { const int m = m0 + 32 * i + c; aok[i] = m < a.M; aoff[i] = (int64_t)h * a.lda + (aok[i] ? m : 0); }
#pragma unroll
  for (int j = 0; j < TN; ++j) { const int n = n0 + 32 * j + c; bok[j] = n < a.N; boff[j] = (int64_t)h * a.ldb + (bok[j] ? n : 0); }

  floatx16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // wavefront w takes the chunks w, w + 4, ... of 2 * kTnUK rows
  constexpr int CH = 2 * kTnUK;
  for (int64_t k = k_lo + (int64_t)w * CH; k < k_hi; k += 4 * CH) {
    float av[kTnUK][TM], bv[kTnUK][TN];
    if (k + CH <= k_hi) {
#pragma unroll
      for (int u = 0; u < kTnUK; ++u) {
        const T* __restrict__ ar = A + (k + 2 * u) * a.lda;
        const T* __restrict__ br = B + (k + 2 * u) * a.ldb;
#pragma unroll
        for (int i = 0; i < TM; ++i) av[u][i] = load_one<T>(ar + aoff[i]);
#pragma unroll
        for (int j = 0; j < TN; ++j) bv[u][j] = load_one<T>(br + boff[j]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < kTnUK; ++u) {
        const int64_t kr = k + 2 * u + h;
        const bool rok = kr < k_hi;
        const int64_t kc = rok ? k + 2 * u : k_lo - h;       // kc + h stays inside [k_lo, k_hi)
        const T* __restrict__ ar = A + kc * a.lda;
        const T* __restrict__ br = B + kc * a.ldb;
#pragma unroll
        for (int i = 0; i < TM; ++i) { const float v = load_one<T>(ar + aoff[i]); av[u][i] = rok ? v : 0.f; }
#pragma unroll
        for (int j = 0; j < TN; ++j) { const float v = load_one<T>(br + boff[j]); bv[u][j] = rok ? v : 0.f; }
      }
    }
#pragma unroll
    for (int u = 0; u < kTnUK; ++u) {
#pragma unroll
      for (int i = 0; i < TM; ++i) { if (!aok[i]) av[u][i] = 0.f; }
#pragma unroll
      for (int j = 0; j < TN; ++j) { if (!bok[j]) bv[u][j] = 0.f; }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u][i], bv[u][j], acc[i][j], 0, 0, 0);
    }
  }

  // add the four wavefronts' tiles: (2,3) -> LDS -> (0,1) add; 1 -> LDS -> 0 adds
  auto dump = [&](float* buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) buf[((i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
  };
  auto take = [&](const float* buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += buf[((i * TN + j) * 16 + r) * 64 + lane];
  };
  if (w >= 2) dump(red[w - 2]);
  __syncthreads();
  if (w < 2) take(red[w]);
  __syncthreads();
  if (w == 1) dump(red[0]);
  __syncthreads();
  if (w != 0) return;
  take(red[0]);
  float* __restrict__ P = a.partial + (int64_t)blockIdx.x * a.M * a.N;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + 32 * j + c;
      if (n >= a.N) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + 32 * i + 8 * (r / 4) + 4 * h + (r % 4);
        if (m < a.M) P[(int64_t)m * a.N + n] = acc[i][j][r];
      }
    }
}

// ---- the same contraction with vector requests ------------------------------------------------------------
// The texture path takes as long for a 4-byte request per lane as for a 16-byte one, and the kernel above
// issues one 4-byte request per MFMA: it is bound by that path, not by the matrix pipe or by memory.  Here a
// lane asks for 4 consecutive columns of A at once (and TN consecutive columns of B): component i of the
// request is the lane's operand for column tile i, so tile i holds the columns {4 c + i} and the 32 lanes of a
// row half read 512 contiguous bytes.  The MFMA never sees the permutation; it is undone when the partial tile
// is stored.  One request per four (TN = 1) or four requests per sixteen (TN = 2) MFMAs.  The next chunk's
// requests are issued before the MFMAs of the current one; scheduling barriers keep them there.
// Needs rows of A aligned to TM = 4 elements (2 up to 64 columns: tn_narrow_ok) and, for TN = 2, rows of B aligned to 2.
template <typename T, int N> struct RawVec;
template <> struct RawVec<float, 4> { typedef floatx4 type; };
template <> struct RawVec<float, 2> { typedef float type __attribute__((ext_vector_type(2))); };
template <> struct RawVec<float, 1> { typedef float type; };
template <> struct RawVec<bf16_t, 4> { typedef uint32_t type __attribute__((ext_vector_type(2))); };
template <> struct RawVec<bf16_t, 2> { typedef uint32_t type; };
template <> struct RawVec<bf16_t, 1> { typedef uint16_t type; };

template <typename T, int N>
__device__ __forceinline__ void raw_to_f32(const typename RawVec<T, N>::type& v, uint32_t (&o)[N]) {
  if constexpr (sizeof(T) == 4) {
    if constexpr (N == 1) o[0] = __float_as_uint(v);
    else {
#pragma unroll
      for (int i = 0; i < N; ++i) o[i] = __float_as_uint(v[i]);
    }
  } else {
    if constexpr (N == 1) o[0] = (uint32_t)v << 16;
    else if constexpr (N == 2) { o[0] = v << 16; o[1] = v & 0xffff0000u; }
    else { o[0] = v[0] << 16; o[1] = v[0] & 0xffff0000u; o[2] = v[1] << 16; o[3] = v[1] & 0xffff0000u; }
  }
}

// Two columns a request (TM = 2) leave registers for two sums per column tile, even and odd row pairs: chains half as long for the
// same number of splits.
template <typename T, int TM, int TN, int UK, int WN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_gemm_tn_wide(TnDirectArgs a) {
  // the four wavefronts of a block: WN column tiles of B side by side (all of them read the same rows of A,
  // which then come from HBM once) times WK = 4 / WN interleaved sets of row chunks, added up at the end
  constexpr int CH = 2 * UK, WK = 4 / WN, SUMS = TM == 2 ? 2 : 1;
  typedef typename RawVec<T, TM>::type AV;
  typedef typename RawVec<T, TN>::type BV;
  __shared__ float red[2][TM * TN * 16 * 64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int wn = w % WN, kw = w / WN;
  const int m0 = blockIdx.y * (32 * TM), n0 = (blockIdx.z * WN + wn) * (32 * TN);
  const int64_t k_lo = (int64_t)blockIdx.x * a.rows_per_split;
  const int64_t k_hi = k_lo + a.rows_per_split < a.Kd ? k_lo + a.rows_per_split : a.Kd;
  const T* __restrict__ A = reinterpret_cast<const T*>(a.A);
  const T* __restrict__ B = reinterpret_cast<const T*>(a.B);

  // the lane's columns; a request that starts past the operand is moved to column 0 and cleared
  const int ma = m0 + TM * c, nb = n0 + TN * c;
  uint32_t amask[TM], bmask[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) amask[i] = ma + i < a.M ? 0xffffffffu : 0u;
#pragma unroll
  for (int j = 0; j < TN; ++j) bmask[j] = nb + j < a.N ? 0xffffffffu : 0u;
  // a request is (row pair, uniform over the wavefront) + (lane half and column, 32 bits per lane).  Where the
  // split ends on the first row of a pair both lane halves read that row, and a pair past the end reads the
  // first rows of the split; what is not part of the product is cleared when the values are used.
  const bool two_rows = k_lo + 1 < k_hi;
  const uint32_t acol = (uint32_t)((ma < a.M ? ma : 0) * (int64_t)sizeof(T));      // bytes
  const uint32_t bcol = (uint32_t)((nb < a.N ? nb : 0) * (int64_t)sizeof(T));
  const uint32_t aoff = acol + (uint32_t)(h * a.lda * (int64_t)sizeof(T));
  const uint32_t boff = bcol + (uint32_t)(h * a.ldb * (int64_t)sizeof(T));

  floatx16 sum[SUMS][TM][TN];
#pragma unroll
  for (int b = 0; b < SUMS; ++b)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum[b][i][j][r] = 0.f;

  auto load = [&](int64_t k, AV (&av)[UK], BV (&bv)[UK]) {
#pragma unroll
    for (int u = 0; u < UK; ++u) {
      const int64_t kp = k + 2 * u;
      const int64_t kc = kp < k_hi ? kp : k_lo;
      const bool both = kp + 1 < k_hi || (kp >= k_hi && two_rows);          // rows kc and kc + 1 both lie in the split
      av[u] = *reinterpret_cast<const AV*>(reinterpret_cast<const char*>(A + kc * a.lda) + (both ? aoff : acol));
      bv[u] = *reinterpret_cast<const BV*>(reinterpret_cast<const char*>(B + kc * a.ldb) + (both ? boff : bcol));
    }
  };
  int64_t k = k_lo + (int64_t)kw * CH;
  AV an[UK]; BV bn[UK];
  if (k < k_hi) load(k, an, bn);
  for (; k < k_hi; k += WK * CH) {
    float av[UK][TM], bv[UK][TN];
#pragma unroll
    for (int u = 0; u < UK; ++u) {
      const uint32_t rmask = k + 2 * u + h < k_hi ? 0xffffffffu : 0u;   // cleared by a bit mask, never by a branch
      uint32_t ra[TM], rb[TN];
      raw_to_f32<T, TM>(an[u], ra);
      raw_to_f32<T, TN>(bn[u], rb);
#pragma unroll
      for (int i = 0; i < TM; ++i) av[u][i] = __uint_as_float(ra[i] & (amask[i] & rmask));
#pragma unroll
      for (int j = 0; j < TN; ++j) bv[u][j] = __uint_as_float(rb[j] & (bmask[j] & rmask));
    }
    __builtin_amdgcn_sched_barrier(0);
    const int64_t kn = k + WK * CH;
    load(kn < k_hi ? kn : k, an, bn);                      // past the end: the current chunk again, unused
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < UK; ++u)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          sum[u % SUMS][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[u][i], bv[u][j], sum[u % SUMS][i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }

  floatx16 (&acc)[TM][TN] = sum[0];
  if constexpr (SUMS == 2) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] += sum[1][i][j];
  }

  // add up the row sets of a column tile
  auto dump = [&](float* buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) buf[((i * TN + j) * 16 + r) * 64 + lane] = acc[i][j][r];
  };
  auto take = [&](const float* buf) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] += buf[((i * TN + j) * 16 + r) * 64 + lane];
  };
  if constexpr (WK == 4) {               // (2, 3) -> LDS -> (0, 1) add; 1 -> LDS -> 0 adds
    if (kw >= 2) dump(red[kw - 2]);
    __syncthreads();
    if (kw < 2) take(red[kw]);
    __syncthreads();
    if (kw == 1) dump(red[0]);
    __syncthreads();
    if (kw != 0) return;
    take(red[0]);
  } else if constexpr (WK == 2) {        // the second row set of each column tile -> LDS -> the first adds
    if (kw == 1) dump(red[wn]);
    __syncthreads();
    if (kw != 0) return;
    take(red[wn]);
  }
  // register r of lane (c, h) holds the product of A's lane 8 (r / 4) + 4 h + r % 4 and B's lane c
  float* __restrict__ P = a.partial + (int64_t)blockIdx.x * a.M * a.N;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = nb + j;
      if (n >= a.N) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = m0 + TM * (8 * (r / 4) + 4 * h + (r % 4)) + i;
        if (m < a.M) P[(int64_t)m * a.N + n] = acc[i][j][r];
      }
    }
}

constexpr int kWideUK1 = 8, kWideUK2 = 8;   // row pairs per request batch (TN = 1, TN = 2)

bool gemm_tn_wide_ok(const void* A, int64_t lda, const void* B, int64_t ldb, int N, int dtype) {
  const bool off = tune().gemm_tn_wide == 0;
  const size_t es = dtype == GCN_BF16 ? 2 : 4;
  if (off || (lda % 4) != 0 || ((uintptr_t)A % (4 * es)) != 0) return false;
  if (lda >= (1 << 28) || ldb >= (1 << 28)) return false;      // a lane's offset (one row + a column, in bytes) is kept in 32 bits
  if (N > 32 && ((ldb % 2) != 0 || ((uintptr_t)B % (2 * es)) != 0)) return false;
  return true;
}

// Up to 64 columns of A in fp32: two of them a request (TM = 2), and no matrix operations on a second pair of column tiles that does not
// exist.  M even (and N, beyond 32), so that no request reaches past the end of a row.
// Rows of whole quads otherwise take four columns a request; measured, us with four / two: 2 K rows x 50 x 50 22.6 / 17.3, 20 K x 50 x
// 256 88 / 62, 150 K x 50 x 50 45 / 33, 500 K x 64 x 64 98 / 66 (a copy's rate is 47), 64 x 16 63 / 46, 32 x 128 167 / 109.
// Other rows take k_gemm_tn_direct, and this form only where it gains on it: from 3 2^17 rows on with up to 64 columns of B, from 2^19 on
// with up to 128, from 3 2^18 on with all four column tiles.  us there / here, each pass on other operands: 2 K x 50 x 50 16.2 / 17.3, 140 K
// 27 / 30, 330 K 48 / 50, 400 K 59 / 56, 500 K 68.8 / 68.0, 780 K 97 / 93 (34 x 62, 62 x 34 and 50 x 64 alike, at pitches of 50, 52 and 96);
// 2 K x 50 x 256 22 / 58, 150 K x 50 x 100 42 / 47, 400 K x 50 x 100 88 / 90, 1 M x 50 x 100 229 / 200, 50 x 256 407 / 387; never 50 x 160 (340 / 391) or 50 x 300
// (550 / 760).  Its splits are half as many there, of two sums each: chains as long as k_gemm_tn_direct's, and the same error against 64
// bits (500 K x 50 x 100 2.9e-7; 4.1e-7 with one sum).
static bool tn_narrow_ok(const void* A, int64_t lda, const void* B, int64_t ldb, int64_t Kd, int M, int N, int dtype) {
  if (tune().gemm_tn_wide == 0 || dtype != GCN_F32 || M > 64) return false;
  if (M % 2 != 0 || (lda % 2) != 0 || ((uintptr_t)A % 8) != 0 || lda >= (1 << 28) || ldb >= (1 << 28)) return false;
  if (gemm_tn_wide_ok(A, lda, B, ldb, N, dtype)) return N <= 32 || N % 2 == 0;
  if (N <= 32 || N % 2 != 0 || (ldb % 2) != 0 || ((uintptr_t)B % 8) != 0) return false;
  if (N > 256 || (N > 128 && N <= 192)) return false;
  return Kd >= (N <= 64 ? 3 << 17 : N <= 128 ? 2 << 18 : 3 << 18);
}

// column tiles of B per block in the vector variant: all of B for up to 256 columns
int tn_wide_wn(int N) { return N <= 64 ? 1 : N <= 128 ? 2 : 4; }

// Most splits that the rows admit.  A split costs its partial tile (written, then read by the sum), so it has about 512 rows
// where that gives every compute unit a workgroup, rounded to a whole number of workgroups per compute unit (the last, half
// empty round of a launch costs as much as a full one).  Below, what counts is the chain of row chunks of a workgroup: splits
// get shorter, down to 64 rows for narrow outputs and 512 for wide ones, until there are 256 workgroups.  Measured, us with 512
// rows / the shortest splits / this rule: 4 K rows x 64 x 16 fp32 21 / 11 / 11, 60 K x 50 x 50 21 / 18 / 16, 130 K x 128 x 41 33 /
// 40 / 32, 150 K x 50 x 50 32 / 29 / 25, 2^18 x 50 x 50 34 / 38 / 34, 416 K x 47 x 16 bf16 37 / 33 / 33; on the average of 13 row
// counts up to 500 K and 11 widths in both types 1 / 0.92 / 0.87, against the first at worst 1.08 (130 K x 256 x 47).
static int64_t tn_max_splits(int64_t Kd, int M, int N, int64_t tiles) {
  const int64_t r = (int64_t)M * N / 32;
  const int64_t min_rows = r < 64 ? 64 : r > 512 ? 512 : round_up(r, 64);
  const int64_t per_cu = std::max<int64_t>(1, ceil_div(Kd * tiles, 512 * 256));
  return std::max(ceil_div(Kd, 512), std::min(ceil_div(Kd, min_rows), ceil_div(256 * per_cu, tiles)));
}

// splits of the vector variant: about two blocks per compute unit
int tn_wide_splits(int64_t Kd, int M, int N) {
  const int blocks = tune().gemm_tn_blocks;
  const int64_t tiles = ceil_div(M, 128) * ceil_div(N, (N <= 32 ? 32 : 64) * tn_wide_wn(N));
  int64_t want = ceil_div(blocks, tiles);
  int64_t max_by_k = tn_max_splits(Kd, M, N, tiles);
  int64_t ns = want < max_by_k ? want : max_by_k;
  return (int)(ns < 1 ? 1 : ns);
}

static int tn_direct_tn(int N) { return N <= 32 ? 1 : 2; }

static int tn_direct_splits(int64_t Kd, int M, int N) {
  const int64_t tiles = ceil_div(M, 64) * ceil_div(N, 32 * tn_direct_tn(N));
  int64_t want = ceil_div(1024, tiles);                // about four blocks per compute unit
  int64_t max_by_k = tn_max_splits(Kd, M, N, tiles);
  int64_t ns = want < max_by_k ? want : max_by_k;
  return (int)(ns < 1 ? 1 : ns);
}

size_t gemm_tn_direct_ws_bytes(int64_t Kd, int M, int N) {
  const int ns = std::max(tn_direct_splits(Kd, M, N), tn_wide_splits(Kd, M, N));
  return std::max(std::max(sizeof(float) * (size_t)ns * (size_t)M * (size_t)N, gemm_tn_lds_ws_bytes(Kd, M, N)), gemm_tn_split_ws_bytes(Kd, M, N));
}

bool gemm_tn_takes_split(const void* A, int64_t lda, const void* B, int64_t ldb, int64_t Kd, int M, int N, int dtype, bool beside) {
  return !(beside && gemm_tn_lds_ok(A, lda, B, ldb, Kd, M, N, dtype)) && gemm_tn_split_ok(A, lda, B, ldb, Kd, M, N, dtype);
}

int gemm_tn_direct_partials(const void* A, int64_t lda, const void* B, int64_t ldb, int64_t Kd, int M, int N, int dtype,
                            float* partial, int* nsplit_out, hipStream_t s, int max_blocks, bool beside) {
  if (dtype == GCN_BF16 && gemm_tn_bf16_ok(A, lda, B, ldb, Kd, M, N))
    return gemm_tn_bf16_partials(A, lda, B, ldb, Kd, M, N, partial, nsplit_out, s);
  if (gemm_tn_takes_split(A, lda, B, ldb, Kd, M, N, dtype, beside))
    return gemm_tn_split_partials(A, lda, B, ldb, Kd, M, N, partial, nsplit_out, s, max_blocks);
  if (gemm_tn_lds_ok(A, lda, B, ldb, Kd, M, N, dtype)) return gemm_tn_lds_partials(A, lda, B, ldb, Kd, M, N, partial, nsplit_out, s, max_blocks);
  TnDirectArgs a{A, lda, B, ldb, Kd, M, N, 0, 0, partial};
  const bool narrow = tn_narrow_ok(A, lda, B, ldb, Kd, M, N, dtype);
  if (narrow || gemm_tn_wide_ok(A, lda, B, ldb, N, dtype)) {
    a.nsplit = tn_wide_splits(Kd, M, N);
    a.rows_per_split = round_up(ceil_div(Kd > 0 ? Kd : 1, a.nsplit), 2 * kTnMaxUK);
    *nsplit_out = a.nsplit;
    const int tnw = N <= 32 ? 1 : 2, wnw = tn_wide_wn(N);
    dim3 grid((unsigned)a.nsplit, (unsigned)ceil_div(M, 128), (unsigned)ceil_div(N, 32 * tnw * wnw));
#define GCN_TN_WIDE(TT, TM)                                                                    \
    if (tnw == 1) k_gemm_tn_wide<TT, TM, 1, kWideUK1, 1><<<grid, 256, 0, s>>>(a);               \
    else if (wnw == 1) k_gemm_tn_wide<TT, TM, 2, kWideUK2, 1><<<grid, 256, 0, s>>>(a);          \
    else if (wnw == 2) k_gemm_tn_wide<TT, TM, 2, kWideUK2, 2><<<grid, 256, 0, s>>>(a);          \
    else k_gemm_tn_wide<TT, TM, 2, kWideUK2, 4><<<grid, 256, 0, s>>>(a);
    if (narrow) { GCN_TN_WIDE(float, 2) }
    else if (dtype == GCN_BF16) { GCN_TN_WIDE(bf16_t, 4) } else { GCN_TN_WIDE(float, 4) }
#undef GCN_TN_WIDE
    GCN_CHECK_LAUNCH();
    return GCN_OK;
  }
  a.nsplit = tn_direct_splits(Kd, M, N);
  a.rows_per_split = round_up(ceil_div(Kd > 0 ? Kd : 1, a.nsplit), 2 * kTnMaxUK);
  *nsplit_out = a.nsplit;
  const int tn = tn_direct_tn(N);
  dim3 grid((unsigned)a.nsplit, (unsigned)ceil_div(M, 64), (unsigned)ceil_div(N, 32 * tn));
  if (dtype == GCN_BF16) {
    if (tn == 1) k_gemm_tn_direct<bf16_t, 2, 1, 8><<<grid, 256, 0, s>>>(a);
    else k_gemm_tn_direct<bf16_t, 2, 2, 4><<<grid, 256, 0, s>>>(a);
  } else {
    if (tn == 1) k_gemm_tn_direct<float, 2, 1, 8><<<grid, 256, 0, s>>>(a);
    else k_gemm_tn_direct<float, 2, 2, 4><<<grid, 256, 0, s>>>(a);
  }
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

}  // namespace gcn
