// Device templates of the sparse-times-dense kernels (included by spmm.hip, spmm_f32.hip, spmm_bf16.hip, spmm_dense.hip).
#pragma once
#include <stdlib.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace gcn {

// V elements moved by one request.  Rows need only start on a 4-byte word (2-byte elements alone: on an element): the
// global memory path takes 8- and 16-byte requests at any word address.
template <typename T, int V> struct Vec;
template <> struct Vec<float, 1> { typedef float type; };
template <> struct Vec<float, 2> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Vec<float, 4> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec<bf16_t, 1> { typedef uint16_t type; };
template <> struct Vec<bf16_t, 2> { typedef uint32_t type; };
template <> struct Vec<bf16_t, 4> { typedef uint32_t type __attribute__((ext_vector_type(2), aligned(4))); };
template <> struct Vec<bf16_t, 8> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };

template <typename T, int V>
__device__ __forceinline__ void unpack_vec(const typename Vec<T, V>::type& raw, float (&out)[V]) {
  if constexpr (V == 1) {
    if constexpr (sizeof(T) == 4) out[0] = raw;
    else out[0] = bf16_to_f32(raw);
  } else if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int i = 0; i < V; ++i) out[i] = raw[i];
  } else if constexpr (V == 2) {
    out[0] = __uint_as_float(raw << 16); out[1] = __uint_as_float(raw & 0xffff0000u);
  } else {
#pragma unroll
    for (int i = 0; i < V / 2; ++i) { out[2 * i] = __uint_as_float(raw[i] << 16); out[2 * i + 1] = __uint_as_float(raw[i] & 0xffff0000u); }
  }
}

template <typename T, int V>
__device__ __forceinline__ void load_vec(const T* __restrict__ p, float (&out)[V]) {
  unpack_vec<T, V>(*reinterpret_cast<const typename Vec<T, V>::type*>(p), out);
}

template <typename T, int V>
__device__ __forceinline__ void store_vec(T* __restrict__ p, const float (&v)[V]) {
  if constexpr (V == 1) {
    store_one<T>(p, v[0]);
  } else {
    typename Vec<T, V>::type raw;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < V; ++i) raw[i] = v[i];
    } else if constexpr (V == 2) {
      raw = (uint32_t)f32_to_bf16(v[0]) | ((uint32_t)f32_to_bf16(v[1]) << 16);
    } else {
#pragma unroll
      for (int i = 0; i < V / 2; ++i) raw[i] = (uint32_t)f32_to_bf16(v[2 * i]) | ((uint32_t)f32_to_bf16(v[2 * i + 1]) << 16);
    }
    *reinterpret_cast<typename Vec<T, V>::type*>(p) = raw;
  }
}

// Ordinary rows have 0 .. kHubRowNnz entries: at most this many length classes.
constexpr int kMaxBins = 13;
static_assert(kHubRowNnz == 2048, "kMaxBins counts the classes up to 2048 entries and the empty rows");

struct SpmmK {
  const int64_t* ptr; const int32_t* idx; const float* val;
  // entries of row r that take part: [lo[r], hi[r]); the whole row is lo = ptr, hi = ptr + 1
  const int64_t* lo; const int64_t* hi;
  int accumulate;     // 1: the result is added to what Y holds (a product split in two column ranges)
  const int32_t* wave_rows;
  const int32_t* hub_rows; const int64_t* hub_chunk_ptr; const int32_t* chunk_hub; int64_t n_chunks;
  int64_t n_hub_rows;
  int64_t chunk_lo, hub_lo;   // a launch on a range of rows: first chunk of entries and first hub row it covers (else 0)
  const void* X; int64_t ldx;
  void* Y; int64_t ldy;
  void* Y2; int64_t ldy2;
  const float* bias; const void* Zprev; int64_t ldz; int64_t n_mask_rows;
  float* partial;     // [n_chunks x d] partial rows of hub chunks
  int d; int epilogue;
  uint32_t row_bytes; // ldx in bytes (used by the 32-bit addressing variant)
  uint32_t x_bytes;   // bytes of X that may be read (32-bit addressing variant)
  int S;              // feature slices; block b works on slice b % S (one slice per XCD group)
  int nvec, vps;      // V-wide vectors per row / per slice
  int c_last;         // first column of a row's last vector: d - V where reading past column d is not allowed
  int y_vec;          // Y, Y2 and Zprev are accessed V elements at a time (else one by one) ...
  int y_full;         // ... the last vector of a row included
  int short_rows;     // rows are short: two vectors per lane, so that a wavefront takes more rows (launch_v)
  // ordinary rows: bin b holds the rows wave_rows[bin_row_begin[b] .. bin_row_end[b]) of one length
  // class; 2^bin_log2gr[b] lane groups share a row, so a wavefront takes G >> bin_log2gr[b] rows and
  // the bin's wavefronts are numbered from bin_wave_begin[b].  More than all groups of a wavefront (2^bin_log2gr[b] > G): the
  // four wavefronts of a block share a row, a quarter of its entries each.
  int64_t n_waves;
  int64_t bin_wave_begin[kMaxBins];      // n_waves where there is no such bin
  int64_t bin_row_begin[kMaxBins];
  int64_t bin_row_end[kMaxBins];
  int bin_log2gr[kMaxBins];
};

// One gathered feature vector: X[j, c0 .. c0+V) with c0b = c0 in bytes, as it is stored.  A lane with ok == false gets
// zeros and asks for nothing.
// NARROW: a buffer request with a 32-bit byte offset (24-bit row index times 24-bit row pitch); a lane that wants
// nothing asks past the buffer's end, which the request's range check answers with zeros: no branch around the request,
// so the requests of several entries stay in flight together.  Else a global request under the lane's execution mask.
constexpr uint32_t kNoOffset = 0xfffffff0u;          // past every buffer the narrow form is used for (spmm_launch)
typedef __amdgpu_buffer_rsrc_t XBuf;
template <typename T, int V, bool NARROW>
__device__ __forceinline__ typename Vec<T, V>::type gather_raw(const SpmmK& a, XBuf xb, int32_t j, uint32_t c0b, bool ok) {
  typedef typename Vec<T, V>::type R;
  R r;
  if constexpr (NARROW) {
    uint32_t off = __umul24((uint32_t)j, a.row_bytes) + c0b;
    off = ok ? off : kNoOffset;
    if constexpr (sizeof(R) == 16) { const auto q = __builtin_amdgcn_raw_buffer_load_b128(xb, (int)off, 0, 0); __builtin_memcpy(&r, &q, 16); }
    else if constexpr (sizeof(R) == 8) { const auto q = __builtin_amdgcn_raw_buffer_load_b64(xb, (int)off, 0, 0); __builtin_memcpy(&r, &q, 8); }
    else if constexpr (sizeof(R) == 4) { const auto q = __builtin_amdgcn_raw_buffer_load_b32(xb, (int)off, 0, 0); __builtin_memcpy(&r, &q, 4); }
    else { const auto q = __builtin_amdgcn_raw_buffer_load_b16(xb, (int)off, 0, 0); __builtin_memcpy(&r, &q, 2); }
  } else {
    __builtin_memset(&r, 0, sizeof(R));
    if (ok) r = *reinterpret_cast<const R*>(reinterpret_cast<const char*>(a.X) + ((int64_t)j * a.ldx * (int64_t)sizeof(T) + c0b));
  }
  return r;
}

__device__ __forceinline__ int32_t lane_read(int byte_addr, int32_t v) { return __builtin_amdgcn_ds_bpermute(byte_addr, v); }
__device__ __forceinline__ float lane_read(int byte_addr, float v) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(byte_addr, __float_as_int(v)));
}

// A "team" of 2^lgr lane groups (TL = LPR << lgr consecutive lanes starting at wave lane team_lane0)
// adds up n entries of one sparse row:  acc[q] += sum_k val[k] * X[idx[k], c0[q] .. c0[q]+V), q < NV.
// The team reads idx/val a batch of KB TL entries at a time, KB consecutive ones per lane with one request each (with
// KB = 4 a request may reach past the row's end, not past the arrays' slack), the next batch before the current one is
// used; a lane group then fetches the indices and values of its entries from the owning lanes by cross-lane reads and
// keeps U NV gathered feature vectors in flight (a "round" of U entries).
//   KB = 4: a line of the index streams is asked for once or twice and not once per short batch, of which the L1 would
//           keep none (20 wavefronts with up to 16 teams each touch more lines than it has).  Measured on 2^18 rows with
//           45 entries each, KB = 1 / 4: fp32 width 16 90 / 86 us, width 128 391 / 383, bf16 width 16 90 / 85.
//   KB = 1: short batches, so that most are full and take the rounds without validity checks; what counts where the
//           kernel is bound by instruction issue, as it is with the 8 elements per request of bf16 (width 64 115 / 121 us,
//           width 128 217 / 233).
// Lanes without a feature vector in this slice are handed a column that the slice reads anyway
// and never store.  Different teams of a wavefront may hold rows of
// different length: every cross-lane operation sits outside divergent code and loop exits are
// taken on wave-wide votes.  LGR >= 0 fixes lgr at compile time.
typedef int32_t i32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int KB> struct EntryRegs { typedef i32x4u idx; typedef f32x4u val; };
template <> struct EntryRegs<1> { typedef int32_t idx; typedef float val; };
template <typename T, int V, int LPR, int NV, bool NARROW, int LGR>
__device__ __forceinline__ void team_accumulate(const SpmmK& a, XBuf xb, const int32_t* __restrict__ idx, const float* __restrict__ val, int n,
                                                int lgr_rt, int team_lane0, int gg, int t, const uint32_t (&c0b)[NV], float (&acc)[NV][V]) {
  constexpr int KB = LPR >= 8 && sizeof(T) == 2 ? 1 : 4;          // entries per lane and batch
  // entries per group and round: 64 bytes in flight per lane, or 8 narrow requests (bf16 rows of odd width or pitch, R-MAT of
  // 100 K rows with 23 entries, width 17 / 47 / 301: 86 / 157 / 775 us with 4 in flight, 62 / 108 / 523 with 8)
  constexpr int U = KB == 1 && sizeof(T) * V < 16 ? 8 : 4;
  constexpr int ROUNDS = LPR * KB / U;
  typedef typename EntryRegs<KB>::idx JV;
  typedef typename EntryRegs<KB>::val WV;
  const int lgr = LGR >= 0 ? LGR : lgr_rt;
  const int groups = 1 << lgr;
  const int TL = LPR << lgr;
  const int src0 = (team_lane0 + gg) << 2;          // byte address of the lane holding the group's first entries
  int base = 0;
  JV jreg{}; WV wreg{};
  if (KB * t < n) { jreg = *reinterpret_cast<const JV*>(idx + KB * t); wreg = *reinterpret_cast<const WV*>(val + KB * t); }
  while (__any(base < n)) {
    const int nb = base + KB * TL;
    JV jn{}; WV wn{};
    if (nb + KB * t < n) { jn = *reinterpret_cast<const JV*>(idx + nb + KB * t); wn = *reinterpret_cast<const WV*>(val + nb + KB * t); }
    const int left = n - base;
    const int cnt = left <= 0 ? 0 : (left < KB * TL ? left : KB * TL);
    // all vectors of a round are requested before the first is used
    auto round = [&](int k, auto whole) {
      int32_t j[U]; float w[U]; bool ok[U]; typename Vec<T, V>::type x[U][NV];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if constexpr (KB == 1) {         // entries gg, gg + groups, ...: one lane each
          const int src = src0 + ((U * k + u) << (lgr + 2));
          j[u] = lane_read(src, jreg);
          w[u] = lane_read(src, wreg);
          ok[u] = decltype(whole)::value || (U * k + u) * groups + gg < cnt;
        } else {                         // the 4 entries of team lane k groups + gg
          const int src = src0 + (k << (lgr + 2));
          j[u] = lane_read(src, jreg[u]);
          w[u] = lane_read(src, wreg[u]);
          ok[u] = decltype(whole)::value || U * ((k << lgr) + gg) + u < cnt;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int q = 0; q < NV; ++q) x[u][q] = gather_raw<T, V, NARROW>(a, xb, j[u], c0b[q], ok[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if constexpr (KB > 1 && !decltype(whole)::value) w[u] = ok[u] ? w[u] : 0.f;      // (zero weight times zero where there is no entry)
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          float f[V];
          unpack_vec<T, V>(x[u][q], f);
#pragma unroll
          for (int v = 0; v < V; ++v) acc[q][v] = fmaf(w[u], f[v], acc[q][v]);
        }
      }
    };
    if (__all(cnt == KB * TL)) {
#pragma unroll 1
      for (int k = 0; k < ROUNDS; ++k) round(k, std::true_type{});
    } else {
#pragma unroll 1
      for (int k = 0; k < ROUNDS; ++k) {
        if (!__any(U * k * groups < cnt)) break;
        round(k, std::false_type{});
      }
    }
    jreg = jn; wreg = wn;
    base = nb;
  }
}

// butterfly over the `groups` (power of two) lane groups of LPR lanes that share a row
template <int V, int LPR, int NV>
__device__ __forceinline__ void reduce_groups(float (&acc)[NV][V], int groups) {
  for (int off = LPR; off < LPR * groups; off <<= 1)
#pragma unroll
    for (int q = 0; q < NV; ++q)
#pragma unroll
      for (int v = 0; v < V; ++v) acc[q][v] += __shfl_xor(acc[q][v], off, 64);
}

// epilogue on one element of output row `row`, feature c
template <typename T>
__device__ __forceinline__ void finish_element(const SpmmK& a, int64_t row, int64_t c, float v) {
  if (a.accumulate) v += load_one<T>(reinterpret_cast<const T*>(a.Y) + row * a.ldy + c);
  if (a.bias) v += a.bias[c];
  if (a.Y2) store_one<T>(reinterpret_cast<T*>(a.Y2) + row * a.ldy2 + c, v);
  if (a.epilogue == GCN_EPI_RELU) v = v > 0.f ? v : 0.f;
  else if (a.epilogue == GCN_EPI_MASK && row < a.n_mask_rows) {
    float z = load_one<T>(reinterpret_cast<const T*>(a.Zprev) + row * a.ldz + c);
    v = z > 0.f ? v : 0.f;
  }
  store_one<T>(reinterpret_cast<T*>(a.Y) + row * a.ldy + c, v);
}

// the same on V consecutive elements, written with one vector store per output (bias: only the elements below column d)
template <typename T, int V>
__device__ __forceinline__ void finish_vector(const SpmmK& a, int64_t row, int64_t c0, float (&v)[V]) {
  if (a.accumulate) {
    float old[V];
    load_vec<T, V>(reinterpret_cast<const T*>(a.Y) + row * a.ldy + c0, old);
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] += old[i];
  }
  if (a.bias) {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] += c0 + i < a.d ? a.bias[c0 + i] : 0.f;
  }
  if (a.Y2) store_vec<T, V>(reinterpret_cast<T*>(a.Y2) + row * a.ldy2 + c0, v);
  if (a.epilogue == GCN_EPI_RELU) {
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = v[i] > 0.f ? v[i] : 0.f;
  } else if (a.epilogue == GCN_EPI_MASK && row < a.n_mask_rows) {
    const T* zp = reinterpret_cast<const T*>(a.Zprev) + row * a.ldz + c0;
    float z[V];
    load_vec<T, V>(zp, z);
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = z[i] > 0.f ? v[i] : 0.f;
  }
  store_vec<T, V>(reinterpret_cast<T*>(a.Y) + row * a.ldy + c0, v);
}

// BLOCKS: there are rows that take a block each (make_bins).  A product without them, which large ones are, keeps the shorter
// kernel: with the branch and its code in the same instance R-MAT 2^18 and 500 K short rows lost 0.6 %.
template <typename T, int V, int LPR, int NV, bool NARROW, bool BLOCKS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_spmm(SpmmK a) {
  constexpr int G = 64 / LPR;
  constexpr int kLog2G = G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : G == 8 ? 3 : G == 16 ? 4 : G == 32 ? 5 : 6;
  constexpr int TV = LPR * NV;      // vectors covered by one group
  constexpr int TW = TV * V;        // ... and the features in them
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane / LPR, l = lane % LPR;
  int slice; int64_t item;
  if (gridDim.y == 1) {       // the usual case: 32-bit division
    slice = (int)(blockIdx.x % (unsigned)a.S); item = blockIdx.x / (unsigned)a.S;
  } else {
    const int64_t bid = block_id();
    slice = (int)(bid % a.S); item = bid / a.S;
  }
  const int v_lo = slice * a.vps;
  const int v_hi = v_lo + a.vps < a.nvec ? v_lo + a.vps : a.nvec;
  __shared__ float part[4][TW];
  // (0x00020000: a plain buffer of 32-bit words)
  const XBuf xb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.X), 0, (int)a.x_bytes, 0x00020000);

  // first column of vector vi: the last vector of a row is moved back to end on column d where reading past it is not
  // allowed (its leading elements then repeat the vector before it and are not stored)
  auto column = [&](int vi) -> int { return vi == a.nvec - 1 ? a.c_last : vi * V; };

  const bool chunk = item < a.n_chunks;
  const int64_t wi = (item - a.n_chunks) * 4 + w;
  int b = -1;
  // ---- a block on one row: a run of entries per wavefront, which meet in LDS
  auto on_one_row = [&]() {
    int64_t row, ws; int n; float* partial = nullptr;
    if (chunk) {           // kHubChunkNnz entries of a hub row
      const int64_t c = a.chunk_lo + item;
      const int32_t h = a.chunk_hub[c];
      row = a.hub_rows[h];
      const int64_t cs = a.ptr[row] + (c - a.hub_chunk_ptr[h]) * kHubChunkNnz;      // chunks are cut from the whole row
      const int64_t row_lo = a.lo[row], row_hi = a.hi[row];
      const int64_t s = cs > row_lo ? cs : row_lo;
      const int64_t e = cs + kHubChunkNnz < row_hi ? cs + kHubChunkNnz : row_hi;
      ws = s + (int64_t)w * (kHubChunkNnz / 4);
      const int64_t we = ws + kHubChunkNnz / 4 < e ? ws + kHubChunkNnz / 4 : e;
      n = ws < we ? (int)(we - ws) : 0;
      partial = a.partial + c * a.d;
    } else {               // a whole row: these bins come first, four wavefronts a row, so that all are of one block
      row = a.wave_rows[a.bin_row_begin[b] + (wi - a.bin_wave_begin[b]) / 4];
      const int64_t s = a.lo[row];
      const int all = (int)(a.hi[row] - s), quarter = (all + 3) >> 2, left = all - w * quarter;
      ws = s + (int64_t)w * quarter;
      n = left < 0 ? 0 : left < quarter ? left : quarter;
    }
    for (int t0 = v_lo; t0 < v_hi; t0 += TV) {
      uint32_t c0b[NV];
      float acc[NV][V];
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int vi = t0 + l + LPR * q;
        c0b[q] = (uint32_t)column(vi < v_hi ? vi : v_lo) * (uint32_t)sizeof(T);
#pragma unroll
        for (int v = 0; v < V; ++v) acc[q][v] = 0.f;
      }
      team_accumulate<T, V, LPR, NV, NARROW, kLog2G>(a, xb, a.idx + ws, a.val + ws, n, kLog2G, 0, g, lane, c0b, acc);
      reduce_groups<V, LPR, NV>(acc, G);
      if (g == 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          const int vi = t0 + l + LPR * q;
          const int skip = vi < v_hi ? vi * V - column(vi) : 0;
#pragma unroll
          for (int v = 0; v < V; ++v)
            if (v >= skip) part[w][(l + LPR * q) * V + v - skip] = acc[q][v];
        }
      }
      __syncthreads();
      const int f0 = t0 * V;
      const int f_end = v_hi * V < a.d ? v_hi * V : a.d;
      for (int f = threadIdx.x; f < TW && f0 + f < f_end; f += 256) {
        const float v = (part[0][f] + part[1][f]) + (part[2][f] + part[3][f]);
        if (chunk) partial[f0 + f] = v;
        else finish_element<T>(a, row, f0 + f, v);
      }
      __syncthreads();
    }
  };
  if constexpr (!BLOCKS) {
    if (chunk) { on_one_row(); return; }
  }
  if (wi >= a.n_waves) return;
  // the bin of this wavefront: counted over all bins with their limits in scalar registers (a search would be a chain of
  // dependent loads of the arguments)
#pragma unroll
  for (int i = 0; i < kMaxBins; ++i) b += wi >= a.bin_wave_begin[i] ? 1 : 0;
  const int lgr = BLOCKS && chunk ? kLog2G + 1 : a.bin_log2gr[b];
  if constexpr (BLOCKS) {
    if (lgr > kLog2G) { on_one_row(); return; }
  }

  // ---- ordinary rows: a wavefront takes R = G >> lgr rows of one length class
  const int groups = 1 << lgr;
  const int q0 = g >> lgr, gg = g & (groups - 1);
  const int64_t ri = a.bin_row_begin[b] + (wi - a.bin_wave_begin[b]) * (G >> lgr) + q0;
  const bool has_row = ri < a.bin_row_end[b];
  int64_t row = 0, s = 0; int n = 0;
  if (has_row) { row = a.wave_rows[ri]; s = a.lo[row]; n = (int)(a.hi[row] - s); }
  for (int t0 = v_lo; t0 < v_hi; t0 += TV) {
    uint32_t c0b[NV];
    float acc[NV][V];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int vi = t0 + l + LPR * q;
      c0b[q] = (uint32_t)column(vi < v_hi ? vi : v_lo) * (uint32_t)sizeof(T);
#pragma unroll
      for (int v = 0; v < V; ++v) acc[q][v] = 0.f;
    }
    if (lgr == kLog2G) team_accumulate<T, V, LPR, NV, NARROW, kLog2G>(a, xb, a.idx + s, a.val + s, n, lgr, 0, g, lane, c0b, acc);
    else team_accumulate<T, V, LPR, NV, NARROW, -1>(a, xb, a.idx + s, a.val + s, n, lgr, q0 * (LPR << lgr), gg, lane - q0 * (LPR << lgr), c0b, acc);
    reduce_groups<V, LPR, NV>(acc, groups);
    if (gg == 0 && has_row) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int vi = t0 + l + LPR * q;
        if (vi >= v_hi) continue;
        const int c0 = column(vi);
        if (a.y_vec && (vi < a.nvec - 1 || a.y_full)) {
          finish_vector<T, V>(a, row, c0, acc[q]);
        } else {
#pragma unroll
          for (int v = 0; v < V; ++v)
            if (c0 + v >= vi * V && c0 + v < a.d) finish_element<T>(a, row, c0 + v, acc[q][v]);
        }
      }
    }
  }
}

// one wavefront per (hub row, 64 features): add the chunk partials in chunk order, apply the epilogue
template <typename T>
__global__ __launch_bounds__(256) void k_spmm_hub_finish(SpmmK a) {
  const int lane = threadIdx.x & 63;
  const int64_t tiles = (a.d + 63) / 64;
  const int64_t wi = block_id() * 4 + (threadIdx.x >> 6);
  if (wi >= a.n_hub_rows * tiles) return;
  const int64_t h = a.hub_lo + wi / tiles;
  const int64_t f = (wi % tiles) * 64 + lane;
  if (f >= a.d) return;
  const int64_t row = a.hub_rows[h];
  const int64_t c_lo = a.hub_chunk_ptr[h], c_hi = a.hub_chunk_ptr[h + 1];
  // Chunk order.  A batch of requests is one round trip to memory, which is what bounds the launches on few rows of up to a hundred chunks:
  // 32 at a time; what is left eight at a time, the last ones of the last batch the last chunk's again.  54 and 107 blocks, rows of up to 98
  // chunks: eight at a time and the rest one by one 20.9 and 17.6 us, this way 12.4 and 10.1; 8.7 K blocks of shorter rows 22.7 and 19.5 (35 with
  // batches of 32 alone).
  float v = 0.f;
  int64_t c = c_lo;
  for (; c + 32 <= c_hi; c += 32) {
    float p[32];
#pragma unroll
    for (int u = 0; u < 32; ++u) p[u] = a.partial[(c + u) * a.d + f];
#pragma unroll
    for (int u = 0; u < 32; ++u) v += p[u];
  }
  for (; c < c_hi; c += 8) {
    float p[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) p[u] = a.partial[(c + u < c_hi ? c + u : c_hi - 1) * a.d + f];
#pragma unroll
    for (int u = 0; u < 8; ++u) v = c + u < c_hi ? v + p[u] : v;
  }
  finish_element<T>(a, row, f, v);
}

struct SpmmProf {
  int kind; int dtype; int64_t rows, nnz; double alg, touched, flops;
  int row_chunk = -1, row_chunk_n = 1;   // rows Schedule::chunk_row[row_chunk .. row_chunk + row_chunk_n); -1: all rows
  int64_t whole_nnz = 0, whole_rows = 0; // of the whole matrix, also for a range of its rows
  bool chunks_only = false;              // only the partial rows of long rows: another kernel adds them up
};

// Entries each lane group should get before a row is shared by more groups (GCN_SPMM_EPG overrides, for
// experiments).  Measured on an R-MAT graph with 45 entries per row: 4 / 8 / 16 / 32 / 64 entries per group
// give 460 / 441 / 431 / 427 / 427 us at width 128 and 122 / 113 / 108 / 107 / 110 us at width 16: a
// wavefront that holds more rows keeps more gathers in flight per round trip of its dependent loads.
constexpr int kEntriesPerGroup = 32;
constexpr int kFewestPerGroup = 4;
// A product is short of lane groups (a row has at least one) below this many wavefronts, two per SIMD.  Measured on uniform
// graphs, us with 4 / 8 / 16 / 32 entries per group: 60 K rows of 17 entries bf16 width 32 25 / 17 / 15 / 14, width 16 14 / 12 /
// 10 / 11; of 7 entries, bf16 width 32 13 / 11 / 9 / 9; 30 K rows of 19 entries fp32 width 16 10 / 8 / 8 / 8, width 64 23 / 22 /
// 19 / 17; on R-MAT ones of 20 K to 100 K rows within 3 %, but for width 128 of 100 K rows, 84 / 78 / 73 / 71.
constexpr int kFullWaves = 2048;

static inline int pow2_ceil_i(int x) { int p = 1; while (p < x) p <<= 1; return p; }

// The length classes of the ordinary rows: how many of a wavefront's g_max lane groups share a row of each, and the
// wavefronts they take.  Returns the number of classes, or -1; *blocks: some rows take a block each.
static inline int make_bins(SpmmK& k, const Schedule* sc, const SpmmProf& pf, int g_max, bool narrow, bool* blocks) {
  bool block_rows = false;
  // A product too small to fill the chip is bound by the chain of gathers of a row: its rows are shared by more groups.
  // (by the whole matrix: the sharing sets the order of a row's additions, which may not depend on how many launches the
  // product is made of)
  int epg = tune().spmm_epg > 0 ? tune().spmm_epg : kEntriesPerGroup;
  if (tune().spmm_epg <= 0)
    while (epg > kFewestPerGroup && std::max(pf.whole_rows, pf.whole_nnz / epg) * k.S < (int64_t)kFullWaves * g_max) epg >>= 1;
  // Rows whose gathers, one after the other in a wavefront, would take half as long as the whole product does: a block each.
  // A round of gathers (4 per group) takes about 0.6 us, the product its gathered bytes at 6 TB/s and a launch.  us without /
  // with: R-MAT 8 K rows of 20, width 128 48 / 18, 25 K of 5 69 / 24, bf16 25 K of 20 63 / 23; log-normal 8 K of 45, width 256
  // 113 / 40; 315 products of 2.5 K to 262 K rows and widths 7 to 256 0.84 in the geometric mean; uniform rows have none.
  const double whole_us = 5.0 + (double)pf.whole_nnz * k.d * (pf.dtype == GCN_BF16 ? 2 : 4) / 6e6;
  const int64_t block_from = std::max<int64_t>((int64_t)(4 * g_max * whole_us / (2 * 0.6)), std::max(epg, 16) * g_max);
  // bins of the ordinary rows: class c holds lengths in [2^(31-c), 2^(32-c)), class 32 empty rows
  int n_bins = 0;
  int64_t waves = 0;
  for (int c = 0; c <= 32; ++c) {
    const int64_t row_begin = pf.row_chunk < 0 ? sc->class_begin[c] : sc->chunk_class_begin[pf.row_chunk][c];
    const int64_t row_end = pf.row_chunk < 0 ? sc->class_begin[c + 1] : sc->chunk_class_begin[pf.row_chunk + pf.row_chunk_n][c];
    const int64_t cnt = row_end - row_begin;
    if (cnt <= 0 || pf.chunks_only) continue;
    if (n_bins == kMaxBins) return -1;
    const int64_t len_hi = c >= 32 ? 0 : ((int64_t)1 << (32 - c)) - 1;
    const int64_t want = ceil_div(len_hi > 0 ? len_hi : 1, epg);
    int groups = pow2_ceil_i((int)(want < g_max ? want : g_max));
    if (groups > g_max) groups = g_max;
    int lg = 0; while ((1 << lg) < groups) ++lg;
    const bool whole_block = narrow && (len_hi + 1) / 2 >= block_from;
    block_rows |= whole_block;
    if (whole_block) ++lg;               // (groups is g_max: block_from is a wavefront's share and more)
    const int b = n_bins++;
    k.bin_wave_begin[b] = waves;
    k.bin_row_begin[b] = row_begin;
    k.bin_row_end[b] = row_end;
    k.bin_log2gr[b] = lg;
    waves += whole_block ? 4 * cnt : ceil_div(cnt, g_max >> lg);
  }
  for (int b = n_bins; b < kMaxBins; ++b) { k.bin_wave_begin[b] = waves; k.bin_row_begin[b] = k.bin_row_end[b] = 0; k.bin_log2gr[b] = 0; }
  k.n_waves = waves;
  *blocks = block_rows;
  return n_bins;
}

template <typename T, int V, int LPR, int NV>
static int launch_l(SpmmK& k, const Schedule* sc, const SpmmProf& pf, bool narrow, hipStream_t s) {
  constexpr int G = 64 / LPR;
  bool own_blocks = false;
  if (make_bins(k, sc, pf, G, narrow, &own_blocks) < 0) return fail(GCN_EINVAL, "spmm: more length classes than expected");
  const int64_t waves = k.n_waves;
  const int64_t blocks = (k.n_chunks + ceil_div(waves, 4)) * k.S;
  if (!grid_fits(blocks)) return fail(GCN_EINVAL, "spmm: too many rows for one launch");
  if (blocks > 0) {
    ProfScope ps(pf.kind, s, k.d, pf.dtype, pf.rows, pf.nnz, pf.alg, pf.touched, pf.flops);
    if (own_blocks) k_spmm<T, V, LPR, NV, true, true><<<fold_grid(blocks), dim3(256), 0, s>>>(k);
    else if (narrow) k_spmm<T, V, LPR, NV, true, false><<<fold_grid(blocks), dim3(256), 0, s>>>(k);
    else k_spmm<T, V, LPR, NV, false, false><<<fold_grid(blocks), dim3(256), 0, s>>>(k);
  }
  if (k.n_hub_rows > 0 && !pf.chunks_only) {
    const double fb = 4.0 * (double)k.n_chunks * k.d + (double)sizeof(T) * (double)k.n_hub_rows * k.d;
    ProfScope ps(GCN_K_SPMM_FINISH, s, k.d, pf.dtype, k.n_hub_rows, k.n_chunks, fb, fb, (double)k.n_chunks * k.d);
    const int64_t fw = k.n_hub_rows * ceil_div(k.d, 64);
    k_spmm_hub_finish<T><<<fold_grid(ceil_div(fw, 4)), dim3(256), 0, s>>>(k);
  }
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

// Lanes per row and vectors per lane: one vector per lane and as many lanes as the row (or slice) has vectors, or, for
// short rows, groups of 8 lanes (one 128-byte line per group and request) with two vectors each.
template <typename T, int V>
static int launch_v(SpmmK& k, const Schedule* sc, const SpmmProf& pf, bool narrow, hipStream_t s) {
  if constexpr (sizeof(T) * V == 16) {
    if (k.short_rows) return launch_l<T, V, 8, 2>(k, sc, pf, narrow, s);
  }
  if constexpr (sizeof(T) == 2) {
    if (k.vps <= 1) return launch_l<T, V, 1, 1>(k, sc, pf, narrow, s);
  }
  if (k.vps <= 2) return launch_l<T, V, 2, 1>(k, sc, pf, narrow, s);
  if (k.vps <= 4) return launch_l<T, V, 4, 1>(k, sc, pf, narrow, s);
  if (k.vps <= 8) return launch_l<T, V, 8, 1>(k, sc, pf, narrow, s);
  if (k.vps <= 16) return launch_l<T, V, 16, 1>(k, sc, pf, narrow, s);
  if (k.vps <= 32) return launch_l<T, V, 32, 1>(k, sc, pf, narrow, s);
  return launch_l<T, V, 64, 1>(k, sc, pf, narrow, s);
}

// The kernel's arguments for product a (spmm.hip): everything but the length classes.  *V: elements per request, *narrow:
// 32-bit gather addresses.
int spmm_setup(const SpmmArgs& a, void* ws, SpmmK& k, SpmmProf& pf, int* V, bool* narrow);

// implemented in spmm_f32.hip / spmm_bf16.hip
int spmm_dispatch_f32(SpmmK& k, const Schedule* sc, const SpmmProf& pf, int V, bool narrow, hipStream_t s);
int spmm_dispatch_bf16(SpmmK& k, const Schedule* sc, const SpmmProf& pf, int V, bool narrow, hipStream_t s);

}  // namespace gcn
