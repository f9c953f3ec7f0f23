// C = epilogue((A X) W) in one launch, for products whose time is launches and chains of dependent requests, gfx950.
//
// Sec. 4.1 writes the row task as the product with W^k of the aggregated row.  On some thousand rows the sparse product and the
// dense product that follows it move next to nothing: each takes 5 us, of which a chain of dependent requests (row, range,
// indices, features; operand, W) is most, and the launch between them costs the host as much again.  Here a workgroup of 16
// wavefronts adds up 16 sparse rows, one each, so that a row has all 64 lanes (of long rows 4 or 1, with 4 or 16 wavefronts
// each); W's operands are asked for meanwhile and stay in registers; the rows meet in LDS, and each wavefront multiplies them by
// 16 columns of W on the fp32 matrix pipe.  Both products, us as two kernels / as one (replayed graph): 2 K uniform rows of 5
// entries 64 -> 16 7.7 / 4.9, 100 -> 50 14.0 / 6.2, 128 -> 128 19.4 / 7.1; 4 K rows of 20 8.2 / 5.5, 15.8 / 7.5, 21.8 / 8.2.
//
// The dense half, per wavefront t and lane (c = l % 16, q = l / 16): W is the first operand of the 16x16x4 MFMAs, whose
// four k are 16 u + 4 q + i, so that a lane reads its part of a row from LDS with one request; register r of the result is row c,
// column 16 t + 4 q + r: the lanes of a row store 64 consecutive bytes.
//
// Rows of more than kHubRowNnz entries take a workgroup each.  Where there are many such entries, their chunks are added up by
// the sparse kernel in a launch before this one, and workgroups of this kernel add the partial rows in chunk order.
//
// The same on hundreds of thousands of rows gains nothing: whole row tiles of 64, gathers of some workgroups beside the matrix
// pipes of others, took 214 us on 500 K rows of 6.6 entries 50 -> 50 (the two kernels 217), 180 on R-MAT 2^18 16 -> 128 with
// the mask (158) and 556 on 128 -> 128 (508): what bounds both halves there is the fabric behind L2.
#include <algorithm>

#include "spmm_kernel.h"

namespace gcn {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kRows = 16;                  // sparse rows, and wavefronts, of a workgroup
constexpr int kMaxK = 128, kMaxN = 16 * kRows;
constexpr int kLds = kMaxK + 4;            // floats between two rows in LDS: rows c and lane parts q spread over all banks

struct DenseK {
  SpmmK s;
  const float* W; int64_t ldw; int trans;  // W is [K x N], or [N x K] where trans
  void* C; int64_t ldc; void* C2; int64_t ldc2;
  const float* bias; int relu; const void* mask; int64_t ldmask; int64_t mask_rows;
  int N;
  int vec;                                 // C, C2 and mask rows start on words: four columns at a time
  int store_s;                             // the sparse rows go to s.Y too
  // Blocks of hub rows come first, then those of ordinary rows, the longest before the others: rows [share_row[i],
  // share_row[i + 1]) of the schedule's list get 16, 4 and 1 wavefronts each, in blocks from share_block[i] on.
  int64_t share_row[4], share_block[3], hub_blocks, n_blocks;
  int hub_partials;                        // hub rows come as partial rows, kRows to a block; else one to a block
};
constexpr int kHubChunksDirect = 4;

template <typename T>
__device__ __forceinline__ void load4(const T* __restrict__ p, float (&v)[4]) {
  unpack_vec<T, 4>(*reinterpret_cast<const typename Vec<T, 4>::type*>(p), v);
}

// (up to 16 columns in fp32 the registers leave room for two workgroups a compute unit)
template <typename T, int V, int LPR>
__global__ __launch_bounds__(64 * kRows) __attribute__((amdgpu_waves_per_eu(V * LPR <= 16 ? 8 : 4, 8))) void k_spmm_dense(DenseK a) {
  constexpr int G = 64 / LPR;
  constexpr int kLog2G = G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : G == 8 ? 3 : 4;
  constexpr int kSteps = V * LPR / 16;
  __shared__ __align__(16) float S[kRows * kLds];
  __shared__ int32_t s_row[kRows];
  const int64_t blk = block_id();
  if (blk >= a.n_blocks) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, q = lane >> 4;
  const int d = a.s.d, steps = (d + 15) >> 4;
  const bool hubs = blk < a.hub_blocks, partials = hubs && a.hub_partials;

  // this wavefront's row, or its part of one, and the entries
  int64_t row = -1, s = 0; int n = 0, lw = 4;
  if (!partials) {
    if (hubs) {
      row = a.s.hub_rows[blk];
    } else {
      const int i = blk >= a.share_block[2] ? 2 : blk >= a.share_block[1] ? 1 : 0;
      lw = 4 - 2 * i;
      const int64_t ri = a.share_row[i] + (blk - a.share_block[i]) * (kRows >> lw) + (w >> lw);
      if (ri < a.share_row[i + 1]) row = a.s.wave_rows[ri];
    }
    if (row >= 0) {
      s = a.s.ptr[row];
      const int all = (int)(a.s.ptr[row + 1] - s), share = (all + (1 << lw) - 1) >> lw, first = (w & ((1 << lw) - 1)) * share;
      s += first;
      n = all - first < 0 ? 0 : all - first < share ? all - first : share;
    }
  }
  // W[16 u + 4 q + i][16 w + c], zero beyond K; a column beyond N is of no consequence
  float wv[kSteps][4];
  const bool busy = 16 * w < a.N;
  const int col = 16 * w + c < a.N ? 16 * w + c : a.N - 1;
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    if (!busy || u >= steps) continue;
    const int k0 = 16 * u + 4 * q;
    if (a.trans) {                         // (a request that would pass the end of a row of W ends with it)
      const int k_at = k0 + 4 <= d ? k0 : d - 4, shift = k0 - k_at;
      float x[4];
      load4<float>(a.W + (int64_t)col * a.ldw + k_at, x);
      if (shift & 1) { x[0] = x[1]; x[1] = x[2]; x[2] = x[3]; }
      if (shift & 2) { x[0] = x[2]; x[1] = x[3]; }
#pragma unroll
      for (int i = 0; i < 4; ++i) wv[u][i] = k0 + i < d ? x[i] : 0.f;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = a.W[(int64_t)(k0 + i < d ? k0 + i : d - 1) * a.ldw + col];
        wv[u][i] = k0 + i < d ? x : 0.f;
      }
    }
  }
  // columns K .. the next multiple of 16 of every row are zero
  for (int e = tid; e < kRows * (16 * steps - d); e += 64 * kRows) S[(e / (16 * steps - d)) * kLds + d + e % (16 * steps - d)] = 0.f;

  if (partials) {
    // ---- rows of many entries: their chunks' partial rows in chunk order
    const int64_t h0 = blk * kRows;
    const int rows = (int)(a.s.n_hub_rows - h0 < kRows ? a.s.n_hub_rows - h0 : kRows);
    if (tid < kRows) s_row[tid] = tid < rows ? a.s.hub_rows[h0 + tid] : -1;
    for (int e = tid; e < rows * d; e += 64 * kRows) {
      const int r = e / d, f = e - r * d;
      const int64_t c_lo = a.s.hub_chunk_ptr[h0 + r], c_hi = a.s.hub_chunk_ptr[h0 + r + 1];
      float v = 0.f;
      int64_t k = c_lo;
      for (; k + 8 <= c_hi; k += 8) {      // (eight requests in flight)
        float p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = a.s.partial[(k + u) * d + f];
#pragma unroll
        for (int u = 0; u < 8; ++u) v += p[u];
      }
      for (; k < c_hi; ++k) v += a.s.partial[k * d + f];
      S[r * kLds + f] = v;
      if (a.store_s) store_one<T>(reinterpret_cast<T*>(a.s.Y) + (int64_t)a.s.hub_rows[h0 + r] * a.s.ldy + f, v);
    }
  } else {
    const XBuf xb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(a.s.X), 0, (int)a.s.x_bytes, 0x00020000);
    const int g = lane / LPR, l = lane % LPR;
    // (the last vector of a row may be moved back to end with it)
    auto column = [&](int vi) -> int { return vi == a.s.nvec - 1 ? a.s.c_last : vi * V; };
    const int vi = l, c0 = column(vi < a.s.nvec ? vi : 0), skip = vi * V - c0;
    const uint32_t c0b[1] = {(uint32_t)c0 * (uint32_t)sizeof(T)};
    float acc[1][V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[0][v] = 0.f;
    team_accumulate<T, V, LPR, 1, true, kLog2G>(a.s, xb, a.s.idx + s, a.s.val + s, n, kLog2G, 0, g, lane, c0b, acc);
    reduce_groups<V, LPR, 1>(acc, G);
    if (lane == 0) {       // row r of the tile is that of wavefront r << lw
      if ((w & ((1 << lw) - 1)) == 0) s_row[w >> lw] = (int32_t)row;
      if (w >= (kRows >> lw)) s_row[w] = -1;
    }
    if (g == 0 && vi < a.s.nvec) {
      T* out = reinterpret_cast<T*>(a.s.Y) + row * a.s.ldy + c0;
      const bool keep = a.store_s && lw == 0 && row >= 0, whole = a.s.y_vec && (vi < a.s.nvec - 1 || a.s.y_full);
      if (keep && whole) store_vec<T, V>(out, acc[0]);
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if (v < skip || c0 + v >= d) continue;
        S[w * kLds + c0 + v] = acc[0][v];
        if (keep && !whole) store_one<T>(out + v, acc[0][v]);
      }
    }
    if (lw > 0) {          // the parts of a row, in order; a thread keeps to its column, and row r is not read again once it is written
      __syncthreads();
      auto quad = [&](int k) {
        const float* p = S + k * kLds + tid;
        return (p[0] + p[kLds]) + (p[2 * kLds] + p[3 * kLds]);
      };
      for (int r = 0; tid < d && r < (kRows >> lw); ++r) {
        const float v = lw == 2 ? quad(4 * r) : (quad(0) + quad(4)) + (quad(8) + quad(12));
        S[r * kLds + tid] = v;
        if (a.store_s && s_row[r] >= 0) store_one<T>(reinterpret_cast<T*>(a.s.Y) + (int64_t)s_row[r] * a.s.ldy + tid, v);
      }
    }
  }
  __syncthreads();
  if (!busy) return;

  // ---- 16 rows x K times K x 16
  floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    if (u >= steps) continue;
    const floatx4 sv = *reinterpret_cast<const floatx4*>(S + c * kLds + 16 * u + 4 * q);
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][i], sv[i], acc, 0, 0, 0);
  }
  const int64_t m = s_row[c];
  const int n0 = 16 * w + 4 * q;
  if (m < 0 || n0 >= a.N) return;
  T* __restrict__ C = reinterpret_cast<T*>(a.C) + m * a.ldc + n0;
  T* __restrict__ C2 = a.C2 ? reinterpret_cast<T*>(a.C2) + m * a.ldc2 + n0 : nullptr;
  const T* __restrict__ mk = a.mask && m < a.mask_rows ? reinterpret_cast<const T*>(a.mask) + m * a.ldmask + n0 : nullptr;
  const bool whole = a.vec && n0 + 4 <= a.N;
  float pre[4], v[4], keep[4] = {1.f, 1.f, 1.f, 1.f};
  if (mk && whole) load4<T>(mk, keep);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (mk && !whole && n0 + r < a.N) keep[r] = load_one<T>(mk + r);
    pre[r] = acc[r] + (a.bias && n0 + r < a.N ? a.bias[n0 + r] : 0.f);
    v[r] = a.relu ? (pre[r] > 0.f ? pre[r] : 0.f) : pre[r];
    v[r] = keep[r] > 0.f ? v[r] : 0.f;
  }
  if (whole) {
    if (C2) store_vec<T, 4>(C2, pre);
    store_vec<T, 4>(C, v);
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (n0 + r >= a.N) continue;
      if (C2) store_one<T>(C2 + r, pre[r]);
      store_one<T>(C + r, v[r]);
    }
  }
}

// Lanes per row of nvec vectors, and workgroups that run at once.
int lanes_of(int nvec, int dtype) { return nvec <= 4 ? 4 : nvec <= 8 ? 8 : nvec <= 16 || dtype == GCN_BF16 ? 16 : 32; }
int64_t slots_of(int lanes, int dtype) { return (dtype == GCN_BF16 ? 8 : 4) * lanes <= 16 ? 512 : 256; }

// Workgroups for the rows of a schedule, in the order of their numbers: hub rows, then ordinary ones, the longest first.
struct Shares {
  int64_t row[4], block[3], hub_blocks, n_blocks, slots;
  bool hub_partials;
  int chain;                               // rounds of gathers of the longest ordinary row (by its class), one after the other
};

// Wavefronts per row by its length class: a lane group gathers 4 entries at a time, each round about 0.6 us, so a row of 4 or
// more rounds gets 4 wavefronts and one of 16 or more 16, as long as all workgroups still run at once; else these numbers
// are 8 and 32, or 16 and 64.  (From 8 and 32 on whatever the workgroups, 4 K uniform rows of up to 72 entries 128 -> 128 take 15.6
// instead of 9.9 us: a workgroup more than run at once is a round more.  1296 products of 1 K to 8 K R-MAT and log-normal rows,
// one kernel over two in the geometric mean: 16 and 64 throughout 0.85, this way 0.78.)
//
// A hub row that has a workgroup to itself is 16 chains of up to 256 entries, as long as those of its chunks in the sparse kernel (and
// as exact), if it has no more than kHubChunksDirect of them, which the sums over all hub rows decide: each has three chunks at least.
// Where a wavefront has two lane groups (fp32, more than 64 columns) the chunks are faster.  Measured, two kernels / a workgroup a
// hub row / chunks: one row of 60 K entries 128 -> 128 35 / 275 / 29 us, error against 64 bits 2.0e-7 / 8.3e-7 / 2.0e-7; one of 4 K
// 16 -> 16 8.9 / 7.1 / 9.1, 128 -> 128 26 / 25 / 17.
Shares shares_of(const Schedule* sc, int lanes, int dtype) {
  Shares o{};
  const int g = 64 / lanes;
  // first row of the list that is shorter than len, a power of two
  auto begin = [&](int64_t len) { return sc->class_begin[32 - __builtin_ctzll((unsigned long long)len)]; };
  o.slots = slots_of(lanes, dtype);
  o.hub_partials = sc->n_hub_rows > 0 && (lanes > 16 || sc->n_chunks - 3 * (sc->n_hub_rows - 1) > kHubChunksDirect);
  o.hub_blocks = o.hub_partials ? ceil_div(sc->n_hub_rows, kRows) : sc->n_hub_rows;
  const int64_t fit = round_up(ceil_div(sc->n_wave_rows + sc->n_hub_rows, kRows), o.slots);
  for (int rounds = 4; rounds <= 16; rounds *= 2) {
    o.row[0] = 0; o.row[1] = begin(16 * rounds * g); o.row[2] = begin(4 * rounds * g); o.row[3] = sc->n_wave_rows;
    o.n_blocks = o.hub_blocks;
    for (int i = 0; i < 3; ++i) {
      o.block[i] = o.n_blocks;
      o.n_blocks += ceil_div(o.row[i + 1] - o.row[i], i == 0 ? 1 : i == 1 ? 4 : kRows);
    }
    if (o.n_blocks <= fit) break;
  }
  int c = 0;
  for (int i = 0; i < 3; ++i) {            // the longest row of each share is in the class of its first row
    if (o.row[i + 1] <= o.row[i]) continue;
    while (sc->class_begin[c + 1] <= o.row[i]) ++c;
    const int64_t len = c >= 32 ? 0 : (int64_t)1 << (31 - c);
    o.chain = std::max(o.chain, (int)(len / ((i == 0 ? 16 : i == 1 ? 4 : 1) * 4 * g)));
  }
  return o;
}

template <typename T, int V, int LPR>
int launch_k(DenseK& k, const SpmmProf& pf, hipStream_t s) {
  if (!grid_fits(k.n_blocks)) return fail(GCN_EINVAL, "spmm: too many rows for one launch");
  ProfScope ps(pf.kind, s, k.s.d, pf.dtype, pf.rows, pf.nnz, pf.alg, pf.touched, pf.flops);
  k_spmm_dense<T, V, LPR><<<fold_grid(k.n_blocks), dim3(64 * kRows), 0, s>>>(k);
  GCN_CHECK_LAUNCH();
  return GCN_OK;
}

}  // namespace

// Operands that the kernel takes: fp32 or bf16 rows gathered 16 bytes at a time with 32-bit addresses, 4 to kMaxK columns, 4 to
// kMaxN columns behind W.
bool spmm_dense_ok(const SpmmArgs& a, int N) {
  if (a.part != 0 || a.row_chunk >= 0 || a.no_alloc || a.n_rows == 0) return false;
  if (a.d < 4 || a.d > kMaxK || N < 4 || N > kMaxN) return false;
  SpmmK k{};
  SpmmProf pf;
  int V = 1;
  bool narrow = false;
  if (spmm_setup(a, nullptr, k, pf, &V, &narrow) != GCN_OK) return false;
  return narrow && V * (a.dtype == GCN_BF16 ? 2 : 4) == 16;
}

// Is it faster than the two kernels?  Not where long rows are many, so that the rows are shared by more workgroups than run at
// once, each with W to read: 4096 rows of 1000 entries 128 -> 256 184 us against 77, 2048 of 300 64 -> 64 18.3 / 14.7, 8192 of 128 128 ->
// 128 62 / 42, while less than twice that number gains (R-MAT 4 K rows of 45 128 -> 256 19.4 / 29.3); with more than 4 K rows, which
// are two rounds anyway, up to half more, and an eighth for more than 128 columns (8 K R-MAT rows of 45 128 -> 256 46 / 38).  Nor where
// a long row's chain of gathers outlasts the little that there is to save: narrow products (64 -> 16 on log-normal rows of 45 13.2 /
// 10.4, 16 -> 16 on R-MAT 12.1 / 10.6), and products whose rows are gathered `widened`, wider than the two kernels would (bf16 50 -> 7 on
// R-MAT rows of 20 17.8 / 11.1, 128 -> 32 on log-normal ones of 128 14.1 / 12.0; 100 -> 50 with a hub row 30.6 / 25.0).
// Over 7020 products (1 K to 8 K uniform, R-MAT and log-normal rows of 4 to 128 entries, 14 pairs of widths, both directions and types)
// 0.81 in the geometric mean, under 1 % of them slower by 3 % or more (at most 1.15); with the kernel wherever it applies 4 %, up to 1.8.
bool spmm_dense_pays(const SpmmArgs& a, int N, bool widened) {
  const bool bf16 = a.dtype == GCN_BF16;
  const Shares h = shares_of(a.sched, lanes_of((int)ceil_div(a.d, bf16 ? 8 : 4), a.dtype), a.dtype);
  const int64_t at_once = round_up(ceil_div(a.n_rows, kRows), h.slots);
  if (h.n_blocks > (a.n_rows <= 4096 ? 2 * at_once - 1 : N <= 128 ? at_once + at_once / 2 : at_once + at_once / 8)) return false;
  if (widened && a.sched->n_hub_rows > 0) return false;
  const int kn = a.d * N;
  if (h.chain >= 8 && kn < (bf16 && widened ? 4097 : 2048)) return false;
  return !(bf16 && widened && a.d > 32 && kn < 1024 && h.chain >= 1);
}

int spmm_dense(const SpmmArgs& a, void* ws, const float* W, int64_t ldw, void* C, int64_t ldc, int N, const GemmEpilogue& epi,
               hipStream_t s) {
  DenseK k{};
  SpmmProf pf;
  int V = 1;
  bool narrow = false;
  GCN_TRY(spmm_setup(a, ws, k.s, pf, &V, &narrow));
  const int64_t es = a.dtype == GCN_BF16 ? 2 : 4;
  const int lanes = lanes_of(k.s.nvec, a.dtype);
  const Shares h = shares_of(a.sched, lanes, a.dtype);
  std::copy(h.row, h.row + 4, k.share_row);
  std::copy(h.block, h.block + 3, k.share_block);
  k.hub_blocks = h.hub_blocks; k.n_blocks = h.n_blocks; k.hub_partials = h.hub_partials;
  if (k.hub_partials) {
    SpmmK chunks = k.s;
    SpmmProf cp = pf;
    cp.chunks_only = true;
    cp.kind = GCN_K_SPMM_FINISH;
    cp.alg = cp.touched = 4.0 * (double)a.sched->n_chunks * a.d;
    GCN_TRY(a.dtype == GCN_BF16 ? spmm_dispatch_bf16(chunks, a.sched, cp, V, narrow, s) : spmm_dispatch_f32(chunks, a.sched, cp, V, narrow, s));
  }
  k.s.S = 1; k.s.vps = k.s.nvec;
  k.W = W; k.ldw = ldw; k.trans = epi.b_trans ? 1 : 0;
  k.C = C; k.ldc = ldc; k.C2 = epi.C2; k.ldc2 = epi.ldc2;
  k.bias = epi.bias; k.relu = epi.relu; k.mask = epi.mask; k.ldmask = epi.ldmask; k.mask_rows = epi.mask_rows;
  k.N = N;
  auto words = [&](const void* p, int64_t ld) { return p == nullptr || (((uintptr_t)p % 4) == 0 && (ld * es) % 4 == 0); };
  k.vec = words(C, ldc) && words(epi.C2, epi.ldc2) && words(epi.mask, epi.ldmask);
  k.store_s = a.Y != nullptr;
  const double extra = (double)es * (double)a.n_rows * N * (1.0 + (epi.C2 ? 1.0 : 0.0) + (epi.mask ? 1.0 : 0.0)) + 4.0 * (double)a.d * N -
                       (k.store_s ? 0.0 : (double)es * (double)a.n_rows * a.d);
  pf.alg += extra; pf.touched += extra; pf.flops += 2.0 * (double)a.n_rows * a.d * N;
  if (a.dtype == GCN_BF16) {
    if (lanes == 4) return launch_k<bf16_t, 8, 4>(k, pf, s);
    if (lanes == 8) return launch_k<bf16_t, 8, 8>(k, pf, s);
    return launch_k<bf16_t, 8, 16>(k, pf, s);
  }
  if (lanes == 4) return launch_k<float, 4, 4>(k, pf, s);
  if (lanes == 8) return launch_k<float, 4, 8>(k, pf, s);
  if (lanes == 16) return launch_k<float, 4, 16>(k, pf, s);
  return launch_k<float, 4, 32>(k, pf, s);
}

}  // namespace gcn
