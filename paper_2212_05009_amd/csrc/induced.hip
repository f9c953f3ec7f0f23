// gcn_csr_induced: the normalised adjacency of the subgraph induced by a vertex list, built on the
// device from a whole-graph handle (Sec. 4.3.3: a mini-batch is a subgraph G' = (V', E') of the input
// graph, and convolutions run on it as they do on the whole graph in full-batch training).
//
// The subgraph is a graph of its own: vertex k is vertices[k], its edges are the stored entries
// (vertices[a], vertices[b]) of the parent, and degrees, self-loops and D^-1/2 (A'+I) D^-1/2 are
// those of the subgraph.  The entries of the selected rows whose columns are selected too become
// (row, column) keys in subgraph numbering, one pass over those rows, and the keys go through the
// builder's second half, so sorting, normalisation and the column-major copy are the builder's.
#include <new>

#include "common.h"

namespace gcn {

constexpr int kIndThreads = 256;
static inline dim3 ind_grid(int64_t n) { return fold_grid(ceil_div(n > 0 ? n : 1, kIndThreads)); }

// lid[v] = -1 for every vertex of the parent; the flags and the number of keys (the diagonals come first)
__global__ void k_ind_init(int32_t* __restrict__ lid, int64_t n, int64_t n_sub, int* __restrict__ bad, int64_t* __restrict__ cursor) {
  int64_t i = block_id() * blockDim.x + threadIdx.x;
  if (i < n) lid[i] = -1;
  if (i == 0) { bad[0] = bad[1] = 0; *cursor = n_sub; }
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

static int induced_impl(const gcn_csr_t* A, const int32_t* d_vertices, int64_t n_sub, int flags, hipStream_t s, gcn_csr* B) {
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
  k_ind_init<<<ind_grid(n), kIndThreads, 0, s>>>(lid.as<int32_t>(), n, n_sub, bad, cursor);
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
  const int rc = induced_impl(A, d_vertices, n_sub, flags, (hipStream_t)stream, B);
  if (rc != GCN_OK) { gcn_csr_free(B); return rc; }
  *out = B;
  return GCN_OK;
}
