// Requests to a few rows of a matrix that a range check ends, for the streaming dense kernels (gfx950).
#pragma once
#include "common.h"

namespace gcn {

// A buffer of 16 rows, `left` of them backed: requests past its end are dropped (stores) or answered with zeros (loads) by the
// range check, without a branch.  (0x00020000: a plain buffer of 32-bit words)
typedef __amdgpu_buffer_rsrc_t RowsBuf;
constexpr uint32_t kNoPlace = 0xfffffff0u;
template <typename T>
__device__ __forceinline__ RowsBuf rows_buf(const void* p, int64_t row0, int64_t ld, int left) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(p) + row0 * ld * (int64_t)sizeof(T)), 0,
                                           left * (int)ld * (int)sizeof(T), 0x00020000);
}

// Columns [col, end) of `left` rows from row0 on: their first element and the bytes from there to the end of the last row's, of which no
// request may pass.  (Rows of the full pitch from `col` on would end `col` elements behind the matrix.)
struct RowsRange { int64_t first; int bytes; };
__host__ __device__ constexpr RowsRange rows_range(int64_t row0, int64_t ld, int left, int col, int end, int size) {
  return RowsRange{row0 * ld + col, left > 0 && end > col ? ((left - 1) * (int)ld + end - col) * size : 0};
}
template <typename T>
__device__ __forceinline__ RowsBuf rows_part(const void* p, int64_t row0, int64_t ld, int left, int col, int end) {
  const RowsRange r = rows_range(row0, ld, left, col, end, (int)sizeof(T));
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(p) + r.first * (int64_t)sizeof(T)), 0, r.bytes, 0x00020000);
}

}  // namespace gcn
