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

}  // namespace gcn
