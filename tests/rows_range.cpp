// Host-side check of the ranges that end the requests of the streaming dense kernels (rows_buf.h): for every number of columns, panel of them, rows
// and pitch of a grid the last byte that can pass lies inside the matrix, and every element of the panel can be reached.
//   rows_range       exit 0: holds, 1: does not (with a line that says where)
#include <stdio.h>

#include "rows_buf.h"

int main() {
  long checked = 0;
  for (int n = 1; n <= 1100; n += n < 70 ? 1 : 7)
    for (int panel = 64; panel <= 256; panel += 64)
      for (int64_t ld = n; ld <= n + 20; ld += 5)
        for (int left = -1; left <= 16; ++left)
          for (int n0 = 0; n0 < n; n0 += panel) {
            const int64_t row0 = 48;
            const gcn::RowsRange r = gcn::rows_range(row0, ld, left, n0, n, 4);
            const int64_t matrix = left > 0 ? ((row0 + left - 1) * ld + n) * 4 : 0;      // bytes up to the end of the last row
            const bool ends = left <= 0 ? r.bytes == 0 : r.first * 4 + r.bytes <= matrix;
            // the last column of the panel in the last row, by its place in the range
            const int last = (n < n0 + panel ? n : n0 + panel) - 1 - n0;
            const bool reaches = left <= 0 || (r.first == row0 * ld + n0 && ((left - 1) * ld + last + 1) * 4 <= r.bytes);
            if (!ends || !reaches) {
              printf("n %d panel %d ld %lld rows %d from column %d: first %lld bytes %d\n", n, panel, (long long)ld, left, n0, (long long)r.first, r.bytes);
              return 1;
            }
            ++checked;
          }
  printf("%ld ranges hold\n", checked);
  return checked > 0 ? 0 : 1;
}
