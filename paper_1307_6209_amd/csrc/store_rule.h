// How permuted rows of y are stored. No HIP, so that it can be checked on its own.
#pragma once

#include <cstddef>
#include <cstdint>

namespace sell {

// Permuted rows of y are stored one by one, several to a line. Through the L2, which
// gathers a line's rows: where the product is a short one, whose end waits for
// streaming stores, where x is so small that nothing turns it out, and on
// padding-heavy layouts, whose gathers leave room in the L2. Else they turn x out of it
// and are streamed past it. us, through the L2 / streamed (matrix; FP64, FP32, BF16 /
// FP64 unless named):
//   50,000 rows of up to 48, sigma 1024, C = 16                 13.3 / 14.9, 12.3 / 13.2, 10.2 / 12.8
//   100,000 of up to 24, sigma n, C = 32                        7.7 / 9.0, 7.6 / 8.7, 7.5 / 8.4
//   200,003 of up to 12, sigma n, C = 32 (15, 10, 7 MB)         8.2 / 9.6, 7.5 / 8.9, 7.7 / 8.5
//   120,000 of up to 40, sigma 1024, C = 8 (28, 19, 14 MB)      28.6 / 29.5, 24.9 / 27.4, 22.1 / 27.1
//   93,714 x 2,580 of up to 51, sigma 256, C = 32, 64           11.2 / 11.9, 13.2 / 14.4 in FP64
//   200,003 x 20,000 of up to 48, sigma 1024, C = 8             50.6 / 52.0, 39.9 / 43.1, 40.5 / 44.0
//   200,003 of up to 48, sigma 1024, C = 16 (57, 38, 29 MB)     50.4 / 49.3, 47.4 / 45.4, 48.3 / 45.6
//   power-law 500k, sigma n, C = 16, BF16 / FP64 (13 MB)        19.6 / 18.5
//   power-law 500k, sigma 1024 (beta 0.14), C = 32              27.8 / 28.4, 21.6 / 22.1, 23.3 / 22.9
//   power-law 1M, sigma 1024, C = 32, FP32 (y of 4 MB)          40.2 / 41.2
//   64 power-law matrices of up to 200,000 rows, sigma n        106 / 111
//   power-law 2M, sigma 2^14 (y of 16 MB)                       121 / 119
inline bool keeps_y(int64_t nrows, size_t ysize, int64_t ncols, size_t xsize, int64_t padded, size_t vsize,
                    double beta) {
  constexpr size_t kMiB = 1 << 20;
  const size_t y = (size_t)nrows * ysize, x = (size_t)ncols * xsize, matrix = (size_t)padded * (vsize + 4);
  if (beta < 0.5) return y <= 8 * kMiB;
  if (y > 2 * kMiB) return false;
  return x <= kMiB / 4 || matrix <= (y <= kMiB ? 32 : 16) * kMiB;
}

}  // namespace sell
