// Rules that choose a launch's form from its sizes alone: plain C++, so that they can be checked where there is no GPU.
#pragma once
#include <stdint.h>

namespace rptq {

// Columns of 64 x 256 tiles at a product's end that go out as 64 x 128 tiles, two for one, in the launch of the others; 0: none.
// Tiles beyond a whole number per compute unit (256 of them) leave most of the chip idle at the end.  The tile columns that hold
// them are cut in two where they are 128 tiles at most (so only with up to 128 row tiles, 8192 rows): one small tile per compute
// unit.  More of them come to two on some: 192 in these columns 88 | 101 us, 205 101 | 115 at K = 5120.
// Medians in us, large tiles alone | with the small ones behind them, by rows x columns (tiles, of these in the cut columns):
//                                K = 768        2048           5120           12288
//   Y     2048 x  8704 (1088,  64)  33 |  30     56 |  51      114 | 103      212 | 195
//         2100 x  8000 (1056,  33)  31 |  30     56 |  53      112 | 105      218 | 198
//         2900 x  4099 ( 782,  46)  33 |  32     50 |  47       90 |  81      175 | 157
//         8192 x  3328 (1664, 128)  43 |  40     74 |  71      163 | 151      304 | 285
//         4096 x 20992 (5248, 128) 115 | 114    231 | 224      480 | 465      917 | 898
//   next site's codes
//         2048 x  8704              41 |  38     64 |  59      118 | 108      220 | 203
//   a pair per cluster
//         2048 x  8704              47 |  43     78 |  70      146 | 130      240 | 221
// (4 bits; 3 and 8 bits gain as much; of 1000 points beyond 704 tiles the worst was even.)  From 513 to 704 tiles what competes is
// 64 x 128 tiles throughout, and these are ahead but for 8-bit codes over a long K: 64 x 128 tiles | with the small ones behind:
//                                   K = 768        2048         5120          12288
//   Y     2048 x 4608 (576, 64)    20.0 | 21.0  31.4 | 32.6  59.7 | 60.5  119.5 | 118.3
//         2100 x 4500 (594, 99)    27.4 | 27.2  38.7 | 40.7  69.4 | 73.4  127.9 | 133.8
//         3072 x 3072 (576, 96)    18.8 | 19.9  31.9 | 33.0  61.4 | 62.6  118.7 | 120.1
//   next site's codes, 2048 x 4608 25.6 | 26.2  37.9 | 39.5  65.8 | 67.6  125.3 | 123.9
//   a pair per cluster, the same   25.8 | 27.5  40.3 | 44.2  72.3 | 79.1
//   Y, 8 bits: 0.95 to 1.07 times as long up to K = 4096, 0.96 to 1.00 at 5120 and 6144, 0.85 to 0.97 at 12288
inline int gemm_tail_columns(int64_t M, int64_t N, int slices, int bits, bool pair_per_cluster) {
  constexpr int64_t kUnits = 256, kOneSmallRound = 704;
  const int64_t rows = (M + 63) / 64, tiles = rows * ((N + 255) / 256), over = tiles % kUnits;
  const bool long_k = bits == 8 && slices >= 160 && !pair_per_cluster;
  if (tiles <= (long_k ? 2 * kUnits : kOneSmallRound) || over == 0) return 0;
  const int64_t cols = (over + rows - 1) / rows;
  return 2 * cols * rows <= kUnits ? static_cast<int>(cols) : 0;
}

}  // namespace rptq
