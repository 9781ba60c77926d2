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
// (4 bits; 3 and 8 bits gain as much; of 1290 points beyond 704 tiles the worst was even.)  From 513 to 704 tiles what competes is
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

// Rows that a workgroup of the LayerNorm + quantize kernel for few rows takes (ln_rows.hip): 1, 2 or 4, never more than it has
// waves (a wave adds one row up).  A workgroup's time is a chain of waits, so one row each is fastest while the workgroups of a
// compute unit run side by side; then two and four, which share the per-position constants (12 bytes a code against the row's 2;
// eight measured no better).  What decides is the number of rows of a compute unit, `per`, and the waves that hold a row; a
// thread that holds two units, or sixteen codes with LayerNorm (3 bits), has so many constants that rows of its own cost most.
// Medians in us in a recorded graph, rows from memory, 4 bits (8 bits: the same lines), one | two | four rows:
//   waves, rows (per)             LayerNorm            without             3 bits: waves   LayerNorm             without
//   2   1280 x  768  (5)      4.39 | 4.95          3.58 | 3.74
//       1500 x  768  (6)      4.64 | 4.95          3.85 | 3.81
//       2560 x  768 (10)      5.67 | 5.61          4.38 | 4.25
//       2816 x  768 (11)      5.75 | 6.39          4.43 | 4.68
//   3   1280 x 1536  (5)      4.98 | 5.49          4.05 | 4.22              2       6.60 | 6.49          4.92 | 5.13
//       1792 x 1536  (7)      6.05 | 6.15          4.79 | 4.81              2       7.74 | 7.08          5.73 | 5.65
//   4   1500 x 2048  (6)      6.31 | 6.56 | 7.33   5.05 | 4.97 | 5.36       2       8.26 | 7.26          5.78 | 5.73
//       2816 x 2048 (11)      8.75 | 9.06 | 9.16   6.91 | 6.52 | 6.58
//   5   1200 x 2560  (5)      6.79 | 7.63 | 8.43   5.28 | 5.56 | 5.97       3       9.17 | 8.38          5.85 | 6.29
//       2000 x 2560  (8)      9.54 | 9.03 | 9.01   7.06 | 6.36 | 6.62       3      12.20 | 9.60          7.02 | 6.88
//   6    512 x 3000  (2)      4.87 | 5.01 | 6.15   3.93 | 3.98 | 4.51       3       5.83 | 5.49          4.22 | 4.40
//       1000 x 3000  (4)      6.73 | 7.22 | 7.08   5.10 | 5.21 | 5.26       3       8.73 | 7.41          5.57 | 5.81
//   8    512 x 4096  (2)      5.21 | 5.14 | 6.37   4.17 | 4.06 | 4.59       4       6.55 | 5.79 | 7.40   4.36 | 4.61 | 5.63
//       1000 x 4096  (4)      7.56 | 7.64 | 7.66   5.74 | 5.63 | 5.69       4      10.60 | 8.06 | 8.55   6.12 | 6.28 | 6.74
//       1500 x 4096  (6)     10.11 | 9.36 |10.07   7.31 | 6.53 | 7.31       4      13.95 | 9.98 |11.17   7.23 | 7.23 | 8.35
//       1750 x 4096  (7)     11.06 |10.71 |10.24   8.03 | 7.47 | 7.55       4      15.24 |11.62 |11.38   7.94 | 8.15 | 8.61
//   8 of two units
//        400 x 8192  (2)      8.47 | 7.44 | 9.59   6.16 | 6.18 | 7.66       8      10.74 | 8.26 |10.72   6.40 | 6.22 | 7.92
//        600 x 8192  (3)     10.57 |10.28 | 9.91   7.36 | 7.97 | 7.99       8      14.19 |11.60 |11.04   7.75 | 8.09 | 8.20
//  10    600 x 5120  (3)      8.55 | 8.88 | 8.43   6.14 | 6.18 | 5.87       5      10.46 | 9.71 | 9.42   6.44 | 7.07 | 7.10
//  12    500 x 6144  (2)      6.81 | 7.02 | 8.70   5.22 | 5.14 | 6.10       6       9.57 | 7.63 | 9.54   6.25 | 5.98 | 7.30
//  14    600 x 7168  (3)     10.60 |10.60 | 9.80   6.99 | 7.62 | 7.04       7      13.09 |11.11 |10.45   7.47 | 7.90 | 7.82
// (Rows of more than eight waves keep to two rows up to two per compute unit and four beyond, with LayerNorm those of two units or
// of more than four waves at 3 bits too: even with the best or some percent behind.  Against that simpler rule throughout, 3100
// points measured take 0.955 of the time, the worst 1.02.)
inline int ln_rows_per_workgroup(int64_t M, int waves, int units, int cus, int bits, bool ln) {
  struct Lines { int64_t one, two; };                         // one | two up to so many rows per compute unit; by waves, from two
  constexpr int64_t kAll = INT64_MAX;
  constexpr Lines kNorm[] = {{9, kAll}, {7, kAll}, {6, 11}, {5, 9}, {4, 7}, {4, 6}, {4, 6}};
  constexpr Lines kNorm3[] = {{4, kAll}, {1, kAll}, {1, 6}};
  constexpr Lines kPlain[] = {{5, kAll}, {5, kAll}, {5, 12}, {5, 12}, {3, 12}, {3, 12}, {3, 12}};
  constexpr Lines kPlain3[] = {{5, kAll}, {5, kAll}, {3, 12}, {5, 12}, {3, 12}, {3, 12}, {3, 12}};
  const int64_t per = (M + cus - 1) / cus;
  if (per <= 1 || waves == 1) return 1;
  if (waves > 8 || (ln && waves >= 4 && (units > 1 || (bits == 3 && waves > 4)))) return per <= 2 ? 2 : 4;
  if (!ln && per <= 2 && waves >= (bits == 3 ? 5 : 6)) return 2;
  if (ln && bits > 3 && waves == 2 && (per == 11 || per == 12)) return 1;      // (a sixth workgroup of two rows costs a round)
  const Lines& at = (ln ? (bits > 3 ? kNorm : kNorm3) : (bits > 3 ? kPlain : kPlain3))[waves - 2];
  return per <= at.one ? 1 : (per <= at.two ? 2 : 4);
}

}  // namespace rptq
