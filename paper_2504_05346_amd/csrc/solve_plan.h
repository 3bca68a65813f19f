// Rows and workgroups of the row solver for up to 64 unknowns (k_solve_mfma<2>).  Plain C++: the host tests compile it
// by itself.
#pragma once
#include <cstdint>

namespace thanos {

// Rows that run at once on 256 compute units: eight per unit of up to 96 unknowns; of up to 64, sixteen in workgroups of
// four and twenty in workgroups of five (8 KB of LDS per row; workgroups of four take the same times with room for
// four of them per unit as with room for five).
constexpr int64_t kRowsOf96 = 8 * 256, kRowsOf64 = 16 * 256, kRowsOf64By5 = 20 * 256;

// Five rows to a workgroup where that lets all of them run at once.  With more rows the last round of them is the larger
// for it.  Sweeps of 1024 columns with workgroups of four and of five, us: 1:4 with a given factor 4608 rows 266 and 262,
// 5120 268 and 263, 5376 289 and 301, 8192 345 and 380, 16384 577 and 604; whole calls at 50 % 4608 rows 904 and 886,
// 5120 908 and 882, 5632 959 and 968, 8192 1060 and 1108, 12288 1317 and 1348.  Not for 64 unknowns in each of the
// rows (all_full), where the elimination fills the matrix cores of a unit with sixteen: 2:4 with a given factor 4097 rows 364
// and 369, 5120 371 and 373, 8192 504 and 568, 16384 904 and 987.  With outlier rows, which end at once, again: 5120 x 5120 4:8,
// every tenth, 4420 and 4390.
constexpr int solve_rows_per_group(int64_t c, bool all_full) {
  return !all_full && c > kRowsOf64 && c <= kRowsOf64By5 ? 5 : 4;
}

}  // namespace thanos
