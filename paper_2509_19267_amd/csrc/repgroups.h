// When the many-right-hand-side products take row groups (rep.hip).  Plain
// C++, so that a CPU test can check it.
#pragma once
#include <stdint.h>

namespace rg {

// A quarter as many waves, each with the work of four, so the product must be
// bound by its gathers and not by a wave's latency: so many gathers of 64
// values for each compute unit, in FP32 more than twice as many as in FP64.
// Measured over 100 to 25600 rows, 33 to 256 right-hand sides, stencils of 9 to
// 225 entries, A x and A^T z with their transposes, row by row / in groups, 64
// right-hand sides, us.  FP64: 225 entries 1600 rows (1410 a unit) 91 / 91, 3136
// 109 / 97; 81 entries 3136 rows (910) 78 / 79, 6400 106 / 95; 25 entries 6400
// rows (600) 79 / 83, 12544 (1200) 96 / 91.  FP32: 225 entries 3136 rows (2760)
// 84 / 88, 6400 108 / 99; 81 entries 6400 rows (2020) 78 / 82, 12544 100 / 94.
// And the groups keep a copy of the entries for each order and precision:
// bounded, so that a matrix that fits the card without them still does.
constexpr int64_t RG_GATHERS_F64 = 1100, RG_GATHERS_F32 = 2800;
constexpr int64_t REP_RG_BYTES = 48ll << 30;
constexpr bool rep_rg_fits(int64_t rep, int64_t nnz, int ncu, bool f64) {
  return nnz * ((rep + 63) / 64) >=
             (f64 ? RG_GATHERS_F64 : RG_GATHERS_F32) * ncu &&
         nnz <= REP_RG_BYTES / 32;   // 2 orders, 4 + 8 + 4 bytes an entry
}
// And where the groups gather at most REP_RG_SHARE of the stored entries'
// columns: 0.30 and 0.33 above; at 0.40 (25 entries) 25600 rows 118 / 113 and
// 96 / 96, 128 right-hand sides 163 / 149 and 132 / 120; at 0.50 (9 entries)
// 25600 rows 97 / 100 and 88 / 91, 128 right-hand sides 122 / 125 and 107 / 106.
constexpr double REP_RG_SHARE = 0.45;
constexpr bool rep_rg_pays(int64_t cols, int64_t nnz) {
  return (double)cols <= REP_RG_SHARE * (double)nnz;
}

}  // namespace rg
