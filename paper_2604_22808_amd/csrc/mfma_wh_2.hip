// H + W pass of the inverse transform (see mfma_wh_impl.h).
#include "mfma_wh_impl.h"
namespace fa {
// A plane's coefficients are read by each of its workgroups.  As long as that is not more than ten times the output the pass is
// faster than two; inverse transforms, two passes / one, us: 4 times (8 slices of 16 x 128 x 128 x 128 from the 64 x 64 box) 441 / 387,
// 7 (8 of 32 x 64 x 112 x 128 whole) 611 / 482, 8 (32 x 128 x 64) 641 / 590, 10 (32 x 80 x 80) 497 / 491, 12 (32 x 96 x 96) 700 / 788,
// 16 (16 x 128 x 128) 697 / 890.
bool hw_fits(const WhPassArgs& a) {
  if (a.rows % 16 || a.cols % 16 || a.out_rows % 16 || a.out_cols % 16 || a.rows > 128 || a.cols > 128 || a.out_rows > 128 || a.out_cols > 128 || a.d % 64)
    return false;
  int members;
  wh_tiles(a, nullptr, nullptr, &members);
  return (int64_t)members * a.rows * a.cols <= 10 * (int64_t)a.out_rows * a.out_cols;
}
hipError_t launch_hw_inverse(const WhPassArgs& a, int num_cu, hipStream_t st) {
  switch (a.cols / 16) {
    case 1: return wh_dispatch<1, true>(a, num_cu, st, nullptr);
    case 2: return wh_dispatch<2, true>(a, num_cu, st, nullptr);
    case 3: return wh_dispatch<3, true>(a, num_cu, st, nullptr);
    case 4: return wh_dispatch<4, true>(a, num_cu, st, nullptr);
    case 5: return wh_dispatch<5, true>(a, num_cu, st, nullptr);
    case 6: return wh_dispatch<6, true>(a, num_cu, st, nullptr);
    case 7: return wh_dispatch<7, true>(a, num_cu, st, nullptr);
    case 8: return wh_dispatch<8, true>(a, num_cu, st, nullptr);
  }
  return hipErrorInvalidValue;
}
}  // namespace fa
