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
  if (!eight_rows_fit((int64_t)a.out_cols * a.d)) return false;   // (the launcher refuses them)
  int members;
  wh_tiles(a, nullptr, nullptr, &members);
  return (int64_t)members * a.rows * a.cols <= 10 * (int64_t)a.out_rows * a.out_cols;
}
int wh_items(const WhPassArgs& a) {
  int members;
  wh_tiles(a, nullptr, nullptr, &members);
  return (int)std::min<int64_t>((int64_t)a.seg_end[2] * a.T * (a.d / 64) * members, 0x3fffffff);
}
hipError_t launch_hw_inverse(const WhPassArgs* subs, int n, int num_cu, hipStream_t st) {
  for (int i = 0; i < n; ++i)
    if (subs[i].out_rows != subs[0].out_rows || subs[i].out_cols != subs[0].out_cols) return hipErrorInvalidValue;
  if (n > 1) {
    int kt, kh;
    wh_tiles(subs[0], &kt, &kh, nullptr);
    for (int i = 0; i < n; ++i)
      if (subs[i].cols != 16 && subs[i].cols != 32 && subs[i].cols != 64) return hipErrorInvalidValue;
    if (kt == 1 && kh == 1) return hw_mixed_launch<1, 1>(subs, n, num_cu, st);
    if (kt == 1 && kh == 2) return hw_mixed_launch<1, 2>(subs, n, num_cu, st);
    if (kt == 2 && kh == 1) return hw_mixed_launch<2, 1>(subs, n, num_cu, st);
    if (kt == 2 && kh == 2) return hw_mixed_launch<2, 2>(subs, n, num_cu, st);
    if (kh == 3) return hw_mixed_launch<1, 3>(subs, n, num_cu, st);
    if (kh == 4) return hw_mixed_launch<1, 4>(subs, n, num_cu, st);
    return hipErrorInvalidValue;
  }
  switch (subs[0].cols / 16) {
    case 1: return wh_dispatch<1, true>(subs, 1, num_cu, st, nullptr);
    case 2: return wh_dispatch<2, true>(subs, 1, num_cu, st, nullptr);
    case 3: return wh_dispatch<3, true>(subs, 1, num_cu, st, nullptr);
    case 4: return wh_dispatch<4, true>(subs, 1, num_cu, st, nullptr);
    case 5: return wh_dispatch<5, true>(subs, 1, num_cu, st, nullptr);
    case 6: return wh_dispatch<6, true>(subs, 1, num_cu, st, nullptr);
    case 7: return wh_dispatch<7, true>(subs, 1, num_cu, st, nullptr);
    case 8: return wh_dispatch<8, true>(subs, 1, num_cu, st, nullptr);
  }
  return hipErrorInvalidValue;
}
}  // namespace fa
