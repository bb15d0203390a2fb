// Two W + H passes of the forward transform in one launch (see k_wh_two in mfma_wh_impl.h).
#include "mfma_wh_impl.h"
namespace fa {
bool wh_two_fits(const WhPassArgs& a, const WhPassArgs& b, int num_cu) {
  int kt_a, kh_a, kt_b, kh_b;
  wh_tiles(a, &kt_a, &kh_a, nullptr);
  wh_tiles(b, &kt_b, &kh_b, nullptr);
  // Up to 16 rounds together, where the last rounds of two launches count: 64K tokens, 22 + 2 heads of 64 (routed, 6 rounds) 580 / 556 us per
  // forward apart / together.  Beyond it is worth up to 1.4 %, apart / together: 64 heads of 16 x 64 x 64 x 64, a quarter high (17 rounds) 1508 / 1490, 96
  // (26) 2206 / 2180, 160 (43) 3592 / 3551; 18 of 64^3 x 64 (20) 1888 / 1864; 48 of 32 x 48 x 80 x 128 (75) 4112 / 4115, 96 of 16 x 64 x 64 x 128 (51) 4071 / 4066.
  if ((int64_t)wh_items(a) + wh_items(b) > 16 * (int64_t)num_cu) return false;
  return a.cols == b.cols && a.T == b.T && a.d == b.d && kt_a == 2 && kh_a == 2 && kt_b == 1 && kh_b >= 3 && wh_items(a) >= num_cu && wh_items(b) >= num_cu;
}
hipError_t launch_wh_two(const WhPassArgs& a, const WhPassArgs& b, int num_cu, hipStream_t st, int slots_out[2]) {
#define FA_TWO_CASE(NW_) \
  if (a.cols == 16 * NW_) return b.out_rows > 48 ? wh_two_launch<NW_, 4>(a, b, num_cu, st, slots_out) : wh_two_launch<NW_, 3>(a, b, num_cu, st, slots_out);
  if (!wh_two_fits(a, b, num_cu)) return hipErrorInvalidValue;
  FA_TWO_CASE(2) FA_TWO_CASE(3) FA_TWO_CASE(4) FA_TWO_CASE(5) FA_TWO_CASE(6) FA_TWO_CASE(7) FA_TWO_CASE(8)
#undef FA_TWO_CASE
  return hipErrorInvalidValue;
}
}  // namespace fa
