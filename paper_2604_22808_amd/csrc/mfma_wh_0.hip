// W + H pass of the forward transform, W = 16 .. 64 (see mfma_wh_impl.h).
#include "mfma_wh_impl.h"
namespace fa {
bool wh_fits(int T, int d, int H, int W, int kh, int kw) {
  if (H % 16 != 0 || W % 16 != 0 || H > 128 || W > 128 || kh % 16 != 0 || kw % 16 != 0) return false;
  // (More than 64 H coefficients do not fit the accumulators of one workgroup; cutting them into parts, as the inverse does, was
  // not measured in this direction.  The launcher refuses rows that lie too far apart.)
  return kh <= 64 && d % 64 == 0 && eight_rows_fit((int64_t)T * kw * d);
}
hipError_t launch_wh_pass_0(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out) {
  switch (subs[0].cols / 16) {
    case 1: return wh_dispatch<1, false>(subs, n, num_cu, st, slots_out);
    case 2: return wh_dispatch<2, false>(subs, n, num_cu, st, slots_out);
    case 3: return wh_dispatch<3, false>(subs, n, num_cu, st, slots_out);
    case 4: return wh_dispatch<4, false>(subs, n, num_cu, st, slots_out);
  }
  return hipErrorInvalidValue;
}
}  // namespace fa
