// W + H pass of the forward transform, W = 80 .. 128 (see mfma_wh_impl.h).
#include "mfma_wh_impl.h"
namespace fa {
hipError_t launch_wh_pass_1(const WhPassArgs* subs, int n, int num_cu, hipStream_t st, int* slots_out) {
  switch (subs[0].cols / 16) {
    case 5: return wh_dispatch<5, false>(subs, n, num_cu, st, slots_out);
    case 6: return wh_dispatch<6, false>(subs, n, num_cu, st, slots_out);
    case 7: return wh_dispatch<7, false>(subs, n, num_cu, st, slots_out);
    case 8: return wh_dispatch<8, false>(subs, n, num_cu, st, slots_out);
  }
  return hipErrorInvalidValue;
}
}  // namespace fa
