// H + W pass of the inverse transform (see mfma_iwh_impl.h).
#include "mfma_iwh_impl.h"
namespace fa {
bool iwh_fits(const IwhPassArgs& a, int num_cu) {
  if (a.H % 16 != 0 || a.H > 128 || (a.W != 16 && a.W != 32 && a.W != 64)) return false;
  // A workgroup expands its rows one after the other: with fewer than two items of 16 rows per compute unit
  // the two passes are faster (6 slices of 16 x 64 x 64 x 64 from the 32 x 32 box: 42 us, one pass 66; 16K tokens 10 us, one
  // pass 18).  From larger boxes the pass that keeps the output in its accumulators (mfma_wh_impl.h) is faster: 5 slices of
  // 64^3 x 128 from the 32 x 32 box 210 us here, 185 there; 8 of 64 x 64 x 32 x 128 from the 32 x 16 box 146 / 158, of 64 x 32 x 64 x 128 from
  // the 16 x 16 box 111 / 137.
  if ((int64_t)a.n_slices * a.T * (a.d / 64) * (a.H / 16) < 2 * num_cu) return false;
  return (a.kh == 16 || a.kh == 32) && (a.kw == 16 || a.kw == 32) && a.kh * a.kw <= 512 && a.kw <= a.W && (a.d == 64 || a.d == 128);
}
hipError_t launch_iwh_pass(const IwhPassArgs& a, int num_cu, hipStream_t st) {
  switch (a.W / 16) {
    case 1: return iwh_dispatch<1>(a, num_cu, st);
    case 2: return iwh_dispatch<2>(a, num_cu, st);
    case 4: return iwh_dispatch<4>(a, num_cu, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace fa
