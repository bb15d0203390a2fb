// W + H pass of the forward transform, W = 16 .. 64 (see mfma_wh_impl.h).
#include "mfma_wh_impl.h"
namespace fa {
bool wh_fits(const WhPassArgs& a) {
  if (a.H % 16 != 0 || a.W % 16 != 0 || a.kh % 16 != 0 || a.kw % 16 != 0 || a.kh > a.H || a.kw > a.W) return false;
  // Decided by the plane, not by the box kept of it: the two ways sum their products in another order and round another
  // input, so a coefficient has to come from the same one whichever box it is computed on (a head's coefficients are taken on
  // the low box, the low+mid box or the whole grid, by what the call knew beforehand, and its outputs must not tell).
  // More than 64 H coefficients do not fit the accumulators.  Wider tensors (the projected forward's X) have their 128-byte
  // pieces a whole row apart: 16 x 128 channels measured 805 us in two passes, 810 in one.  Each workgroup that shares a plane
  // reads it again from the L2: with four the pass is 15 % faster than two passes (W = 64), with five (80 x 48 kept of
  // 80 x 48) 4 % faster, beyond that the repeated reads cost more than the plane between the axes saved.
  return a.H <= 64 && (a.d == 64 || a.d == 128) && a.W / 16 <= (a.H <= 32 ? 8 : 5);
}
hipError_t launch_wh_pass_0(const WhPassArgs& a, int num_cu, hipStream_t st, int* slots_out) {
  switch (a.W / 16) {
    case 1: return wh_dispatch<1>(a, num_cu, st, slots_out);
    case 2: return wh_dispatch<2>(a, num_cu, st, slots_out);
    case 3: return wh_dispatch<3>(a, num_cu, st, slots_out);
    case 4: return wh_dispatch<4>(a, num_cu, st, slots_out);
  }
  return hipErrorInvalidValue;
}
}  // namespace fa
