// Dispatcher of the DCT axis pass (paper sections 3.2, 3.7): picks the addressing mode of the launch; the kernel is in
// mfma_dct_impl.h and is instantiated once per mode in mfma_dct_<mode>.hip.
#include <hip/hip_runtime.h>

#include "ctx.h"

namespace fa {

hipError_t launch_mfma_dct_plain(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out);
hipError_t launch_mfma_dct_plain_tot(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out);
hipError_t launch_mfma_dct_scatter(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out);
hipError_t launch_mfma_dct_scatter_en(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out);
hipError_t launch_mfma_dct_gather(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out);

bool mfma_dct_supported(int n_in, int n_out) {
  return n_in % 16 == 0 && n_in >= 16 && n_in <= 128 && n_out >= 1 && n_out <= 128;
}

int mfma_dct_tiles(int n_in, int n_out) {
  const int mt = (n_out + 31) / 32;
  return mt == 3 && n_in != 48 && n_in != 80 && n_in != 96 ? 4 : mt;   // (dispatch_mode: variants with three tiles exist for these)
}

hipError_t launch_mfma_dct_pass(const DctPassArgs* subs, int n, int num_cu, hipStream_t st, int* waves_out) {
  const DctPassArgs& first = subs[0];
  if (n < 1 || n > 3) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i) {
    const DctPassArgs& a = subs[i];
    if (a.inner % 64 != 0 || a.inner % a.d != 0 || !mfma_dct_supported(a.n, a.n_out) || a.ldm < a.n) return hipErrorInvalidValue;
    if (a.perm_in && (a.perm_out || !a.masks || !a.in_alt)) return hipErrorInvalidValue;
    if (a.energy_part && !a.perm_out) return hipErrorInvalidValue;
    if (a.n != first.n || mfma_dct_tiles(a.n, a.n_out) > mfma_dct_tiles(first.n, first.n_out) || !a.perm_in != !first.perm_in ||
        !a.perm_out != !first.perm_out || !a.energy_part != !first.energy_part || !a.tot_part != !first.tot_part)
      return hipErrorInvalidValue;
  }
  if (first.perm_in) return launch_mfma_dct_gather(subs, n, num_cu, st, waves_out);
  if (first.perm_out) return first.energy_part ? launch_mfma_dct_scatter_en(subs, n, num_cu, st, waves_out)
                                               : launch_mfma_dct_scatter(subs, n, num_cu, st, waves_out);
  return first.tot_part ? launch_mfma_dct_plain_tot(subs, n, num_cu, st, waves_out) : launch_mfma_dct_plain(subs, n, num_cu, st, waves_out);
}

}  // namespace fa
