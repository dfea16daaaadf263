// The fp16 attention kernels (attn.hpp) in a translation unit of their own:
// their accumulators are named accumulation registers, and the check that the
// compiler uses none itself (tests/test_attn_registers.py) compiles this file.
#include "host.hpp"

namespace still {

template <int D2>
static void launch(const AttnArgs& a, bool track, dim3 grid, hipStream_t st) {
  constexpr int KT = xatt_kb(D2) / 128;
  if (track)
    hipLaunchKernelGGL((xattn_f16_kernel<ATT_TT, D2, true, KT>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((xattn_f16_kernel<ATT_TT, D2, false, KT>), grid, dim3(256), 0, st, a);
}

hipError_t launch_xattn_f16(const AttnArgs& a, bool track, int splits, hipStream_t st) {
  const dim3 grid((unsigned)((a.t + ATT_TT - 1) / ATT_TT * a.H * a.nc * splits));
  if (a.d2 == 128) launch<128>(a, track, grid, st);
  else if (a.d2 == 256) launch<256>(a, track, grid, st);
  else launch<512>(a, track, grid, st);
  return hipGetLastError();
}

}  // namespace still
