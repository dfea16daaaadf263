// The fp16 attention kernels (attn.hpp) in a translation unit of their own:
// their accumulators are named accumulation registers, and the check that the
// compiler uses none itself (tests/test_attn_registers.py) compiles this file.
#include "host.hpp"

namespace still {

template <int TT, int D2>
static void launch(const AttnArgs& a, bool track, dim3 grid, hipStream_t st) {
  constexpr int KT = xatt_kb(TT, D2) / 128;
  if (track)
    hipLaunchKernelGGL((xattn_f16_kernel<TT, D2, true, KT>), grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((xattn_f16_kernel<TT, D2, false, KT>), grid, dim3(256), 0, st, a);
}

template <int TT>
static void launch(const AttnArgs& a, bool track, int splits, hipStream_t st) {
  const dim3 grid((unsigned)((a.t + TT - 1) / TT * a.H * a.nc * splits));
  if (a.d2 == 128) launch<TT, 128>(a, track, grid, st);
  else if (a.d2 == 256) launch<TT, 256>(a, track, grid, st);
  else launch<TT, 512>(a, track, grid, st);
}

hipError_t launch_xattn_f16(const AttnArgs& a, bool track, int splits, hipStream_t st) {
  if (xatt_tt(a.t) == 64) launch<64>(a, track, splits, st);
  else launch<128>(a, track, splits, st);
  return hipGetLastError();
}

}  // namespace still
