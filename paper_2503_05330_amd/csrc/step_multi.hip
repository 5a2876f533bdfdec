// csd — launches of the device-side loops (many steps per launch).
#include "csd_launch.h"

namespace csd {

void launch_multi(const IndexView& v, const MultiArgs& m, bool general, hipStream_t st) {
  const uint32_t grid = (uint32_t)v.P, block = (uint32_t)v.N * kWave;
  const int32_t L = m.a.L;
  if (general) {
    if (L <= 8) step_multi_kernel<8, true, 4, false><<<grid, block, 0, st>>>(v, m);
    else if (L <= 16) step_multi_kernel<16, true, 4, false><<<grid, block, 0, st>>>(v, m);
    else step_multi_kernel<32, true, 4, false><<<grid, block, 0, st>>>(v, m);
  } else {
    if (L <= 8) step_multi_kernel<8, false, 4, false><<<grid, block, 0, st>>>(v, m);
    else if (L <= 16) step_multi_kernel<16, false, 4, false><<<grid, block, 0, st>>>(v, m);
    else step_multi_kernel<32, false, 4, false><<<grid, block, 0, st>>>(v, m);
  }
}

void launch_multi_loop(const IndexView& v, const MultiArgs& m, hipStream_t st) {
  const uint32_t grid = (uint32_t)v.P, block = (uint32_t)v.N * kWave;
  const int32_t L = m.a.L;
  if (L <= 8) step_multi_kernel<8, true, 4, true><<<grid, block, 0, st>>>(v, m);
  else if (L <= 16) step_multi_kernel<16, true, 4, true><<<grid, block, 0, st>>>(v, m);
  else step_multi_kernel<32, true, 4, true><<<grid, block, 0, st>>>(v, m);
}

}  // namespace csd
