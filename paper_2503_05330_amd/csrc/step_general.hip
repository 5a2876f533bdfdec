// csd — launches of the general step through the index: tree and list pools, own history,
// back-off.
#include "csd_launch.h"

namespace csd {

void launch_step_general(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N), block = step_wave_threads(false);
  if (v.kmax <= 4) {                             // the usual gram lengths: loops unrolled to 4
    if (a.L <= 8) step_wave_kernel<8, true, LdsWave, false, 4><<<grid, block, 0, st>>>(v, in, a);
    else if (a.L <= 16) step_wave_kernel<16, true, LdsWave, false, 4><<<grid, block, 0, st>>>(v, in, a);
    else step_wave_kernel<32, true, LdsWave, false, 4><<<grid, block, 0, st>>>(v, in, a);
  }
  else if (a.L <= 8) step_wave_kernel<8, true, LdsWave, false, CSD_MAX_QUERY_LEN><<<grid, block, 0, st>>>(v, in, a);
  else if (a.L <= 16) step_wave_kernel<16, true, LdsWave, false, CSD_MAX_QUERY_LEN><<<grid, block, 0, st>>>(v, in, a);
  else step_wave_kernel<32, true, LdsWave, false, CSD_MAX_QUERY_LEN><<<grid, block, 0, st>>>(v, in, a);
}

}  // namespace csd
