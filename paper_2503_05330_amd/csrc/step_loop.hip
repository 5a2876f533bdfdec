// csd — launches of the accept-driven loop's step.
#include "csd_launch.h"

namespace csd {

void launch_step_loop(const IndexView& v, const StepIn& in, const DraftArgs& a, const LoopTail& tail,
                      hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N), block = step_wave_threads(false);
  if (a.L <= 8) step_loop_kernel<8, 4><<<grid, block, 0, st>>>(v, in, a, tail);
  else if (a.L <= 16) step_loop_kernel<16, 4><<<grid, block, 0, st>>>(v, in, a, tail);
  else step_loop_kernel<32, 4><<<grid, block, 0, st>>>(v, in, a, tail);
}

}  // namespace csd
