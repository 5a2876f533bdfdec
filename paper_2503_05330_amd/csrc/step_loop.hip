// csd — launches of the accept-driven loop's step.
#include "csd_launch.h"

namespace csd {

template <bool POOLS>
static void launch(const IndexView& v, const StepIn& in, const DraftArgs& a, const LoopTail& tail, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N), block = step_wave_threads(false);
  if (a.L <= 8) step_loop_kernel<8, 4, POOLS><<<grid, block, 0, st>>>(v, in, a, tail);
  else if (a.L <= 16) step_loop_kernel<16, 4, POOLS><<<grid, block, 0, st>>>(v, in, a, tail);
  else step_loop_kernel<32, 4, POOLS><<<grid, block, 0, st>>>(v, in, a, tail);
}

void launch_step_loop(const IndexView& v, const StepIn& in, const DraftArgs& a, const LoopTail& tail,
                      hipStream_t st) {
  // (code that a launch does not run still costs it time: 16 x 1024, 7.1 us a step with the pools' and
  // options' code, 6.8 without)
  if (a.pool_mode != CSD_POOL_DAG || v.options != 0) launch<true>(v, in, a, tail, st);
  else launch<false>(v, in, a, tail, st);
}

}  // namespace csd
