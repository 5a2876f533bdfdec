// csd — launches of the usual step: exact matching through the index, DAG pool, at most one
// token per path.
#include "csd_launch.h"

namespace csd {

// From this many rows on (256 CUs x 4 rows of the regular layout are resident at once) the
// one-wave kernel runs with the small LDS layout.
constexpr int64_t kSmallLdsRows = 2048;

void launch_step(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st) {
  const int64_t rows = (int64_t)v.P * v.N;
  const uint32_t grid = xcd_grid(rows), block = step_wave_threads(false);
  if (v.kmax <= 4) {                             // the usual gram lengths: loops unrolled to 4
    if (a.L <= 8 && rows >= kSmallLdsRows)       // more rows than fit the chip at once
      step_wave_many_kernel<4><<<grid, block, 0, st>>>(v, in, a);
    else if (a.L <= 8)
      step_wave_kernel<8, false, LdsWave, false, 4><<<grid, block, 0, st>>>(v, in, a);
    else if (a.L <= 16)
      step_wave_kernel<16, false, LdsWave, false, 4><<<grid, block, 0, st>>>(v, in, a);
    else
      step_wave_kernel<32, false, LdsWave, false, 4><<<grid, block, 0, st>>>(v, in, a);
  } else if (a.L <= 8 && rows >= kSmallLdsRows)
    step_wave_many_kernel<8><<<grid, block, 0, st>>>(v, in, a);
  else if (a.L <= 8)
    step_wave_kernel<8, false, LdsWave, false, 8><<<grid, block, 0, st>>>(v, in, a);
  else if (a.L <= 16)
    step_wave_kernel<16, false, LdsWave, false, 8><<<grid, block, 0, st>>>(v, in, a);
  else
    step_wave_kernel<32, false, LdsWave, false, 8><<<grid, block, 0, st>>>(v, in, a);
}

}  // namespace csd
