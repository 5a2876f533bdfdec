// csd — launches of a step of several tokens through the index, DAG pool: without the code of the
// pools and options, which costs a launch time although it is not run (16 x 1024, 1 .. 9 tokens a
// path: 7.2 us, 6.96 without).
#include "csd_launch.h"

namespace csd {

template <int QC>
static void launch(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N), block = step_wave_threads(false);
  if (a.L <= 8) step_wave_kernel<8, false, LdsWave, false, QC, true><<<grid, block, 0, st>>>(v, in, a);
  else if (a.L <= 16) step_wave_kernel<16, false, LdsWave, false, QC, true><<<grid, block, 0, st>>>(v, in, a);
  else step_wave_kernel<32, false, LdsWave, false, QC, true><<<grid, block, 0, st>>>(v, in, a);
}

void launch_step_several(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st) {
  if (v.kmax <= 4) launch<4>(v, in, a, st);              // the usual gram lengths: loops unrolled to 4
  else launch<CSD_MAX_QUERY_LEN>(v, in, a, st);
}

}  // namespace csd
