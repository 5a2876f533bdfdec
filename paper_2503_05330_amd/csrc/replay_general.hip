// csd — launches of a replay's steps side by side through the index: tree and list pools, own
// history, back-off.
#include "csd_launch.h"

namespace csd {

template <int QC>
static void launch(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N * steps);
  if (a.L <= 8) replay_wave_kernel<8, true, LdsWave, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else if (a.L <= 16) replay_wave_kernel<16, true, LdsWave, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else replay_wave_kernel<32, true, LdsWave, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
}

void launch_replay_general(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  if (v.kmax <= 4) launch<4>(v, steps, a, st);
  else launch<CSD_MAX_QUERY_LEN>(v, steps, a, st);
}

}  // namespace csd
