// csd — launches of a replay's steps side by side: exact matching through the index, DAG pool.
#include "csd_launch.h"

namespace csd {

// From this many drafts on the small LDS layout is used (as in launch_step).
constexpr int64_t kSmallLdsDrafts = 2048;

template <class LDS, int QC>
static void launch(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N * steps);
  if (a.L <= 8) replay_wave_kernel<8, false, LDS, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else if (a.L <= 16) replay_wave_kernel<16, false, LDS, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else replay_wave_kernel<32, false, LDS, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
}

void launch_replay(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const bool many = (int64_t)v.P * v.N * steps >= kSmallLdsDrafts;
  if (v.kmax <= 4) many ? launch<LdsWaveSmall, 4>(v, steps, a, st) : launch<LdsWave, 4>(v, steps, a, st);
  else many ? launch<LdsWaveSmall, 8>(v, steps, a, st) : launch<LdsWave, 8>(v, steps, a, st);
}

}  // namespace csd
