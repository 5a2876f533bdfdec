// csd — launches of a replay's steps side by side with one-edit matching through the variant index.
#include "csd_launch.h"

namespace csd {

// Two rows a CU are under way with LdsWaveFuzzy, so with more drafts than that some wait for others, and
// the rows with many matches, which set the time, start last.  Beyond it they are left to workgroups (us for
// reset, append of the past and replay, all by waves / so: 512 drafts, 16 paths x 1024 tokens, 32 / 33; 768,
// 32 x 2048, 55 / 51; 1536, 64 x 4096, 170 / 153; 4800, 40 problems of 5 x 1000, 95 / 57; 6144, 12 problems of 16 x
// 1024, 269 / 171.  The drafts of 64 x 4096 alone, for two sets of inputs, 107 / 35 + 31 and 52 / 31 + 5, the same
// behind either form of the append).  The replay alone, where it is near or loses: tree and list pool, 16 x 1024,
// 640 drafts 71 / 74 and 48 / 53, paths nearly equal 68 / 53 and 67 / 55, 768 drafts 79 / 74 and 56 / 54; queries of
// six over six symbols, 64 x 1024, 324 / 348.
constexpr int64_t kOneTurn = 512;

template <int QC>
static void launch(const IndexView& v, int32_t steps, const DraftArgs& a, int32_t* rest_list, hipStream_t st) {
  const int64_t drafts = (int64_t)v.P * v.N * steps;
  const uint32_t grid = xcd_grid(drafts);
  if (drafts > kOneTurn) {
    const RestList list = RestList::in(rest_list, false, (int32_t)(grid / 8));
    if (a.L <= 8) replay_leave_kernel<8, QC><<<grid, kWave, 0, st>>>(v, steps, a, list);
    else if (a.L <= 16) replay_leave_kernel<16, QC><<<grid, kWave, 0, st>>>(v, steps, a, list);
    else replay_leave_kernel<32, QC><<<grid, kWave, 0, st>>>(v, steps, a, list);
    if (a.pool_mode != CSD_POOL_DAG || v.options != 0) replay_left_kernel<QC, true><<<256, kScanBlock, 0, st>>>(v, steps, a, list);
    else replay_left_kernel<QC, false><<<256, kScanBlock, 0, st>>>(v, steps, a, list);
    return;
  }
  if (a.L <= 8) replay_wave_kernel<8, true, LdsWaveFuzzy, true, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else if (a.L <= 16) replay_wave_kernel<16, true, LdsWaveFuzzy, true, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else replay_wave_kernel<32, true, LdsWaveFuzzy, true, QC><<<grid, kWave, 0, st>>>(v, steps, a);
}

void launch_replay_fuzzy(const IndexView& v, int32_t steps, const DraftArgs& a, int32_t* rest_list, hipStream_t st) {
  if (v.kmax <= 4) launch<4>(v, steps, a, rest_list, st);
  else launch<CSD_MAX_QUERY_LEN>(v, steps, a, rest_list, st);
}

}  // namespace csd
