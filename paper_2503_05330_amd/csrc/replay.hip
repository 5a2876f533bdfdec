// csd — launches of a replay's steps side by side: exact matching through the index, DAG pool.
#include "csd_launch.h"

namespace csd {

// From this many drafts on the small LDS layout is used (as in launch_step).
constexpr int64_t kSmallLdsDrafts = 2048;

// (Problems whose histories fit a workgroup's LDS take replay_staged_kernel from fewer drafts on; the figures
// below are of such problems, before they did.)
// From this many drafts on those with few matches are made with four or eight lanes each.  Three
// kernels in a row have their latency: us, a wave per draft / by quads, eights and the rest: 1024
// drafts (16 paths x 64 steps) 8.6 / 32, 3072 (64 x 48, long histories) 12.5 / 31 (with a fourth kernel of
// 4 us, before the rest were one), 49152 (64 problems x 16 paths x 48 steps) 73 / 42 (8 + 13 + 21), 393216 (1024
// problems, 24 steps) 533 / 159 (56 + 57 + 46).  Where the paths agree in most tokens nearly all rows are
// left over; the host does not know.
constexpr int64_t kQuadDrafts = 1 << 15;

template <class LDS, int QC>
static void launch(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N * steps);
  if (a.L <= 8) replay_wave_kernel<8, false, LDS, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else if (a.L <= 16) replay_wave_kernel<16, false, LDS, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
  else replay_wave_kernel<32, false, LDS, false, QC><<<grid, kWave, 0, st>>>(v, steps, a);
}

// From this many drafts on a workgroup of replay_eight_kernel pools sixteen waves' rows: below, its
// workgroups with four fit the chip at once and have fewer turns (64 problems x 48 steps, 49152
// drafts, 20 us; 1024 problems x 24 steps, 393216 drafts, 74 us with four waves' rows, 60 with sixteen).
constexpr int64_t kPooledDrafts = 1 << 17;

void launch_replay_rest(const RestArgs& args, hipStream_t st) {
  const bool q4 = args.ix.kmax <= 4;
  auto* kernel = args.a.L <= 8    ? (q4 ? replay_rest_kernel<8, 4> : replay_rest_kernel<8, 8>)
                 : args.a.L <= 16 ? (q4 ? replay_rest_kernel<16, 4> : replay_rest_kernel<16, 8>)
                                  : (q4 ? replay_rest_kernel<32, 4> : replay_rest_kernel<32, 8>);
  kernel<<<8 * 2 * kRestTurn, 4 * kWave, 0, st>>>(args);
}

template <int LCAP, int QC, bool EDGE>
static void launch_quads(const IndexView& v, int32_t steps, const DraftArgs& a, u64* rest, int32_t* rest_list,
                         hipStream_t st) {
  const int64_t drafts = (int64_t)v.P * v.N * steps;
  const auto grid = [&](int64_t rows) { return (uint32_t)((drafts + 8 * rows - 1) / (8 * rows) * 8); };   // rows per workgroup
  replay_quad_kernel<LCAP, QC, EDGE><<<grid(4 * kQuadRows), 256, 0, st>>>(v, steps, a, rest);
  const bool pooled = drafts >= kPooledDrafts;
  const RestList list = RestList::in(rest_list, false, (int32_t)(grid((pooled ? 16 : 4) * kQuadRows) / 8) * (pooled ? 16 : 4) * kQuadRows);
  if (pooled) replay_eight_kernel<16, LCAP, QC, EDGE><<<grid(16 * kQuadRows), 256, 0, st>>>(v, steps, a, rest, list);
  else replay_eight_kernel<4, LCAP, QC, EDGE><<<grid(4 * kQuadRows), 256, 0, st>>>(v, steps, a, rest, list);
  launch_replay_rest(RestArgs{v, steps, a, list}, st);
}

template <int QC>
static void launch_quads(const IndexView& v, int32_t steps, const DraftArgs& a, u64* rest, int32_t* rest_list,
                         hipStream_t st) {
  auto* launch = a.score_mode == 0 ? (a.L <= 8 ? launch_quads<8, QC, false> : a.L <= 16 ? launch_quads<16, QC, false> : launch_quads<32, QC, false>)
                                   : (a.L <= 8 ? launch_quads<8, QC, true> : a.L <= 16 ? launch_quads<16, QC, true> : launch_quads<32, QC, true>);
  launch(v, steps, a, rest, rest_list, st);
}

void launch_replay(const IndexView& v, int32_t steps, const DraftArgs& a, u64* rest, int32_t* rest_list,
                   hipStream_t st) {
  const int64_t drafts = (int64_t)v.P * v.N * steps;
  if (drafts >= kQuadDrafts && a.k == v.kmax) {
    if (v.kmax <= 4) launch_quads<4>(v, steps, a, rest, rest_list, st);
    else launch_quads<8>(v, steps, a, rest, rest_list, st);
    return;
  }
  const bool many = drafts >= kSmallLdsDrafts;
  if (v.kmax <= 4) many ? launch<LdsWaveSmall, 4>(v, steps, a, st) : launch<LdsWave, 4>(v, steps, a, st);
  else many ? launch<LdsWaveSmall, 8>(v, steps, a, st) : launch<LdsWave, 8>(v, steps, a, st);
}

}  // namespace csd
