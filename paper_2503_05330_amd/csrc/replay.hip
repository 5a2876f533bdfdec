// csd — launches of a replay's steps side by side: exact matching through the index, DAG pool.
#include "csd_launch.h"

namespace csd {

// From this many drafts on the small LDS layout is used (as in launch_step).
constexpr int64_t kSmallLdsDrafts = 2048;

// (Where a problem's rows are many enough to pay for a CU replay_staged_kernel comes first. The figures up to 1024 problems
// are of such sizes, before it did; those behind of sizes that come here.)
// From this many drafts on those with few matches are made with four or eight lanes each.  Three
// kernels in a row have their latency: us, a wave per draft / by quads, eights and the rest: 1024
// drafts (16 paths x 64 steps) 8.6 / 32, 3072 (64 x 48, long histories) 12.5 / 31 (with a fourth kernel of
// 4 us, before the rest were one), 49152 (64 problems x 16 paths x 48 steps) 73 / 42 (8 + 13 + 21), 393216 (1024
// problems, 24 steps) 533 / 159 (56 + 57 + 46).  Whole passes: 64 problems of 32 x 1024, 24 steps (49152 drafts) 144 / 132, 64
// steps 255 / 213, 4 of 64 x 4096, 128 steps (32768) 369 / 355, 8 of 64 x 2048, 64 steps (32768) 305 / 302, 4096 of 4 x 64, 2
// steps (32768) 96 / 77; but 16 of 32 x 2048, 64, 128 steps (32768, 65536) 203, 250 / 227, 284; below, 2000 of 8 x 512, 2
// steps (32000) 112 / 99, 64 of 32 x 1024, 8 steps (16384) 97 / 103, 4 of 64 x 4096, 48 steps (12288) 241 / 266.  Where the paths
// agree in most tokens nearly all rows are left over (8 of 64 x 2048, 64 steps, all but 5 % 7037 / 11865); the host
// does not know.
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
// drafts, 20 us; 1024 problems x 24 steps, 393216 drafts, 74 us with four waves' rows, 60 with sixteen; passes of sizes that come
// here, four / sixteen: 64 problems of 32 x 1024, 24 steps, 49152 drafts, 132 / 145, 64 steps 206 / 213, 512 of 40 x 512, 24
// steps, 491520, 445 / 450).
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
