// csd — launches of a replay's steps side by side: exact matching through the index, DAG pool, many
// problems whose histories fit a workgroup's LDS.
#include "csd_launch.h"
#include "csd_staged.cuh"

namespace csd {

// Whether it pays to hand a whole CU to each problem, or share of one: only where its rows are many.  Fits of both
// forms' times, ns, for paths that agree in all but 20 % of their tokens (650 sizes: 14 shapes of 2 .. 256 paths of 64 ..
// 4096 positions, 1 .. 4096 problems, 2 .. 250 steps; both fits miss by a tenth on average).  Without them, from 2560
// drafts on, 243 of the 650 took longer than by the launches, up to 2.3 times (us of a replay, launches / this: 4096
// problems of 4 x 256, 4 steps 31 / 138, 1 of 256 x 64, 16 steps 18 / 48, 1024 of 16 x 1024, 2 steps 59 / 89), by them 27.
// Batches keep what they gain: 64 problems of 16 x 1024, 48 steps 52 / 32, 1024, 24 steps 254 / 142.
// Paths that agree in all but 5 % have the line elsewhere, on either side (256 problems of 64 x 64, 16 steps 621 / 282, 64
// of 13 x 777, 16 steps 54 / 96), which the sizes do not tell.  us of reset, append and replay by the agreement, 20 %, 5 %,
// 2 % apart: 64 problems 100, 146, 168 / 67, 90, 103, 1024 533, 1024, 1119 / 328, 688, 790.  Queries of two: 64 2092 /
// 276, 1024 12358 / 1728; drafts of 16: 64 141 / 72, 1024 423 / 311.  Four symbols, where all rows are left over: 256
// 50142 / 50956.
constexpr int64_t kStagedDrafts = 5 << 10;     // (below, the launches are a wave per draft: 14 .. 19 us in all)
constexpr int64_t kCus = 256;

static bool staged_pays(int64_t P, int64_t N, int64_t max_len, int64_t shares, int64_t per, int64_t drafts) {
  const int64_t groups = P * shares, turns = (groups + kCus - 1) / kCus;
  const int64_t cells = N * staged_stride((int32_t)max_len);
  const int64_t spans = N * ((max_len + 511) / 512);     // of positions that a wave passes by the table at once
  const int64_t staged = 6000 + turns * (3000 + 100 * spans + cells / 2 + 23 * per) + 16 * groups;
  const int64_t in_quads = drafts > (1 << 15) ? drafts - (1 << 15) : 0;
  const int64_t launches = 14000 + (drafts - in_quads) / 2 + in_quads / 16 + P * cells / 1500 + drafts * cells / 41000;
  return 20 * staged < 19 * launches;
}

int32_t replay_staged_shares(const IndexView& v, int32_t steps, const DraftArgs& a) {
  const int64_t rows = (int64_t)v.N * steps, drafts = rows * v.P;
  if (v.gram == nullptr || v.eps > 0 || v.options != 0 || a.pool_mode != CSD_POOL_DAG || drafts < kStagedDrafts || a.k != v.kmax ||
      a.L > 16 || v.N > kStagedPaths || (int64_t)v.N * staged_stride(v.max_len) > kStagedCells)
    return 0;
  // a workgroup for each CU, with enough rows to pay for reading the histories
  constexpr int64_t kLeastRows = 128;
  int64_t shares = kCus / v.P, most = rows / kLeastRows;
  shares = shares < most ? shares : most;
  const int64_t least = (rows + kStagedRows - 1) / kStagedRows;
  shares = shares > least ? shares : least;
  const int64_t per = (rows + shares - 1) / shares;
  shares = (rows + per - 1) / per;                       // (no share without rows)
  return staged_pays(v.P, v.N, v.max_len, shares, per, drafts) ? (int32_t)shares : 0;
}

void launch_replay_staged(const IndexView& v, const ReplayIn& in, int32_t shares, const DraftArgs& a, int32_t* step_meta,
                          int32_t* done, int32_t* rest_list, hipStream_t st) {
  const uint32_t grid = (uint32_t)(((int64_t)v.P * shares + 7) / 8 * 8);
  const int32_t per = (v.N * in.steps + shares - 1) / shares;
  const StagedArgs args{v, in, shares, step_meta, done, a, RestList::in(rest_list, true, (int32_t)(grid / 8) * per)};
  auto of = [&](auto lcap, auto edge) {
    constexpr int LCAP = lcap();
    constexpr bool EDGE = edge();
    return v.kmax == 3 ? replay_staged_kernel<LCAP, 3, EDGE> : v.kmax == 4 ? replay_staged_kernel<LCAP, 4, EDGE> : replay_staged_kernel<LCAP, 0, EDGE>;
  };
  const std::integral_constant<int, 8> l8;
  const std::integral_constant<int, 16> l16;
  auto* kernel = a.score_mode == 0 ? (a.L <= 8 ? of(l8, std::false_type{}) : of(l16, std::false_type{}))
                                   : (a.L <= 8 ? of(l8, std::true_type{}) : of(l16, std::true_type{}));
  kernel<<<grid, kStagedThreads, 0, st>>>(args);
  IndexView w = v;
  w.meta_old = w.meta_new = step_meta;
  launch_replay_rest(RestArgs{w, in.steps, a, args.list}, st);
}

}  // namespace csd
