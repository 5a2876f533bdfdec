// csd — launches of a replay's steps side by side: exact matching through the index, DAG pool, many
// problems whose histories fit a workgroup's LDS.
#include "csd_launch.h"
#include "csd_staged.cuh"

namespace csd {

// From this many drafts on.  us for reset, append of the past and replay, the launches for the append and the
// drafts / this, problems of 16 x 1024 positions x 24 steps: 2 (32 steps) 31 / 38, 4 37 / 41, 8 53 / 45, 16 77 / 53, 32 84 /
// 60, 64 100 / 61, 128 79 / 66, 200 88 / 73, 300 127 / 119, 1024 340 / 275; 64 of 8 x 512 38 / 30, of 4 x 256 26 / 23.
// Paths that agree in all but 20 %, 5 %, 2 % of their tokens: 64 100, 146, 168 / 67, 90, 103, 1024 533, 1024, 1119 /
// 328, 688, 790.  Queries of two: 64 2092 / 276, 1024 12358 / 1728; drafts of 16: 64 141 / 72, 1024 423 / 311.  Four
// symbols, where all rows are left over: 256 50142 / 50956.
constexpr int64_t kStagedDrafts = 5 << 9;

int32_t replay_staged_shares(const IndexView& v, int32_t steps, const DraftArgs& a) {
  const int64_t rows = (int64_t)v.N * steps, drafts = rows * v.P;
  if (v.gram == nullptr || v.eps > 0 || v.options != 0 || a.pool_mode != CSD_POOL_DAG || drafts < kStagedDrafts || a.k != v.kmax ||
      a.L > 16 || v.N > kStagedPaths || (int64_t)v.N * staged_stride(v.max_len) > kStagedCells)
    return 0;
  // a workgroup for each CU, with enough rows to pay for reading the histories
  constexpr int64_t kCus = 256, kLeastRows = 128;
  int64_t shares = kCus / v.P, most = rows / kLeastRows;
  shares = shares < most ? shares : most;
  const int64_t least = (rows + kStagedRows - 1) / kStagedRows;
  shares = shares > least ? shares : least;
  const int64_t per = (rows + shares - 1) / shares;
  return (int32_t)((rows + per - 1) / per);              // (no share without rows)
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
