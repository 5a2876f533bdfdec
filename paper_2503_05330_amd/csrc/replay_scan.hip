// csd — launches of a replay's steps side by side with matching by scan.
#include "csd_launch.h"

namespace csd {

// Problems of up to this many positions are scanned two rows a CU.  With more, rows of thousands of
// matches set the time, which go through the walks' tables class by class, and those are half the
// size there (us, one row a CU / two, one edit, queries of three tokens: 32 x 2048 positions, 16 steps,
// 187 / 186; 64 x 2048, 12 steps, 1567 / 1709; 32 x 4096 1376 / 2227).  Nor do longer queries' predicates
// fit 64 registers, or the code of the pools and options (tree pool, 16 x 1024, 86 / 97).
constexpr int64_t kPairPositions = 1 << 16;

void launch_replay_scan(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N * steps);
  const bool general = a.pool_mode != CSD_POOL_DAG || v.options != 0;
  const bool fuzzy = v.eps > 0, q4 = v.kmax <= 4;
  const bool pair = !general && q4 && (int64_t)v.N * v.max_len <= kPairPositions;
  auto* kernel = pair      ? (fuzzy ? replay_scan_pair_kernel<4, true> : replay_scan_pair_kernel<4, false>)
                 : general ? (fuzzy ? (q4 ? replay_scan_kernel<4, true, true> : replay_scan_kernel<8, true, true>)
                                    : (q4 ? replay_scan_kernel<4, true, false> : replay_scan_kernel<8, true, false>))
                           : (fuzzy ? (q4 ? replay_scan_kernel<4, false, true> : replay_scan_kernel<8, false, true>)
                                    : (q4 ? replay_scan_kernel<4, false, false> : replay_scan_kernel<8, false, false>));
  kernel<<<grid, kScanBlock, 0, st>>>(v, steps, a);
}

}  // namespace csd
