// csd — launches of a replay's steps side by side with matching by scan.
#include "csd_launch.h"

namespace csd {

void launch_replay_scan(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N * steps);
  const bool general = a.pool_mode != CSD_POOL_DAG || v.options != 0;
  const bool fuzzy = v.eps > 0, q4 = v.kmax <= 4;
  auto* kernel = general ? (fuzzy ? (q4 ? replay_scan_kernel<4, true, true> : replay_scan_kernel<8, true, true>)
                                  : (q4 ? replay_scan_kernel<4, true, false> : replay_scan_kernel<8, true, false>))
                         : (fuzzy ? (q4 ? replay_scan_kernel<4, false, true> : replay_scan_kernel<8, false, true>)
                                  : (q4 ? replay_scan_kernel<4, false, false> : replay_scan_kernel<8, false, false>));
  kernel<<<grid, kScanBlock, 0, st>>>(v, steps, a);
}

}  // namespace csd
