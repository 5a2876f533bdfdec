// csd — launches of the step with matching by scan.
#include "csd_launch.h"

namespace csd {

void launch_step_scan(const IndexView& v, const StepIn& in, const DraftArgs& a, const ScanSlices& sl,
                      hipStream_t st) {
  const int64_t rows = (int64_t)v.P * v.N;
  // few rows: n_slices workgroups per row, the rows dealt to the 8 XCDs
  const uint32_t grid = sl.n > 1 ? (uint32_t)((rows + 7) / 8 * sl.n * 8) : xcd_grid(rows);
  // the general kernels (POOLS) take the tree and list pools, own history, back-off and steps
  // of several tokens
  const bool general = a.pool_mode != CSD_POOL_DAG || v.options != 0 || in.n > 1;
  const bool fuzzy = v.eps > 0, q4 = v.kmax <= 4;
  auto* kernel = general ? (fuzzy ? (q4 ? step_scan_kernel<4, true, true> : step_scan_kernel<8, true, true>)
                                  : (q4 ? step_scan_kernel<4, true, false> : step_scan_kernel<8, true, false>))
                         : (fuzzy ? (q4 ? step_scan_kernel<4, false, true> : step_scan_kernel<8, false, true>)
                                  : (q4 ? step_scan_kernel<4, false, false> : step_scan_kernel<8, false, false>));
  kernel<<<grid, kScanBlock, 0, st>>>(v, in, a, sl);
}

}  // namespace csd
