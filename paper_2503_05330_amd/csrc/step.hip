// csd — launches of the usual step: exact matching through the index, DAG pool, at most one
// token per path.
#include "csd_launch.h"

namespace csd {

// From this many rows on (256 CUs x 4 rows of the regular layout are resident at once) the
// one-wave kernel runs with the small LDS layout.
constexpr int64_t kSmallLdsRows = 2048;

void launch_step(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st) {
  const int64_t rows = (int64_t)v.P * v.N;
  const uint32_t grid = xcd_grid(rows), block = step_wave_threads(false);
  // (what an index has not, home blocks, is not asked for: 65536 rows 81.6 us, with one form for both 84.8)
  auto launch = [&](auto qc, auto blocks) {
    constexpr int QC = qc();
    constexpr bool BLOCKS = blocks();
    if (a.L <= 8 && rows >= kSmallLdsRows)       // more rows than fit the chip at once
      step_wave_many_kernel<QC, BLOCKS><<<grid, block, 0, st>>>(v, in, a);
    else if (a.L <= 8)
      step_wave_kernel<8, false, LdsWave, false, QC, false, BLOCKS><<<grid, block, 0, st>>>(v, in, a);
    else if (a.L <= 16)
      step_wave_kernel<16, false, LdsWave, false, QC, false, BLOCKS><<<grid, block, 0, st>>>(v, in, a);
    else
      step_wave_kernel<32, false, LdsWave, false, QC, false, BLOCKS><<<grid, block, 0, st>>>(v, in, a);
  };
  auto of = [&](auto qc) {
    if (v.buckets.mask > v.buckets.block) launch(qc, std::true_type{});
    else launch(qc, std::false_type{});
  };
  if (v.kmax <= 4) of(std::integral_constant<int, 4>{});   // the usual gram lengths: loops unrolled to 4
  else of(std::integral_constant<int, 8>{});
}

}  // namespace csd
