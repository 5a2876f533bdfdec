// csd — launches of the accept-driven loop with all its steps in one launch.
#include "csd_launch.h"
#include "csd_loop.cuh"

namespace csd {

void launch_loop(const LoopArgs& m, const int32_t* future_tok, const float* future_prob, hipStream_t st) {
  // as far as the steps and the last one's targets reach
  const int64_t reach = (int64_t)m.steps * (m.a.L + 1) + m.a.L;
  const int32_t ahead = reach < m.ix.max_len ? (int32_t)reach : m.ix.max_len, chunks = (ahead + 255) / 256;
  // (a grid's threads are less than 2^32; a workgroup takes several paths beyond this many workgroups)
  constexpr int32_t kFillGroups = 1 << 22;
  const int32_t rows = m.ix.P * m.ix.N, most = kFillGroups / chunks;   // (at most 2^16 chunks: CSD_MAX_POSITIONS)
  const int32_t row_groups = rows < most ? rows : most;
  loop_fill_kernel<<<(uint32_t)(row_groups * chunks), 256, 0, st>>>(m.ix, future_tok, future_prob, ahead, chunks, row_groups);
  if (hipPeekAtLastError() != hipSuccess) return;        // (the caller sees it: no steps on histories that were not filled)
  if (m.a.L > 8) launch_loop_long(m, st);
  else if (m.ix.kmax == 2) launch_loop_kernel<8, 2>(m, st);
  else if (m.ix.kmax == 3) launch_loop_kernel<8, 3>(m, st);
  else launch_loop_kernel<8, 4>(m, st);
}

}  // namespace csd
