// csd — launches of the accept-driven loop with all its steps in one launch.
#include "csd_launch.h"
#include "csd_loop.cuh"

namespace csd {

void launch_loop(const LoopArgs& m, const int32_t* future_tok, const float* future_prob, hipStream_t st) {
  // as far as the steps and the last one's targets reach
  const int64_t reach = (int64_t)m.steps * (m.a.L + 1) + m.a.L;
  const int32_t ahead = reach < m.ix.max_len ? (int32_t)reach : m.ix.max_len, chunks = (ahead + 255) / 256;
  loop_fill_kernel<<<(uint32_t)(m.ix.P * m.ix.N * chunks), 256, 0, st>>>(m.ix, future_tok, future_prob, ahead, chunks);
  if (m.a.L <= 8) launch_loop_steps<8>(m, st);
  else launch_loop_long(m, st);
}

}  // namespace csd
