// csd — launches of the accept-driven loop with all its steps in one launch: drafts of more than eight tokens.
#include "csd_launch.h"
#include "csd_loop.cuh"

namespace csd {

void launch_loop_long(const LoopArgs& m, hipStream_t st) {
  if (m.ix.kmax == 4) launch_loop_long_four(m, st);
  else if (m.ix.kmax == 3) launch_loop_kernel<16, 3>(m, st);
  else launch_loop_long_two(m, st);
}

}  // namespace csd
