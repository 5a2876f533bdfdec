// csd — launches of the accept-driven loop with all its steps in one launch: drafts of more than eight
// tokens, queries of four (compiled beside the others).
#include "csd_launch.h"
#include "csd_loop.cuh"

namespace csd {

void launch_loop_long_four(const LoopArgs& m, hipStream_t st) { launch_loop_kernel<16, 4>(m, st); }

}  // namespace csd
