// csd — launches of the accept-driven loop with all its steps in one launch: drafts of more than eight tokens.
#include "csd_launch.h"
#include "csd_loop.cuh"

namespace csd {

void launch_loop_long(const LoopArgs& m, hipStream_t st) { launch_loop_steps<16>(m, st); }

}  // namespace csd
