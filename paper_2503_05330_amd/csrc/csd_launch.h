// csd — launches of the decode step's kernels.  Every family of instantiations has a source
// file of its own, so that they compile side by side.
#pragma once

#include "csd_bins.cuh"
#include "csd_kernels.cuh"

namespace csd {

// a bulk append, sorted by bins of buckets (v.meta_new: v.meta_old)
void launch_append_bins(const IndexView& v, const StepIn& in, const Bins& b, bool maybe_empty, hipStream_t st);

// exact matching through the index, the usual step: DAG pool, at most one token per path
void launch_step(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st);
// the same for steps of several tokens
void launch_step_several(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st);
// the same with the tree and list pools, own history, back-off
void launch_step_general(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st);
// one-edit matching through the variant index
void launch_step_fuzzy(const IndexView& v, const StepIn& in, const DraftArgs& a, hipStream_t st);
// matching by scan
void launch_step_scan(const IndexView& v, const StepIn& in, const DraftArgs& a, const ScanSlices& sl,
                      hipStream_t st);
// one step of the accept-driven loop
void launch_step_loop(const IndexView& v, const StepIn& in, const DraftArgs& a, const LoopTail& tail,
                      hipStream_t st);
// the same with all its steps in one launch (exact matching through the index, DAG pool without options,
// queries of kmax = 2 .. 4 tokens, at most kLoopPaths paths, drafts of up to kLoopLanes tokens)
struct LoopArgs;
void launch_loop(const LoopArgs& m, const int32_t* future_tok, const float* future_prob, hipStream_t st);
void launch_loop_long(const LoopArgs& m, hipStream_t st);   // its steps, drafts of more than eight tokens
void launch_loop_long_two(const LoopArgs& m, hipStream_t st);    // ... of queries of two
void launch_loop_long_four(const LoopArgs& m, hipStream_t st);   // ... and four
// many steps per launch: a replay (general: tree and list pools, own history) / the accept-driven loop
void launch_multi(const IndexView& v, const MultiArgs& m, bool general, hipStream_t st);
void launch_multi_loop(const IndexView& v, const MultiArgs& m, hipStream_t st);

// a replay of many small problems, append and drafts in one launch: workgroups per problem (0: not to be launched
// so), and the launch
int32_t replay_staged_shares(const IndexView& v, int32_t steps, const DraftArgs& a);
void launch_replay_staged(const IndexView& v, const ReplayIn& in, int32_t shares, const DraftArgs& a, int32_t* step_meta,
                          int32_t* done, int32_t* rest_list, hipStream_t st);
void launch_replay_rest(const RestArgs& args, hipStream_t st);   // the rows left to a wave each

// a replay, all steps side by side (v.meta_old: the paths' ends after every step, see
// replay_append_kernel; a: the outputs of the first step): exact matching through the index /
// with the tree and list pools, own history, back-off / one edit through the index / by scan
void launch_replay(const IndexView& v, int32_t steps, const DraftArgs& a, u64* rest,
                   int32_t* rest_list, hipStream_t st);
void launch_replay_general(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st);
void launch_replay_fuzzy(const IndexView& v, int32_t steps, const DraftArgs& a, int32_t* rest_list,
                         hipStream_t st);
void launch_replay_scan(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st);

}  // namespace csd
