// csd — launches of a replay's steps side by side with matching by scan.
#include "csd_launch.h"

namespace csd {

// Whether a replay's rows are scanned two a CU (replay_scan_pair_kernel).  It takes
// * more drafts than CUs; with edits twice as many (at fewer a row has a CU for itself, or nearly);
// * problems in which rows of more than a workgroup's worth of matches are rare: those go through tables of
//   half the size, class by class.  How many positions a row matches falls with the tokens that an
//   edit leaves of its query, so the largest problem depends on them;
// * queries of up to four tokens, without pools and options (other code does not fit 64 registers).
// us, one row a CU / two, tokens by Zipf's law from 32000 (paths nearly equal), drafts of 8:
//   one edit, queries of three: 4 x 256, 64 steps 18.9 / 20.4 (15.1 / 16.5), 16 x 1024, 18 steps 41.5 / 46.2 (32.8 /
//   30.6), 32 steps 54 / 49, 64 steps 84 / 73 (57 / 49), 32 problems of 16 x 512, 12 steps 296 / 203 (213 / 151), 32 x
//   1024, 16 steps 124 / 149, 24 steps 134 / 148 (68 / 61), 64 x 1024, 12 steps 233 / 254; drafts of 16: 16 x 1024, 64
//   steps 119 / 99, 32 x 1024, 24 steps 189 / 239, 64 x 1024 339 / 411; of 32: 16 x 1024, 32 steps 127 / 110
//   queries of four: 32 x 1024, 24 steps 89 / 82 (69 / 62), 64 x 1024 144 / 143 (115 / 101)
//   queries of two: 16 x 512, 32 steps 147 / 136, 64 problems of 8 x 256 275 / 202, 16 x 1024, 40 steps 419 / 643, 20 x
//   1000 454 / 2335
//   two edits, queries of four: 16 x 1024, 24 steps 111 / 133, 40 steps 193 / 184, 32 x 2048 2113 / 7285; of three: 16 x
//   512, 32 steps 204 / 197, 8 problems 454 / 388, 16 x 1024, 40 steps 1064 / 2724
//   exact, queries of three: 16 x 512, 18 steps 23.5 / 21.3, 32 x 2048, 24 steps 79 / 64; of two: 16 x 1024, 40 steps
//   40 / 34, 32 x 2048 121 / 131; of one: 64 problems of 8 x 256 229 / 138 (12 symbols), 16 x 512, 32 steps 78 / 99
static bool scan_pairs(const IndexView& v, int32_t steps, const DraftArgs& a) {
  constexpr int64_t kCus = 256;
  const int64_t positions = (int64_t)v.N * v.max_len, drafts = (int64_t)v.P * v.N * steps;
  const int32_t left = a.k - v.eps;
  const int32_t most_log2 = left >= 3 ? 16 : left == 2 ? 14 : v.eps > 0 ? 13 : 12;
  return v.kmax <= 4 && left >= 1 && positions <= (int64_t)1 << most_log2 &&
         drafts >= (v.eps > 0 || left < 2 ? 2 * kCus : kCus + 1);
}

void launch_replay_scan(const IndexView& v, int32_t steps, const DraftArgs& a, hipStream_t st) {
  const uint32_t grid = xcd_grid((int64_t)v.P * v.N * steps);
  const bool general = a.pool_mode != CSD_POOL_DAG || v.options != 0;
  const bool fuzzy = v.eps > 0, q4 = v.kmax <= 4;
  const bool pair = !general && scan_pairs(v, steps, a);
  auto* kernel = pair      ? (fuzzy ? replay_scan_pair_kernel<4, true> : replay_scan_pair_kernel<4, false>)
                 : general ? (fuzzy ? (q4 ? replay_scan_kernel<4, true, true> : replay_scan_kernel<8, true, true>)
                                    : (q4 ? replay_scan_kernel<4, true, false> : replay_scan_kernel<8, true, false>))
                           : (fuzzy ? (q4 ? replay_scan_kernel<4, false, true> : replay_scan_kernel<8, false, true>)
                                    : (q4 ? replay_scan_kernel<4, false, false> : replay_scan_kernel<8, false, false>));
  kernel<<<grid, kScanBlock, 0, st>>>(v, steps, a);
}

}  // namespace csd
