// csd — launches of the bulk append whose postings are sorted by range of buckets first.
#include "csd_launch.h"

namespace csd {

template <bool FUZZY, int QC>
static void launch(const IndexView& v, const StepIn& in, const Bins& b, bool maybe_empty, hipStream_t st) {
  bin_sort_kernel<FUZZY, QC><<<(uint32_t)(v.P * b.sources), kBinSource, 0, st>>>(v, in, b);
  bin_file_kernel<<<(uint32_t)(v.P * b.bins), 1024, 0, st>>>(v, b, maybe_empty ? 1 : 0);
  bin_rest_kernel<FUZZY, QC><<<(uint32_t)(v.P * kRestGroups), 256, 0, st>>>(v, b);
}

void launch_append_bins(const IndexView& v, const StepIn& in, const Bins& b, bool maybe_empty, hipStream_t st) {
  const bool q4 = v.kmax <= 4;
  if (v.eps > 0) q4 ? launch<true, 4>(v, in, b, maybe_empty, st) : launch<true, CSD_MAX_QUERY_LEN>(v, in, b, maybe_empty, st);
  else q4 ? launch<false, 4>(v, in, b, maybe_empty, st) : launch<false, CSD_MAX_QUERY_LEN>(v, in, b, maybe_empty, st);
}

}  // namespace csd
