// csd — the bulk append of few large problems: the postings are sorted by range of buckets first.
//
// An append with a thread per position claims every slot with an atomic on memory, and those run at
// the memory's side of the fabric, 1.1e10 per second for the whole chip: 2.6e5 postings 22 us, 1.3e6 (one
// edit) 88 us.  Sorted by bins they take 8 + 10 + 2 and 11 + 19 .. 24 + 5: two passes over the records, one over the
// index.  A bin of buckets is one workgroup's, which claims in LDS, and the home block of its grams, so that nearly all of a
// chain is (with sequences through the whole table the last launch filed what found its first bucket full, 15 .. 21 us
// behind 14 with one edit):
//   bin_sort_kernel   stores tokens and probabilities, and each workgroup's records (bucket, posting)
//                     ordered by bin; a counting sort in LDS, no atomic on memory
//   bin_file_kernel   a workgroup per bin gathers its runs of records, claims slots on its fill counts and
//                     stores its buckets as whole lines; a posting that finds no slot near is set aside
//   bin_rest_kernel   files those (hundreds of one gram) along their chains, which lead to other bins, with atomics
//                     on memory, and replaces the paths' ends
// sorted_append (csd.hip) says which appends take it.
#pragma once

#include "csd_common.cuh"
#include "csd_index.cuh"

namespace csd {

constexpr int32_t kBinSource = 1024;   // positions of a sorting workgroup, all of one path
constexpr int32_t kMostBins = 1024;    // bins of a problem, and sorting workgroups of it
constexpr int32_t kBinBuckets = 1024;  // of a bin at most: 64 KB of LDS
constexpr int32_t kRestGroups = 512;   // workgroups of bin_rest_kernel per problem

struct BinRecord {
  int32_t bucket, posting;      // bucket: above kBinStep bits the gram's step within its home block
};
constexpr int kBinStep = 20;
struct Bins {
  BinRecord* records;           // [P][sources][kBinSource * variants]
  uint32_t* runs;               // [P][bins][sources]: a bin's records of a source, first << 16 | how many
  int32_t* over;                // postings that find no slot near; a part for each bin:
  int32_t* over_first;          // [P][bins]
  int32_t* over_count;          // [P][bins]
  int32_t* over_used;           // parts given out in this append; behind it: postings set aside in all
  int32_t* ends;                // rows like meta's: the paths' new ends
  int32_t chunks, sources;      // sorting workgroups per path, per problem
  int32_t variants;             // postings per position at most
  int32_t bins, buckets_log2;   // per problem; buckets of a bin
};

// Sum of x over the threads of the workgroup before this one, and over all (`part`: a word per wave).
template <int THREADS>
__device__ __forceinline__ int32_t block_prefix(int32_t x, int32_t* part, int tid, int32_t& total) {
  const int lane = tid & (kWave - 1), wave = tid >> 6;
  int32_t sum = x;
#pragma unroll
  for (int d = 1; d < kWave; d *= 2) {
    const int32_t below = __shfl_up(sum, d);
    if (lane >= d) sum += below;
  }
  if (lane == kWave - 1) part[wave] = sum;
  __syncthreads();
  int32_t before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < THREADS / kWave; ++w) {
    before += w < wave ? part[w] : 0;
    total += part[w];
  }
  return before + sum - x;
}

// The last of the kMostBins entries of an ascending list that is not above x (the first one is not).
__device__ __forceinline__ int32_t last_not_above(const int32_t* list, int32_t x) {
  int32_t at = 0;
#pragma unroll
  for (int32_t half = kMostBins / 2; half > 0; half /= 2) at += list[at + half] <= x ? half : 0;
  return at;
}

template <bool FUZZY, int QC>
__global__ __launch_bounds__(kBinSource) void bin_sort_kernel(IndexView ix, StepIn in, Bins b) {
  constexpr int kVariants = FUZZY ? QC + 1 : 1;
  __shared__ int32_t count[kMostBins], part[kBinSource / kWave];
  __shared__ BinRecord sorted[kBinSource * kVariants];   // (they go to memory as one stream)
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
  const int32_t row = (int32_t)blockIdx.x / b.chunks, chunk = (int32_t)blockIdx.x - row * b.chunks;
  const int32_t p = row / ix.N, i = row - p * ix.N, source = i * b.chunks + chunk;
  if (blockIdx.x == 0 && tid < 2) b.over_used[tid] = 0;
  NewTokens<QC> x;
  x.load(ix, in, row, chunk * kBinSource + tid);
  for (int32_t c = tid; c < b.bins; c += kBinSource) count[c] = 0;
  const int32_t cnt = x.count(ix);
  uint32_t flags = x.store(ix, in.prob != nullptr, row, cnt);
  if (chunk == 0 && tid < kWave) {
    if (tid == 0 && x.most() > cnt) flags |= CSD_STATUS_CAPACITY;
    store_end(ix, in, row, x.len, cnt, b.ends, lane);
  }
  if (flags) atomicOr(ix.status, flags);
  int32_t at[kVariants], step[kVariants], rank[kVariants];
  uint32_t live = 0;
#pragma unroll
  for (int v = 0; v < kVariants; ++v) {
    bool on = x.filed(ix, cnt) && v <= ix.kmax;
    if (v >= 2) on = on && x.G[v - 1] != x.G[v - 2];     // (else the same string as variant v - 1)
    const GramHash gh = variant_hash(x.G, ix.kmax, v);
    at[v] = (int32_t)(gh.h & ix.buckets.mask);
    step[v] = (int32_t)(gh.step & ix.buckets.block);
    live |= on ? 1u << v : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int v = 0; v < kVariants; ++v)
    if (live >> v & 1u) rank[v] = atomicAdd(&count[at[v] >> b.buckets_log2], 1);
  __syncthreads();
  int32_t total;
  const int32_t mine = tid < b.bins ? count[tid] : 0;
  const int32_t first = block_prefix<kBinSource>(mine, part, tid, total);
  if (tid < b.bins) {
    b.runs[((int64_t)p * b.bins + tid) * b.sources + source] = (uint32_t)first << 16 | (uint32_t)mine;
    count[tid] = first;
  }
  __syncthreads();
  const int32_t pos = x.pos(ix, i);
#pragma unroll
  for (int v = 0; v < kVariants; ++v)
    if (live >> v & 1u)
      sorted[count[at[v] >> b.buckets_log2] + rank[v]] = BinRecord{at[v] | step[v] << kBinStep, FUZZY ? variant_posting(pos, v) : pos};
  __syncthreads();
  BinRecord* records = b.records + ((int64_t)p * b.sources + source) * (kBinSource * b.variants);
  for (int32_t f = tid; f < total; f += kBinSource) records[f] = sorted[f];
}

// maybe_empty: see append_problem_kernel.
static __global__ __launch_bounds__(1024) void bin_file_kernel(IndexView ix, Bins b, int32_t maybe_empty) {
  __shared__ int4 table[kBinBuckets * 4];
  __shared__ int32_t fill[kBinBuckets], before[kMostBins], first[kMostBins], part[1024 / kWave];
  __shared__ int32_t n_over, over_at;
  const int tid = (int)threadIdx.x;
  const int32_t p = (int32_t)blockIdx.x / b.bins, bin = (int32_t)blockIdx.x - p * b.bins;
  const int32_t buckets = 1 << b.buckets_log2;
  int32_t* gram = ix.gram + ((int64_t)p * ((int64_t)ix.buckets.mask + 1) + ((int64_t)bin << b.buckets_log2)) * kBucketWords;
  const uint32_t run = tid < b.sources ? b.runs[(int64_t)blockIdx.x * b.sources + tid] : 0u;
  int32_t lens = 1;
  if (maybe_empty) {                                     // uniform over the launch
    lens = 0;
    for (int32_t j = tid; j < ix.N; j += 1024) lens |= ix.meta_old[((int64_t)p * ix.N + j) * ix.meta_stride];
  }
  if (tid == 0) n_over = 0;
  int32_t total;
  before[tid] = block_prefix<1024>((int32_t)(run & 0xFFFFu), part, tid, total);
  first[tid] = (int32_t)(run >> 16);
  if (tid == 0) over_at = total > 0 ? atomicAdd(b.over_used, total) : 0;
  const bool empty = __syncthreads_or(lens) == 0;        // (and the lists above are whole)
  if (empty) {
    for (int32_t x = tid; x < buckets * 4; x += 1024) table[x] = int4{-1, -1, -1, -1};
    for (int32_t x = tid; x < buckets; x += 1024) fill[x] = 0;
  } else {
    for (int32_t x = tid; x < buckets * 4; x += 1024) {
      const int4 words = reinterpret_cast<const int4*>(gram)[x];
      table[x] = words;
      if ((x & 3) == 0) fill[x >> 2] = words.x;
    }
  }
  __syncthreads();
  const BinRecord* records = b.records + (int64_t)p * b.sources * (kBinSource * b.variants);
  int32_t* slots = reinterpret_cast<int32_t*>(table);
  auto file = [&](auto at_once) {                        // records of a thread that are in flight together
    constexpr int kAtOnce = decltype(at_once)::value;
    constexpr uint32_t kTogether = 8;
    for (int32_t f0 = tid; f0 < total; f0 += kAtOnce * 1024) {
      BinRecord rec[kAtOnce];
#pragma unroll
      for (int y = 0; y < kAtOnce; ++y) {
        const int32_t f = f0 + y * 1024 < total ? f0 + y * 1024 : f0;
        const int32_t s = last_not_above(before, f);
        rec[y] = records[(int64_t)s * (kBinSource * b.variants) + first[s] + (f - before[s])];
      }
#pragma unroll
      for (int y = 0; y < kAtOnce; ++y) {
        if (f0 + y * 1024 >= total) continue;
        const int32_t local = rec[y].bucket & (buckets - 1);
        // the first bucket, then the others near (all this bin's) eight at a time
        const GramHash gh{(uint32_t)local, (uint32_t)rec[y].bucket >> kBinStep};
        bool open = true;
        auto claim = [&](uint32_t at) {
          const int32_t c = atomicAdd(&fill[at], 1);
          if (c < kBucketSlots) {
            slots[at * kBucketWords + 1 + c] = rec[y].posting;
            open = false;
          }
        };
        if (fill[local] < kBucketSlots) claim((uint32_t)local);   // (a full bucket is passed without an atomic)
        for (uint32_t r = 1; r < kNear && open; r += kTogether) {
          uint32_t at[kTogether];
          int32_t filled[kTogether];
#pragma unroll
          for (uint32_t z = 0; z < kTogether; ++z) {
            at[z] = (gh.h + (r + z) * gh.step) & ((uint32_t)buckets - 1u);
            filled[z] = r + z < kNear ? fill[at[z]] : kBucketSlots;
          }
#pragma unroll
          for (uint32_t z = 0; z < kTogether; ++z)
            if (open && filled[z] < kBucketSlots) claim(at[z]);
        }
        if (open) b.over[over_at + atomicAdd(&n_over, 1)] = rec[y].posting;
      }
    }
  };
  if (total <= 1024) file(std::integral_constant<int, 1>{});   // uniform over the workgroup
  else file(std::integral_constant<int, 6>{});
  __syncthreads();
  for (int32_t x = tid; x < buckets * 4; x += 1024) {
    int4 words = table[x];
    if ((x & 3) == 0) words.x = fill[x >> 2];
    reinterpret_cast<int4*>(gram)[x] = words;
  }
  if (tid == 0) {
    b.over_first[blockIdx.x] = over_at;
    b.over_count[blockIdx.x] = n_over;
    if (n_over > 0) atomicAdd(b.over_used + 1, n_over);
  }
}

// gram_insert_from for the postings of several lanes (`members`) that have one gram: a claim takes as many slots
// of a bucket as it is seen to have left.  (Frequent grams: hundreds of waves after the same buckets.)
__device__ __forceinline__ void gram_insert_group(int32_t* tbl, Buckets tb, GramHash gh, uint32_t r0,
                                                  u64 members, int32_t posting, int lane) {
  const bool mine = (members >> lane & 1u) != 0;
  int32_t rank = (int32_t)__popcll(members & ((1ull << lane) - 1ull));   // among those without a slot
  int32_t left = (int32_t)__popcll(members);
  const uint32_t turns = gram_turns(tb);
  for (; r0 < turns; r0 += kWave) {
    const uint32_t r = r0 + lane;
    const int32_t fill = r < turns ? gram_bucket(tbl, gh, r, tb)[0] : kBucketSlots;
    u64 m = wave_ballot(fill < kBucketSlots);
    while (m) {
      const int first = (int)__ffsll((long long)m) - 1;
      m &= m - 1;
      int32_t* b = gram_bucket(tbl, gh, r0 + (uint32_t)first, tb);
      const int32_t open = kBucketSlots - __builtin_amdgcn_readlane(fill, first);
      const int32_t want = open < left ? open : left;
      int32_t c = 0;
      if (lane == 0) c = atomicAdd(b, want);
      c = __builtin_amdgcn_readfirstlane(c);
      int32_t got = kBucketSlots - c;
      got = got < 0 ? 0 : (got < want ? got : want);
      if (mine && rank >= 0 && rank < got) b[1 + c + rank] = posting;
      rank -= got;                                  // negative: stored
      left -= got;
      if (left == 0) return;
    }
  }
}

// The posting of each lane whose near buckets are full (`open`: the lane has one), on along its chain: lanes
// that share one as a group; the others claim in the next three buckets, a lane for itself, and what is
// left then (a long chain) is the whole wave's.
// (us, bin_rest_kernel of 64 paths x 4096 tokens with one edit, when all that found their first bucket full came
// here: a wave inserting posting by posting 65 with a lane for every one, 31 with them spread over the waves, in groups 23.)
constexpr int kGroupLanes = 4;
__device__ __forceinline__ void file_along_chain(int32_t* gram, Buckets tb, GramHash gh, int32_t posting,
                                                 bool open, int lane) {
  auto file_groups = [&](uint32_t r0, int least) {
    u64 left = wave_ballot(open);
    while (left) {                                       // uniform over the wave
      const int t = (int)__ffsll((long long)left) - 1;
      const GramHash g{(uint32_t)__builtin_amdgcn_readlane((int)gh.h, t),
                       (uint32_t)__builtin_amdgcn_readlane((int)gh.step, t)};
      const u64 same = wave_ballot(gh.h == g.h && gh.step == g.step) & left;
      left &= ~same;
      if (__popcll(same) < least) continue;
      gram_insert_group(gram, tb, g, r0, same, posting, lane);
      if (same >> lane & 1u) open = false;
    }
  };
  file_groups(kNear, kGroupLanes);
  for (uint32_t r = kNear; r < kNear + 3u && r < gram_turns(tb); ++r) {
    if (wave_ballot(open) == 0) return;
    int32_t* b = gram_bucket(gram, gh, r, tb);
    if (open && b[0] < kBucketSlots) {
      const int32_t c = atomicAdd(b, 1);
      if (c < kBucketSlots) {
        b[1 + c] = posting;
        open = false;
      }
    }
  }
  file_groups(kNear + 3u, 1);
}

template <bool FUZZY, int QC>
__global__ __launch_bounds__(256) void bin_rest_kernel(IndexView ix, Bins b) {
  __shared__ int32_t before[kMostBins], first[kMostBins], part[256 / kWave];
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
  const int32_t p = (int32_t)blockIdx.x / kRestGroups, group = (int32_t)blockIdx.x - p * kRestGroups;
  for (int32_t x = group * 256 + tid; x < ix.N * ix.meta_stride; x += kRestGroups * 256)
    if (x % ix.meta_stride <= ix.tail_len) {
      const int64_t at = (int64_t)p * ix.N * ix.meta_stride + x;
      ix.meta_new[at] = b.ends[at];
    }
  if (__builtin_amdgcn_readfirstlane(b.over_used[1]) == 0) return;
  constexpr int kEach = kMostBins / 256;                 // consecutive bins of a thread
  int32_t counts[kEach], sum = 0;
#pragma unroll
  for (int y = 0; y < kEach; ++y) {
    const int32_t bin = tid * kEach + y;
    counts[y] = bin < b.bins ? b.over_count[(int64_t)p * b.bins + bin] : 0;
    first[bin] = bin < b.bins ? b.over_first[(int64_t)p * b.bins + bin] : 0;
    sum += counts[y];
  }
  int32_t total, at = block_prefix<256>(sum, part, tid, total);
#pragma unroll
  for (int y = 0; y < kEach; ++y) {
    before[tid * kEach + y] = at;
    at += counts[y];
  }
  __syncthreads();
  int32_t* gram = ix.gram + (int64_t)p * ((int64_t)ix.buckets.mask + 1) * kBucketWords;
  // few to a wave where there are few: what a chain's first buckets do not take a wave files one by one
  constexpr int32_t kWaves = kRestGroups * (256 / kWave);
  int32_t each = (total + kWaves - 1) / kWaves;
  each = each < kWave ? each : kWave;
  for (int32_t f0 = (group * (256 / kWave) + (tid >> 6)) * each; f0 < total; f0 += kWaves * each) {   // uniform over the wave
    const bool on = lane < each && f0 + lane < total;
    const int32_t f = on ? f0 + lane : f0, bin = last_not_above(before, f);
    const int32_t posting = b.over[first[bin] + (f - before[bin])];
    const int32_t v = FUZZY ? posting >> kVariantShift : 0;
    const int32_t pos = FUZZY ? posting & ((1 << kVariantShift) - 1) : posting;
    const int32_t e = pos & ((1 << ix.eshift) - 1);
    const int32_t* tok = ix.tok + ((int64_t)p * ix.N + (pos >> ix.eshift)) * ix.max_len;
    int32_t G[QC];
#pragma unroll
    for (int a = 0; a < QC; ++a) G[a] = tok[e - 1 - (a < ix.kmax ? a : 0)];
    file_along_chain(gram, ix.buckets, variant_hash(G, ix.kmax, v), posting, on, lane);
  }
}

}  // namespace csd
