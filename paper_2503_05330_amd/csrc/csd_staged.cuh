// csd — a replay of many small problems in one launch: a workgroup has a problem's histories in LDS.
//
// As launches for the append, the quads of lanes, the eights and the rows left over, every draft gathers its
// bucket, its postings' tokens and its matches' continuations from memory, all problems at once: out of the L2
// between one use of a line and the next (1024 problems of 16 x 1024 positions, 24 steps: 37 + 58 + 58 + 45 us
// for 134 MB of histories).  Here a workgroup reads its problem's histories once, as a stream.  It has its rows'
// queries (a row: a path at a step) in a hash table in LDS and passes all positions by it, so no row follows a
// chain of the index (a fourth of the first buckets are full); the index gets the postings of the new positions,
// whose round trips travel meanwhile.  Rows are then walked class by class, as many to a wave as their matches
// leave room for.  us, the launches before / this: 64 problems x 48 steps 46 / 28 + 4, 1024 x 24 steps 198 / 132 + 5
// (the launch for the rows left over, of which there are hardly any).  What bounds it is what a workgroup does
// one after the other, with a CU to itself (medians of 64 problems, 192 rows, and 1024, 384 rows): histories
// 3.9, 6.6 us, positions by the table 6.9, 8.3 (half of it hashing), classes 1.2, walks 6.7, 9.2, the rest 2.5.
// Steps to it: the look-up by quads in the index, sixteen lanes for chains 26 + 13 and 136 + 22; all candidates
// at once where they are found, a wave's 9.4 for 6.9; walks in loops over the layers instead of unrolled 31 for 26.
#pragma once

#include "csd_kernels.cuh"

namespace csd {

constexpr int kStagedThreads = 1024, kStagedWaves = kStagedThreads / kWave;
constexpr int32_t kStagedCells = 1 << 14;      // positions of a problem at most: 128 KB with their probabilities
constexpr int32_t kStagedPaths = 256;
constexpr int32_t kStagedRows = 384;           // rows that a workgroup drafts at most
constexpr int32_t kStagedMatches = 256;        // most matches of a row (four a lane of a wave)
constexpr int32_t kStagedMost = 3072;          // matches of all its rows that are listed (beyond, twice as many are placed)
constexpr int32_t kStagedGiveUp = 1 << 14;     // matches of all its rows beyond which they are all left over
constexpr int32_t kStagedHuge = 2 * kStagedWaves;   // rows of more than a wave's worth of matches that it drafts
constexpr int32_t kStagedLeft = 0xFFFF;        // matches of a row that is left over (no row has as many)
constexpr int32_t kStagedCandidates = 2048, kStagedNone = 0xFFFF;
constexpr int kRowBits = 9;                    // of a row's number in an entry of the table or of a list
static_assert(kStagedRows < 1 << kRowBits, "a row's number, and one more");

// A path's cells in LDS.
__host__ __device__ __forceinline__ int32_t staged_stride(int32_t max_len) { return (max_len + 3) & ~3; }

// Rows by their matches: more than sixteen, up to sixteen, eight, four, two, one.
enum StagedClass { kMany, kSixteen, kEight, kFour, kTwo, kOne, kStagedClasses };
__device__ __forceinline__ constexpr int staged_rows_at_once(int c) {   // rows of a class that a wave takes
  return c == kMany ? 1 : c == kSixteen ? 4 : c == kEight || c == kOne ? 8 : c == kFour ? 16 : 32;
}

struct __align__(16) LdsStaged {
  static constexpr int kFront = CSD_MAX_QUERY_LEN, kBehind = 16;   // cells that a gram and a window may read beyond
  static constexpr int kSlotsLog2 = 11;
  static constexpr uint32_t kMore = 1u << kRowBits, kTag = ~(2u * kMore - 1u), kNone = ~0u;
  int32_t tok[kFront + kStagedCells + kBehind];
  uint32_t pq[kStagedCells + kBehind];
  // the queries: hash (its high bits: the slot) | others are chained behind | row; kNone: no query
  union {
    uint32_t table[1 << kSlotsLog2];
    uint16_t found[kStagedMost];               // afterwards: packed positions of the matches, row by row
  };
  uint16_t next[kStagedRows];                  // the row chained behind this one, or kStagedRows
  uint16_t first[kStagedRows];                 // place of the row's first match
  uint32_t matches[kStagedMost];               // (half of) the rows' matches, as found: packed position | number of the row's matches before it | row
  int32_t n_found[kStagedRows];
  uint16_t lists[3][kStagedRows];              // number of the row, up to sixteen matches above; two classes a list, from its ends
  uint16_t rest[kStagedRows];
  int32_t len[kStagedPaths];                   // lengths before the call
  uint16_t candidates[kStagedCandidates];      // packed positions whose gram may be a query
  int32_t count[kStagedClasses], n_rest, n_candidates, n_matches, n_placed, n_huge, last;
  __device__ __forceinline__ uint16_t& listed(int of_class, int32_t at) {
    const int list = of_class <= kSixteen ? 0 : of_class == kEight || of_class == kOne ? 1 : 2;
    return lists[list][of_class == kMany || of_class == kEight || of_class == kFour ? at : kStagedRows - 1 - at];
  }
};
static_assert(sizeof(LdsStaged) <= 160 * 1024, "the LDS of a CU");

// n of a counter for the whole wave, by its first lane.  (A condition that the compiler cannot know: where a
// loop's turn ended in another `lane == 0`, it took the other lanes round the loop without the first.)
__device__ __forceinline__ int32_t wave_reserve(int32_t* counter, int32_t n, int lane) {
  int32_t at = 0;
  consume_here(lane);
  if (lane == 0) at = atomicAdd(counter, n);
  return __builtin_amdgcn_readfirstlane(at);
}

// Hash of the newest kmax of the QC tokens, for the table of queries alone: four instructions a token.
template <int QC>
__device__ __forceinline__ uint32_t query_hash_of(const int32_t (&Q)[QC], int32_t kmax) {
  uint32_t acc = kGramSeed;
#pragma unroll
  for (int x = 0; x < QC; ++x)
    if (x < kmax) {                                      // (uniform over the launch)
      acc ^= acc >> 15;
      acc = __umul24((uint32_t)Q[x], 0x9E3779u) + __builtin_rotateleft32(acc, 11);
    }
  return acc * 0xC2B2AE35u;
}

// A match's continuation in LDS.
struct StagedWindow {
  const int32_t* tok;
  const uint32_t* pq;
  int32_t rem;                                 // layers that it reaches, at most L
};

// The walk of a row by a wave, S matches a lane: a layer's successors one after the other.
template <int S, bool EDGE>
__device__ __forceinline__ DraftOut staged_wave_walk(const DraftArgs& a, const StagedWindow (&w)[S], int lane) {
  DraftOut o;
  int32_t cur = 0, ud[S], vd[S];
#pragma unroll
  for (int x = 0; x < S; ++x) ud[x] = 0;
  for (int32_t d = 1; d <= a.L; ++d) {                   // uniform over the wave
    u64 lives[S], from_cur[S], left[S], any = 0;
    uint32_t pd[S];
#pragma unroll
    for (int x = 0; x < S; ++x) {
      vd[x] = w[x].tok[d - 1];
      pd[x] = w[x].pq[d - 1];
      lives[x] = wave_ballot(d <= w[x].rem);
      left[x] = from_cur[x] = d == 1 ? lives[x] : lives[x] & wave_ballot(ud[x] == cur);
      any |= from_cur[x];
    }
    if (any == 0) break;                                 // a leaf
    Cand best = cand_none();
#pragma unroll
    for (int y = 0; y < S; ++y)
      while (left[y]) {                                  // uniform over the wave
        const int32_t token = __builtin_amdgcn_readlane(vd[y], (int)__ffsll((long long)left[y]) - 1);
        uint32_t count = 0, sum = 0;
#pragma unroll
        for (int x = 0; x < S; ++x) {
          const u64 equal = wave_ballot(vd[x] == token), same = equal & (EDGE ? from_cur[x] : lives[x]);
          left[x] &= ~equal;
          count += (uint32_t)__popcll(same);
          sum += lanes_of(same, pd[x]);
        }
        best = cand_best(best, Cand{weight_key(pack_cs(count, wave_sum(sum)), a.alpha_q), token});
      }
    cur = best.v;
    o.tok = lane == d - 1 ? best.v : o.tok;
    o.key = lane == d - 1 ? best.key : o.key;
    o.key_sum += best.key;
    o.n = d;
#pragma unroll
    for (int x = 0; x < S; ++x) ud[x] = vd[x];
  }
  return o;
}

struct StagedArgs {
  IndexView ix;                 // meta_old: the paths' ends before the call, meta_new: after it (may be the same)
  ReplayIn in;
  int32_t shares;               // workgroups of a problem
  int32_t* step_meta;           // [steps][P][N][meta_stride]: ends after each step, for the rows left over
  int32_t* done;                // see append_kernel; the line of a problem's first row counts its shares
  DraftArgs a;
  RestList list;
};

// KMAX: length of a gram, or 0: up to eight tokens, at run time.
template <int LCAP, int KMAX, bool EDGE>
__global__ __launch_bounds__(kStagedThreads) void replay_staged_kernel(StagedArgs args) {
  constexpr int QC = KMAX > 0 ? KMAX : CSD_MAX_QUERY_LEN, kWords = (QC + 3) & ~3;
  __shared__ LdsStaged s;
  const IndexView& ix = args.ix;
  const DraftArgs& a = args.a;
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t xcd = blockIdx.x & 7;
  const int32_t shares = args.shares, number = (int32_t)(xcd * (gridDim.x >> 3) + (blockIdx.x >> 3)), p = number / shares;
  const int32_t N = ix.N, L = a.L, max_len = ix.max_len, kmax = KMAX > 0 ? KMAX : ix.kmax;
  const int32_t of_problem = args.in.steps * N, per = (of_problem + shares - 1) / shares;
  const int32_t first = (number - p * shares) * per;     // of the problem's rows
  const int32_t n_rows = first + per < of_problem ? per : of_problem - first;
  if (p >= ix.P || n_rows <= 0) return;                  // uniform over the workgroup (the host leaves no share without rows)
  const int32_t stride = staged_stride(max_len), e_mask = (1 << ix.eshift) - 1;
  const int32_t steps = (first + n_rows - 1) / N + 1;    // that the workgroup's rows see
  const int64_t rows = (int64_t)ix.P * N;

  struct Row {                                           // path, step, row among all steps' rows
    int32_t i, t, out;
  };
  auto row_of = [&](int32_t nth) {
    Row r;
    r.t = (int32_t)((uint32_t)(first + nth) / (uint32_t)N);
    r.i = first + nth - r.t * N;
    r.out = (r.t * ix.P + p) * N + r.i;
    return r;
  };
  auto length_at = [&](int32_t j, int32_t t) {           // after step t
    const int32_t grown = s.len[j] + t + 1;
    return grown < max_len ? grown : max_len;
  };
  auto cell_of = [&](int32_t j, int32_t e) { return (int32_t)__umul24((uint32_t)j, (uint32_t)stride) + e; };
  // the QC tokens before index e of path j, newest first (fewer than kmax exist: others' cells)
  auto tokens_before = [&](int32_t j, int32_t e, int32_t (&t)[QC]) {
    const int32_t* before = s.tok + LdsStaged::kFront + cell_of(j, e);
#pragma unroll
    for (int x = 0; x < QC; ++x) t[x] = before[-1 - x];
  };
  auto differ = [&](const int32_t (&t)[QC], const int32_t (&q)[QC]) {
    int32_t d = 0;
#pragma unroll
    for (int x = 0; x < QC; ++x) d |= x < kmax ? t[x] ^ q[x] : 0;
    return d != 0;
  };

  // ---- the paths' lengths, the new tokens and the histories
  const int32_t n_new = steps * N;
  auto new_cell = [&](int32_t x) {                       // new token x of the problem in the step's input
    const int32_t t = (int32_t)((uint32_t)x / (uint32_t)N);
    return (int64_t)t * rows + (int64_t)p * N + (x - t * N);
  };
  int32_t new_tok = 0;
  float new_prob = 1.0f;
  if (tid < n_new) {
    new_tok = args.in.tok[new_cell(tid)];
    if (args.in.prob) new_prob = args.in.prob[new_cell(tid)];
  }
  if (tid < N) s.len[tid] = ix.meta_old[((int64_t)p * N + tid) * ix.meta_stride];
  for (int32_t x = tid; x < 1 << LdsStaged::kSlotsLog2; x += kStagedThreads) s.table[x] = LdsStaged::kNone;
  if (tid < kStagedRows) s.n_found[tid] = 0;
  if (tid < kStagedClasses) s.count[tid] = 0;
  if (tid == 0) s.n_rest = s.n_candidates = s.n_matches = s.n_placed = s.n_huge = 0;
  lds_barrier<kStagedThreads>();
  const int32_t per_path = (stride + 255) / 256, chunks = N * per_path;   // a chunk: 256 cells of a path, four a lane
  constexpr int kAtOnce = 4;
  for (int32_t c0 = wave; c0 < chunks; c0 += kAtOnce * kStagedWaves) {   // uniform over the wave
    Run4 tok[kAtOnce], pq[kAtOnce];
    int32_t to[kAtOnce];
#pragma unroll
    for (int x = 0; x < kAtOnce; ++x) {
      const int32_t c = c0 + x * kStagedWaves, j = c < chunks ? c / per_path : 0, at = (c - j * per_path) * 256 + 4 * lane;
      const bool on = c < chunks && at < s.len[j];
      to[x] = on ? cell_of(j, at) : -1;
      const int64_t from = (int64_t)(p * N + j) * max_len + (on ? at : 0);
      tok[x] = *reinterpret_cast<const Run4*>(ix.tok + from);
      pq[x] = *reinterpret_cast<const Run4*>(ix.pq + from);
    }
#pragma unroll
    for (int x = 0; x < kAtOnce; ++x)
      if (to[x] >= 0) {
        *reinterpret_cast<int4*>(s.tok + LdsStaged::kFront + to[x]) = int4{tok[x].x[0], tok[x].x[1], tok[x].x[2], tok[x].x[3]};
        *reinterpret_cast<int4*>(s.pq + to[x]) = int4{pq[x].x[0], pq[x].x[1], pq[x].x[2], pq[x].x[3]};
      }
  }
  lds_barrier<kStagedThreads>();                         // (a path's last four cells may hold what lay behind its end)
  for (int32_t x = tid; x < n_new; x += kStagedThreads) {
    if (x >= kStagedThreads) {
      new_tok = args.in.tok[new_cell(x)];
      if (args.in.prob) new_prob = args.in.prob[new_cell(x)];
    }
    const int32_t t = (int32_t)((uint32_t)x / (uint32_t)N), i = x - t * N, e = s.len[i] + t;
    if (e >= max_len) continue;
    const uint32_t q = args.in.prob ? quantize_prob(new_prob) : 65536u;
    s.tok[LdsStaged::kFront + cell_of(i, e)] = new_tok;
    s.pq[cell_of(i, e)] = q;
    if (x >= first && x < first + n_rows) {              // the share's own are appended by it
      const int64_t to = (int64_t)(p * N + i) * max_len + e;
      ix.tok[to] = new_tok;
      ix.pq[to] = q;
    }
  }
  lds_barrier<kStagedThreads>();

  // ---- a thread a row: its query to the table, its new position to the index, the path's end
  int32_t signed_off = 0;
  if (shares > 1 && tid == 0) signed_off = atomicAdd(&args.done[(int64_t)p * N * kBucketWords], 1);   // (the old ends have been read)
  Filing<QC> filing;
  const bool has_row = tid < n_rows;
  bool leave = false;
  uint32_t flags = 0;
  if (wave * kWave < n_rows) {                           // uniform over the wave
    const Row r = row_of(has_row ? tid : 0);
    const int32_t old = s.len[r.i], len = length_at(r.i, r.t), e = old + r.t;
    const bool appended = has_row && e < max_len;
    int32_t Q[QC], G[QC];
    tokens_before(r.i, len, Q);
    tokens_before(r.i, e < max_len ? e : 0, G);
    // (no home blocks: an index has them from 12 positions a bucket on, eight is what its buckets are for)
    filing.claim(ix.gram + (int64_t)p * ((int64_t)ix.buckets.mask + 1) * kBucketWords, Buckets{ix.buckets.mask, ix.buckets.mask}, kmax, G,
                 appended && e >= kmax, (r.i << ix.eshift) | e);
    if (has_row) flags = !appended ? CSD_STATUS_CAPACITY : (Q[0] < 0 || Q[0] >= ix.vocab) ? CSD_STATUS_TOKEN_RANGE : 0u;
    leave = has_row && len < kmax;                       // no gram to look for: scanned for by a wave
    if (has_row && !leave) {
      const uint32_t h = query_hash_of(Q, kmax);
      uint32_t* slot = &s.table[h >> (32 - LdsStaged::kSlotsLog2)];
      const uint32_t before = atomicExch(slot, (h & LdsStaged::kTag) | (uint32_t)tid);
      s.next[tid] = (uint16_t)(before == LdsStaged::kNone ? kStagedRows : before & (LdsStaged::kMore - 1u));
      if (before != LdsStaged::kNone) atomicOr(slot, LdsStaged::kMore);   // (whichever row is the slot's by now)
    }
    if (has_row) {
      int32_t* end = args.step_meta + (int64_t)r.out * ix.meta_stride;
      int32_t w[12];
#pragma unroll
      for (int x = 0; x < 12; ++x)
        w[x] = x == 0 ? len : (x - 1 < (QC < 11 ? QC : 11) && x - 1 < ix.tail_len && x - 1 < len) ? Q[x - 1 < QC ? x - 1 : 0] : 0;
#pragma unroll
      for (int x = 0; x < 12; x += 4)
        if (x < ix.meta_stride) *reinterpret_cast<int4*>(end + x) = int4{w[x], w[x + 1], w[x + 2], w[x + 3]};
    }
  }
  lds_barrier<kStagedThreads>();

  // ---- all positions by the table of queries: those whose gram may be one are listed
  auto rows_of = [&](int32_t j, int32_t e, auto&& match) {   // the rows that a position matches; e < 0: none
    int32_t g[QC];
    tokens_before(j, e < 0 ? 0 : e, g);
    const uint32_t h = query_hash_of(g, kmax);
    int32_t nth = e < 0 ? kStagedRows : (int32_t)(s.table[h >> (32 - LdsStaged::kSlotsLog2)] & (LdsStaged::kMore - 1u));
    while (wave_ballot(nth < kStagedRows) != 0) {        // uniform over the wave
      const bool is_row = nth < kStagedRows;
      const Row r = row_of(is_row ? nth : 0);
      int32_t q[QC];
      tokens_before(r.i, length_at(r.i, r.t), q);
      match(is_row && j != r.i && e < length_at(j, r.t) && !differ(g, q), nth);
      nth = is_row ? s.next[nth] : kStagedRows;
    }
  };
  auto candidate = [&](int32_t j, int32_t e) {
    rows_of(j, e, [&](bool is_match, int32_t nth) {
      int32_t n = kStagedMatches;
      if (is_match) n = atomicAdd(&s.n_found[nth], 1);
      const u64 hits = wave_ballot(n < kStagedMatches);
      if (hits == 0) return;                             // uniform over the wave
      const int32_t at = wave_reserve(&s.n_matches, (int32_t)__popcll(hits), lane) + (int32_t)__popcll(hits & ((1ull << lane) - 1ull));
      if (n < kStagedMatches && at < kStagedMost) s.matches[at] = (uint32_t)((j << ix.eshift) | e) << 17 | (uint32_t)(n << kRowBits) | (uint32_t)nth;
    });
  };
  constexpr int kEach = 8;                               // consecutive positions of a lane
  const int32_t spans_of_path = (stride + kEach * kWave - 1) / (kEach * kWave);
  auto given_up = [&]() {                                // too many matches: all rows are left over
    return __builtin_amdgcn_readfirstlane(*(volatile int32_t*)&s.n_matches) > kStagedGiveUp;
  };
  auto stream = [&](auto&& take) {
    for (int32_t c = wave; c < N * spans_of_path && !given_up(); c += kStagedWaves) {   // uniform over the wave
      const int32_t j = c / spans_of_path, e0 = ((c - j * spans_of_path) * kWave + lane) * kEach, end = length_at(j, steps - 1);
      if (e0 - kEach * lane >= end) continue;              // uniform over the wave
      const int32_t* at = s.tok + LdsStaged::kFront + cell_of(j, e0 < end ? e0 : 0);
      int32_t w[kWords + kEach];                           // tokens e0 - kWords and on (the last is not looked at)
#pragma unroll
      for (int x = 0; x < kWords + kEach; x += 4) {
        const int4 r = *reinterpret_cast<const int4*>(at - kWords + x);
        w[x] = r.x;
        w[x + 1] = r.y;
        w[x + 2] = r.z;
        w[x + 3] = r.w;
      }
      uint32_t todo = 0, h[kEach], entry[kEach];
#pragma unroll
      for (int r = 0; r < kEach; ++r) {
        int32_t g[QC];
#pragma unroll
        for (int x = 0; x < QC; ++x) g[x] = w[kWords + r - 1 - x];
        h[r] = query_hash_of(g, kmax);
        entry[r] = s.table[h[r] >> (32 - LdsStaged::kSlotsLog2)];
      }
#pragma unroll
      for (int r = 0; r < kEach; ++r) {
        const bool may = entry[r] != LdsStaged::kNone && ((entry[r] & LdsStaged::kMore) != 0 || ((entry[r] ^ h[r]) & LdsStaged::kTag) == 0);
        todo |= may && e0 + r >= kmax && e0 + r < end ? 1u << r : 0u;
      }
      if (wave_ballot(todo != 0) != 0) take(j, e0, todo);  // uniform over the wave
    }
  };
  stream([&](int32_t j, int32_t e0, uint32_t todo) {
    const uint32_t up_to = wave_prefix(__popc(todo));    // candidates of the lanes up to this one
    const int32_t total = __builtin_amdgcn_readlane((int)up_to, kWave - 1);
    int32_t to = wave_reserve(&s.n_candidates, total, lane);
    if (to + total <= kStagedCandidates) {               // uniform over the wave
      to += (int32_t)up_to - __popc(todo);
      for (; todo != 0; todo &= todo - 1u) s.candidates[to++] = (uint16_t)((j << ix.eshift) | (e0 + __ffs(todo) - 1));
    } else {                                             // no room: at once
      for (int32_t x = to + lane; x < kStagedCandidates; x += kWave) s.candidates[x] = kStagedNone;
      while (wave_ballot(todo != 0) != 0) {              // uniform over the wave
        candidate(j, todo != 0 ? e0 + __ffs(todo) - 1 : -1);
        todo &= todo - 1u;                               // 0 stays 0
      }
    }
  });
  lds_barrier<kStagedThreads>();
  const int32_t n_listed = __builtin_amdgcn_readfirstlane(s.n_candidates);
  const int32_t n_candidates = n_listed < kStagedCandidates ? n_listed : kStagedCandidates;
  for (int32_t x0 = wave * kWave; x0 < n_candidates && !given_up(); x0 += kStagedThreads) {   // uniform over the wave
    const int32_t pos = x0 + lane < n_candidates ? s.candidates[x0 + lane] : kStagedNone;
    candidate(pos != kStagedNone ? pos >> ix.eshift : 0, pos != kStagedNone ? pos & e_mask : -1);
  }
  lds_barrier<kStagedThreads>();

  // ---- the rows' classes, and where their matches go
  filing.settle();
  const int32_t n_matches = __builtin_amdgcn_readfirstlane(s.n_matches);
  const bool again = n_matches > kStagedMost;            // more than the list holds: the candidates a second time
  const int32_t most = again ? 2 * kStagedMost : kStagedMost;
  uint16_t* found = again ? reinterpret_cast<uint16_t*>(s.matches) : s.found;   // (the table is asked again)
  if (wave * kWave < n_rows) {                           // uniform over the wave
    auto before = [&](u64 mask) { return (int32_t)__popcll(mask & ((1ull << lane) - 1ull)); };
    int32_t M = has_row && !leave ? s.n_found[tid] : 0;
    leave = leave || M > kStagedMatches || (has_row && n_matches > kStagedGiveUp);
    // of the rows that take a wave several matches a lane, a few; of all, those whose matches have room
    const u64 huge = wave_ballot(!leave && M > kWave);
    if (huge) {                                          // uniform over the wave
      const int32_t at = wave_reserve(&s.n_huge, (int32_t)__popcll(huge), lane) + before(huge);
      leave = leave || (M > kWave && at >= kStagedHuge);
    }
    M = leave ? 0 : M;
    const uint32_t up_to = wave_prefix((uint32_t)M);
    const int32_t first_of = wave_reserve(&s.n_placed, __builtin_amdgcn_readlane((int)up_to, kWave - 1), lane) + (int32_t)up_to - M;
    leave = leave || (M > 0 && first_of + M > most);     // (a lane without a row has none, wherever its wave's part ends)
    if (leave) s.n_found[tid] = kStagedLeft;
    if (leave) s.rest[atomicAdd(&s.n_rest, 1)] = (uint16_t)tid;
    if (has_row) s.first[tid] = (uint16_t)first_of;
    const bool drafts = has_row && !leave;
    const u64 in_class[kStagedClasses] = {wave_ballot(drafts && M > 16),          wave_ballot(drafts && M > 8 && M <= 16),
                                          wave_ballot(drafts && M > 4 && M <= 8), wave_ballot(drafts && M > 2 && M <= 4),
                                          wave_ballot(drafts && M == 2),          wave_ballot(drafts && M <= 1)};
    int32_t n = 0, of_class = 0, at = 0;                 // (a lane reserves for a class)
    u64 members = 0;
#pragma unroll
    for (int c = 0; c < kStagedClasses; ++c) {
      n = lane == c ? (int32_t)__popcll(in_class[c]) : n;
      const bool is_of = (in_class[c] >> lane & 1ull) != 0;
      of_class = is_of ? c : of_class;
      members = is_of ? in_class[c] : members;
    }
    if (n > 0) at = atomicAdd(&s.count[lane], n);
    at = __shfl(at, of_class) + before(members);
    if (drafts) s.listed(of_class, at) = (uint16_t)(tid | (M <= 16 ? M : 0) << kRowBits);
  }
  lds_barrier<kStagedThreads>();
  if (!again) {
    for (int32_t x = tid; x < n_matches; x += kStagedThreads) {
      const uint32_t m = s.matches[x], nth = m & ((1u << kRowBits) - 1u);
      if (s.n_found[nth] <= kStagedMatches) found[s.first[nth] + (m >> kRowBits & 255u)] = (uint16_t)(m >> 17);
    }
  } else if (n_matches <= kStagedGiveUp) {
    auto place = [&](int32_t j, int32_t e) {
      constexpr int kPlaced = 16;                        // (above the row's count: its matches that have their place)
      rows_of(j, e, [&](bool is_match, int32_t nth) {
        if (is_match && (s.n_found[nth] & kStagedLeft) <= kStagedMatches)
          found[s.first[nth] + (atomicAdd(&s.n_found[nth], 1 << kPlaced) >> kPlaced)] = (uint16_t)((j << ix.eshift) | e);
      });
    };
    if (n_listed <= kStagedCandidates)
      for (int32_t x0 = wave * kWave; x0 < n_candidates; x0 += kStagedThreads) {   // uniform over the wave
        const int32_t pos = x0 + lane < n_candidates ? s.candidates[x0 + lane] : kStagedNone;
        place(pos != kStagedNone ? pos >> ix.eshift : 0, pos != kStagedNone ? pos & e_mask : -1);
      }
    else
      stream([&](int32_t j, int32_t e0, uint32_t todo) {
        while (wave_ballot(todo != 0) != 0) {            // uniform over the wave
          place(j, todo != 0 ? e0 + __ffs(todo) - 1 : -1);
          todo &= todo - 1u;                             // 0 stays 0
        }
      });
  }
  lds_barrier<kStagedThreads>();

  // ---- the rows with more matches than are drafted here, or fewer tokens than a gram: listed for a wave each
  const int32_t n_rest = __builtin_amdgcn_readfirstlane(s.n_rest);
  if (n_rest > 0 && wave == kStagedWaves - 1) {          // uniform over the wave
    const int32_t to = wave_reserve(args.list.count(xcd, true), n_rest, lane);
    for (int32_t x = lane; x < n_rest; x += kWave) *args.list.unit(xcd, true, to + x) = p * of_problem + first + (int32_t)s.rest[x];
  }

  // ---- the walks, class by class, a wave's turn at a time
  auto load_targets = [&](const Row& r, int sub, auto& target) {   // of the layers that the lane keeps
    constexpr int kKept = sizeof(target) / sizeof(int32_t);
#pragma unroll
    for (int x = 0; x < kKept; ++x) {
      const int32_t d = sub * kKept + x;
      target[x] = a.targets ? a.targets[(int64_t)r.out * L + (d < L ? d : 0)] : 0;
    }
  };
  auto window = [&](const Row& r, bool on, int32_t pos) {   // (a lane without a match: the first cell's)
    const int32_t j = on ? pos >> ix.eshift : 0, e = on ? pos & e_mask : 0;
    const int32_t rem = length_at(j, r.t) - e, cell = cell_of(j, e);
    return StagedWindow{s.tok + LdsStaged::kFront + cell, s.pq + cell, on ? (rem < L ? rem : L) : 0};
  };
  int32_t count[kStagedClasses];
#pragma unroll
  for (int c = 0; c < kStagedClasses; ++c) count[c] = __builtin_amdgcn_readfirstlane(s.count[c]);
  for (int32_t nth_turn = wave;; nth_turn += kStagedWaves) {   // uniform over the wave
    int32_t turn = nth_turn;
    int c = 0;
#pragma unroll
    for (int x = 0; x < kStagedClasses; ++x) {
      const int32_t turns = (count[x] + staged_rows_at_once(x) - 1) / staged_rows_at_once(x);
      if (c == x && turn >= turns) {
        turn -= turns;
        ++c;
      }
    }
    if (c == kStagedClasses) break;
    auto listed = [&](auto lanes, int of_class) {        // a row by G lanes with a match each
      constexpr int G = lanes();
      const int32_t x = turn * (kWave / G) + lane / G, sub = lane & (G - 1);
      const bool on = x < count[of_class];
      const int32_t entry = s.listed(of_class, on ? x : 0), nth = entry & ((1 << kRowBits) - 1);
      const Row r = row_of(nth);
      int32_t target[GroupDraft<G, LCAP>::kKept], v[LCAP], pr[LCAP];
      load_targets(r, sub, target);
      const bool has = on && sub < entry >> kRowBits;
      const StagedWindow w = window(r, has, found[has ? s.first[nth] + sub : 0]);
#pragma unroll
      for (int d = 0; d < LCAP; ++d) {
        v[d] = w.tok[d];
        pr[d] = (int32_t)w.pq[d];
      }
      GroupDraft<G, LCAP> draft;
      group_walk<G, LCAP, EDGE>(a, (uint32_t)w.rem << 25, v, pr, on,
                                [&](auto layer, bool going, const Cand& best) { draft.choose(layer(), going, best, sub); });
      draft.store(a, r.out, on, sub, target);
    };
    if (c == kFour) listed(std::integral_constant<int, 4>{}, kFour);
    else if (c == kTwo) listed(std::integral_constant<int, 2>{}, kTwo);
    else if (c == kEight) listed(std::integral_constant<int, 8>{}, kEight);
    else if (c == kSixteen) listed(std::integral_constant<int, 16>{}, kSixteen);
    else if (c == kOne) {                                // its continuation, if any, is the draft
      constexpr int G = 8, kKept = GroupDraft<G, LCAP>::kKept;
      const int32_t x = turn * (kWave / G) + lane / G, sub = lane & (G - 1);
      const bool on = x < count[kOne];
      const int32_t entry = s.listed(kOne, on ? x : 0), nth = entry & ((1 << kRowBits) - 1);
      const Row r = row_of(nth);
      int32_t target[kKept];
      load_targets(r, sub, target);
      const bool has = entry >> kRowBits != 0;
      const StagedWindow w = window(r, has, found[has ? s.first[nth] : 0]);
      GroupDraft<G, LCAP> draft;
      draft.n = w.rem;
      uint32_t sum = 0;
#pragma unroll
      for (int y = 0; y < kKept; ++y) {
        const int32_t d = sub * kKept + y;
        const int32_t tok = w.tok[d];
        const uint32_t pq = w.pq[d];
        const bool in = d < w.rem;
        draft.tok[y] = in ? tok : -1;
        draft.key[y] = in ? weight_key(pack_cs(1u, pq), a.alpha_q) : 0ull;
        sum += in ? pq : 0u;
      }
      group_stages<G>([&](auto move) { sum += move(sum); });
      draft.key_sum = weight_key(pack_cs((uint32_t)w.rem, sum), a.alpha_q);
      draft.store(a, r.out, on, sub, target);
    } else {                                             // the wave
      const int32_t nth = s.listed(kMany, turn) & ((1 << kRowBits) - 1), M = __builtin_amdgcn_readfirstlane(s.n_found[nth]) & kStagedLeft;
      const Row r = row_of(nth);
      const int32_t target = a.targets ? a.targets[(int64_t)r.out * L + (lane < L ? lane : 0)] : 0;
      auto walk = [&](auto n) {
        constexpr int S = n();
        StagedWindow w[S];
#pragma unroll
        for (int x = 0; x < S; ++x) {
          const bool has = lane + x * kWave < M;
          w[x] = window(r, has, found[has ? s.first[nth] + lane + x * kWave : 0]);
        }
        return staged_wave_walk<S, EDGE>(a, w, lane);
      };
      const DraftOut o = M <= kWave ? walk(std::integral_constant<int, 1>{})
                                    : walk(std::integral_constant<int, kStagedMatches / kWave>{});
      write_outputs<kWave>(a, r.out, o, lane);
      if (a.targets) write_accept(a, r.out, o, target, lane);
    }
  }
  filing.finish();

  // ---- the paths' ends, by the share that has read the old ones last
  if (flags) atomicOr(ix.status, flags);
  if (shares > 1) {
    if (tid == 0) s.last = signed_off == shares - 1;
    lds_barrier<kStagedThreads>();
    if (!s.last) return;                                 // uniform over the workgroup
    if (tid == 0) args.done[(int64_t)p * N * kBucketWords] = 0;
  }
  for (int32_t x = tid; x < N * ix.meta_stride; x += kStagedThreads) {
    const int32_t i = x / ix.meta_stride, w = x - i * ix.meta_stride, len = length_at(i, args.in.steps - 1), a = w - 1;
    int32_t word = w == 0 ? len : 0;
    if (a >= 0 && a < ix.tail_len && a < len) {
      const int32_t e = len - 1 - a, old = s.len[i];     // (the share may not have the last steps' tokens on chip)
      word = e < old ? s.tok[LdsStaged::kFront + cell_of(i, e)] : args.in.tok[(int64_t)(e - old) * rows + (int64_t)p * N + i];
    }
    ix.meta_new[((int64_t)p * N) * ix.meta_stride + x] = word;
  }
}

}  // namespace csd
