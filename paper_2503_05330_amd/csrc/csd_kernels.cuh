// csd — the kernels: reset, append, the decode step (a drafting and an
// appending wave per path in index mode, one 1024-thread workgroup per path —
// or several, sharing its scan — in scan mode), accept, the stand-in model of
// the accept-driven loop, and the kernels behind the debug dumps.
#pragma once

#include "csd_common.cuh"
#include "csd_dag.cuh"
#include "csd_index.cuh"
#include "csd_match.cuh"
#include "csd_quad.cuh"

namespace csd {

// Rows (problem, path) up to which several waves share the append of a path: more rows fill the chip
// with one each.
constexpr int64_t kSplitRows = 1 << 16;

// done (see append_kernel), counters (see RestList): null unless the handle is new.
static __global__ __launch_bounds__(256) void reset_kernel(IndexView ix, int64_t gram_words, ScanSlices sl,
                                                           int32_t* done, int32_t* counters) {
  int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * 256;
  int64_t rows = (int64_t)ix.P * ix.N;
  if (sl.n > 1)
    for (int64_t r = t; r < rows; r += stride) sl.state[r] = 0ull;
  for (int64_t r = t; r < rows * ix.meta_stride; r += stride) ix.meta_new[r] = 0;
  if (done)
    for (int64_t r = t; r < rows && r < kSplitRows; r += stride) done[r * kBucketWords] = 0;
  if (counters)
    for (int64_t w = t; w < RestList::kCounters; w += stride) counters[w] = 0;
  for (int64_t w = t; w < gram_words; w += stride) ix.gram[w] = (w & (kBucketWords - 1)) ? -1 : 0;
  if (t == 0) *ix.status = 0u;
}

// Append only, any number of tokens per path: `chunks` workgroups per (problem, path), a thread
// per new position.  The path's end is replaced in place (a captured launch goes on from where the
// one before it was) by the row's wave that reads the old end last, of those that have a position
// to append (another one finds nothing to do at the new end either).  done: for each row, a line
// apart, the waves that have read its end; 0 between launches.  They sign off while their claims are
// in flight: 64 paths x 4096 tokens take 22.5 us, with a second buffer for the new ends and no
// sign-off 21.7, with the counts of sixteen rows to a line 47 (an atomic takes a line of memory 12 ns).
// (scalar registers: with more of them a SIMD has seven waves, 4 problems of 64 x 2048 35 us for 34)
template <bool INDEX, bool FUZZY, int QC, bool LOOK = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_sgpr(96))) void append_kernel(IndexView ix, StepIn in, int32_t chunks, int32_t* done) {
  // (a problem's paths' first chunks, then their second ones: path by path, the workgroups without work, those behind a
  // count, would fall to the same XCDs: 64 paths, 1024 of 4096 offered taken of each 12.9 / 10.1 us, all 25.0 / 23.4; all
  // problems' first chunks first, 4 problems 40 for 34)
  const int32_t p = (int32_t)blockIdx.x / (ix.N * chunks), in_problem = (int32_t)blockIdx.x - p * (ix.N * chunks);
  const int32_t chunk = in_problem / ix.N, row = p * ix.N + (in_problem - chunk * ix.N), tid = (int32_t)threadIdx.x, lane = tid & (kWave - 1);
  const int32_t waves = chunks * (int32_t)(blockDim.x / kWave);   // of the row
  const int32_t wave = chunk * (int32_t)(blockDim.x / kWave) + (tid >> 6);
  int32_t before = -1, busy = 0, word = 0;               // before: waves that signed off earlier
  append_positions<INDEX, FUZZY, QC, LOOK>(
      ix, in, p, row - p * ix.N, chunk * (int32_t)blockDim.x, chunks * (int32_t)blockDim.x, chunk == 0, tid,
      [&](int32_t end, int32_t cnt) {
        const int32_t parts = (cnt + kWave - 1) / kWave;
        busy = __builtin_amdgcn_readfirstlane(parts < waves ? parts : waves);
        word = end;
        if (wave >= busy) return;
        if (busy == 1) store_end_word(ix, row, word, lane);
        else if (lane == 0) before = atomicAdd(&done[row * kBucketWords], 1);
      });
  if (busy > 1 && __builtin_amdgcn_readfirstlane(before) == busy - 1) {
    store_end_word(ix, row, word, lane);
    if (lane == 0) done[row * kBucketWords] = 0;
  }
}

// The same with one workgroup per problem, for batches of problems: slots are claimed on fill
// counts in LDS.  (Atomics on memory run at the memory's side of the fabric here, 1.1e10 per
// second whatever the addresses.)  maybe_empty: the caller has appended nothing since the reset;
// whether the index holds postings all the same (of a graph's appends) the paths' lengths tell, which
// arrive while the LDS is cleared.  With counts a problem that takes less than a posting per bucket
// files with atomics on memory after all (us, up to 16 tokens taken of those offered / half of them
// on average, without and with that: 1024 problems of 16 paths, 512 offered: 77, 26 / 82, 82; 128 of 64,
// 2048: 202, 21 / 405, 406; 4096 of 4, 128: 53, 32 / 55, 61).  TABLE: the buckets
// themselves are in LDS too, and go to memory as a whole.  BLOCKS: an index with home blocks (see Buckets).  The paths' ends are replaced in place, by
// way of `ends`, rows like theirs (1024 problems of 16 x 1024 tokens 110 .. 112 us; where `ends` stay the
// new ends 109; 114 to 118 by way of LDS, with a lane per word before or after the loop or with the
// tokens from the lanes that have them: registers and instructions of the loop are what counts here).
template <bool FUZZY, int QC, bool TABLE, bool BLOCKS>
__global__ __launch_bounds__(1024) void append_problem_kernel(IndexView ix, StepIn in, int32_t maybe_empty, int32_t* ends) {
  extern __shared__ int4 shared[];
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
  const int32_t p = (int32_t)blockIdx.x, n_buckets = (int32_t)ix.buckets.mask + 1;
  int32_t* gram = ix.gram + (int64_t)p * n_buckets * kBucketWords;
  int32_t* fill = reinterpret_cast<int32_t*>(shared);
  int4* table = shared + n_buckets / 4;                  // (at least 4 buckets)
  int32_t* slots = TABLE ? reinterpret_cast<int32_t*>(table) : gram;
  // a wave per run of 256 positions of a path, the next run's loads in flight
  constexpr int32_t kRun = 4 * kWave;
  const int32_t runs = (in.n + kRun - 1) / kRun;
  int32_t i = 0, run = __builtin_amdgcn_readfirstlane(tid >> 6);   // this wave's: path, run of it
  auto settle = [&]() {                                  // run number -> (path, run)
    while (run >= runs && i < ix.N) {
      run -= runs;
      ++i;
    }
  };
  settle();
  NewTokens4<QC> next;
  auto request = [&]() {
    if (i < ix.N) next.load(ix, in, (int64_t)p * ix.N + i, run * kRun, lane);   // uniform over the wave
  };
  request();
  if (in.counts) {                                       // (every wave adds them up for itself: no barrier)
    int32_t sum = 0;
    for (int32_t j = lane; j < ix.N; j += kWave) {
      const int32_t want = in.counts[(int64_t)p * ix.N + j];
      sum += want < 0 ? 0 : (want > in.n ? in.n : want);
    }
#pragma unroll
    for (int x = 1; x < kWave; x *= 2) sum += __shfl_xor(sum, x);
    if ((int64_t)__builtin_amdgcn_readfirstlane(sum) * (FUZZY ? ix.kmax + 1 : 1) < n_buckets) {
      for (int32_t j = __builtin_amdgcn_readfirstlane(tid >> 6); j < ix.N; j += 16)
        append_path<true, FUZZY, QC>(ix, in, p, j, kWave, lane);
      return;
    }
  }
  bool empty = false;
  if (maybe_empty) {                                     // uniform over the launch
    int32_t lens = 0;
    for (int32_t j = tid; j < ix.N; j += 1024) lens |= ix.meta_old[((int64_t)p * ix.N + j) * ix.meta_stride];
    if (TABLE)
      for (int32_t x = tid; x < n_buckets * 4; x += 1024) table[x] = int4{-1, -1, -1, -1};
    for (int32_t b = tid; b < n_buckets; b += 1024) fill[b] = 0;
    empty = __syncthreads_or(lens) == 0;
  }
  if (!empty) {                                          // (each thread the words that it has cleared)
    if (TABLE)
      for (int32_t x = tid; x < n_buckets * 4; x += 1024) table[x] = reinterpret_cast<const int4*>(gram)[x];
    for (int32_t b = tid; b < n_buckets; b += 1024) fill[b] = gram[b * kBucketWords];
    __syncthreads();
  }
  uint32_t flags = 0;
  while (i < ix.N) {
    const NewTokens4<QC> x = next;
    const int32_t path = i;
    const bool head = run == 0;
    run += 16;
    settle();
    request();
    const int64_t row = (int64_t)p * ix.N + path;
    const int32_t cnt = x.count(ix);
    flags |= x.store(ix, in, row, cnt);
    file_positions_own<FUZZY, QC, 4>(slots, fill, Buckets{ix.buckets.mask, BLOCKS ? ix.buckets.block : ix.buckets.mask}, ix.kmax, x.tok, x.filed(ix, cnt), x.pos(ix, path));
    if (head) {                                          // the path's first run
      if (lane == 0 && x.most() > cnt) flags |= CSD_STATUS_CAPACITY;
      store_end(ix, in, row, x.len, cnt, ends, lane);
    }
  }
  __syncthreads();                                       // everything has been claimed, the old ends read
  for (int32_t x = tid; x < ix.N * ix.meta_stride; x += 1024)
    if (x % ix.meta_stride <= ix.tail_len) {
      const int64_t at = (int64_t)p * ix.N * ix.meta_stride + x;
      ix.meta_new[at] = ends[at];
    }
  if (TABLE) {
    for (int32_t x = tid; x < n_buckets * 4; x += 1024) {
      int4 words = table[x];
      if ((x & 3) == 0) words.x = fill[x >> 2];
      reinterpret_cast<int4*>(gram)[x] = words;
    }
  } else {
    for (int32_t b = tid; b < n_buckets; b += 1024) gram[b * kBucketWords] = fill[b];
  }
  if (flags) atomicOr(ix.status, flags);
}

// Draft tokens, scores, length and (optionally) accept length of one row.
// `target` is the lane's target token (lanes < L), loaded by the caller.
template <int BLOCK>
__device__ __forceinline__ void write_outputs(const DraftArgs& a, int32_t row, const DraftOut& o,
                                              int tid) {
  const int32_t L = a.L;
  bool live = tid < o.n;
  if (tid < L) {
    a.draft_tokens[(int64_t)row * L + tid] = live ? o.tok : -1;
    if (a.token_scores) a.token_scores[(int64_t)row * L + tid] = live ? key_to_score(o.key) : 0.0f;
  }
  if (tid == 0) {
    a.draft_len[row] = o.n;
    if (a.path_scores) a.path_scores[row] = key_to_score(o.key_sum);
  }
}

// "Draft acceptance": the first lane whose draft token differs from its target.
// Returns the accept length (the same in every lane).
__device__ __forceinline__ int32_t write_accept(const DraftArgs& a, int32_t row, const DraftOut& o,
                                                int32_t target, int tid) {
  bool same = tid < o.n && target == o.tok;
  u64 differs = wave_ballot(!same);
  const int32_t accepted = differs ? (int32_t)__ffsll((long long)differs) - 1 : kWave;
  if (tid == 0) a.accept_len[row] = accepted;
  return accepted;
}

// Lengths of the first LDS::kLens paths into LDS (the scan reads them per tile).
// The caller synchronises the workgroup before using them.
template <int BLOCK, class LDS>
__device__ __forceinline__ void cache_lens(LDS& s, const Paths& y, int tid) {
  for (int32_t j = tid; j < y.N && j < LDS::kLens; j += BLOCK) {
    int32_t old_j = y.old_len(j);
    s.len_old[j] = old_j;
    s.len_new[j] = y.new_len(j, old_j);
  }
}

// The continuations of the M listed matches into windows of 2 L words (tokens, then
// probabilities), one (match, layer) instance per thread; ends with a workgroup barrier.
template <int BLOCK, class LDS>
__device__ __forceinline__ void fetch_windows(LDS& s, const Ctx& c, int32_t M, int32_t L,
                                              int32_t* windows) {
  for (int32_t idx = c.tid; idx < M * L; idx += BLOCK) {
    const int32_t mi = idx / L, d = idx - mi * L + 1;
    uint32_t u, v;
    u64 w;
    if (layer_instance(c.y, s.match[mi], d, 0u, u, v, w)) {
      windows[mi * 2 * L + d - 1] = (int32_t)v;
      windows[mi * 2 * L + L + d - 1] = (int32_t)cs_sum(w);
    }
  }
  block_sync<BLOCK>();
}

// Scan mode.  One 1024-thread workgroup per (problem, path): [append] -> match
// by scan (Eq. 3, or Eq. 4 with one edit) -> DAG (Eq. 5) -> greedy walk ->
// [accept].  With in.n > 0 the launch also performs the step's append; every
// workgroup then reads the other paths through `Paths`, which never touches
// cells written by this launch.  The histories are read straight from memory:
// the q + 1 tokens a position compares are shared with its neighbours in the
// wave, so all but the first load of a line hit the CU's vector cache, and no
// workgroup barrier is needed per tile as staging through LDS would.
// POOLS: also compiled for the tree and list pools (kept out of the DAG-only
// kernels, whose code and register footprint they would enlarge).
// With sl.n > 1 a row's scan is shared by sl.n workgroups (few rows: the scan is
// bound by instruction issue on the row's CU, and most CUs would be idle); the
// one that finishes last does the rest of the row's work.
// FUZZY: matching tolerates one edit (compiled apart from the exact kernel: code a launch
// does not run still costs it time).
// QC: compile-time bound (4 or 8) of the query length: the comparison loops are unrolled to it.
// INDEXED: queries of kmax tokens are looked up in the variant index instead, and the workgroup goes on
// to another row: no wave leaves.
template <int QC, bool POOLS, bool FUZZY, class LDS = LdsScan, bool INDEXED = false>
__device__ __forceinline__ void scan_step(const IndexView& ix, const StepIn& in, const DraftArgs& a,
                                          const ScanSlices& sl, int32_t row, int32_t slice) {
  constexpr int BLOCK = kScanBlock;
  __shared__ LDS s;
  __shared__ int32_t sh_base, sh_total, sh_last;
  const int32_t unit = row * 8 + slice;                  // (timing build only)
  CSD_STAMP(unit, 0, CSD_CLOCK());
  CSD_STAMP(unit, 6, 0ull);
  int32_t p;
  Ctx c = make_ctx(ix, in, row, p);
#ifdef CSD_STAMPS
  c.unit = unit;
#endif
  int32_t st_i = in.n == 1 ? c.y.st[c.i] : 0;           // (first: the head's lengths wait for its load)
  Head me = load_head(c.y, ix.tail_len, c.i);           // length and newest tokens in one read
  const int32_t old_i = me.old_len;
  c.len_i = me.new_len;
  cache_lens<BLOCK>(s, c.y, c.tid);
  if (in.n > 0 && slice == 0) append_path<false, false, QC>(ix, in, p, c.i, BLOCK, c.tid);
  if (in.n <= 1) {                                       // the query follows from what is loaded
    int32_t cnt_i = c.len_i - old_i;
    c.q = a.k < c.len_i ? a.k : c.len_i;
#pragma unroll
    for (int x = 0; x < CSD_MAX_QUERY_LEN; ++x) {
      int32_t v = 0;
      if (x < c.q) v = x < cnt_i ? st_i : pick(me.tail, x - cnt_i);
      c.Q[x] = v;
    }
  } else {
    load_query(c, a.k, old_i);
  }
  if (c.tid == 0) s.n_match = 0;
  lds_barrier<BLOCK>();                 // lengths and the empty list are in LDS; the append's stores,
                                        // which nothing in this launch reads, need not have landed
  DraftOut o;
  const int32_t L = a.L;
  CSD_STAMP(unit, 1, CSD_CLOCK());
  if (c.q > 0) {
    uint16_t* pool = reinterpret_cast<uint16_t*>(s.table) + (c.tid >> 6) * kPoolWords;   // (before the walk)
    // Spans in flight: four where the registers hold their tokens; the wave's candidates pooled where each
    // is compared token by token (without edits the filter settles most).  us a step, exact, queries of 6,
    // few symbols, four spans unpooled / two pooled: 16 x 1024 8.6 / 9.1, 64 problems 32.5 / 33.6; of 3, 64
    // problems of 8 x 512 14.2 / 14.6.  Edits and queries beyond four tokens, two spans / four, pooled: one edit,
    // 16 x 1024 19.3 / 19.6, 64 problems 84 / 79, 64 x 4096 71 / 61; two edits, 16 x 1024 30.6 / 34.6, 64
    // problems 396 / 436 (one kernel serves both: its predicates spill).
    constexpr int kSpans = (std::is_same<LDS, LdsScanPair>::value || (FUZZY && QC > 4)) ? 2 : 4;
    static_assert(sizeof(s.table) >= BLOCK / kWave * kPoolWords * sizeof(uint16_t), "a pool per wave");
    ListSink<LDS> sink{&s};
    if (INDEXED && c.q == ix.kmax) match_variants<BLOCK, QC>(s, c, sink);
    else match_scan<BLOCK, FUZZY, QC, FUZZY, kSpans>(s, c, sink, slice, sl.n, pool);
    block_sync<BLOCK>();
    int32_t M = s.n_match;
    CSD_STAMP(unit, 2, CSD_CLOCK());
    CSD_STAMP(unit, 8, (unsigned long long)M);
    if (POOLS && (ix.options & 2)) {
      // query back-off (never with slices): no match, so the query loses its oldest token and
      // the scan runs again; every thread sees the same M and q, so the barriers pair up
      while (M == 0 && c.q > 1) {
        block_sync<BLOCK>();            // everybody has read the count before anybody pushes again
        --c.q;
        match_scan<BLOCK, FUZZY, QC, FUZZY, kSpans>(s, c, sink, 0, 1, pool);
        block_sync<BLOCK>();
        M = s.n_match;
      }
    }
    if (sl.n > 1) {
      // hand this slice's matches to the row's list in memory.  One 64-bit word per row
      // holds the matches listed so far (low half) and the slices finished, over all
      // launches (high half): a slice reserves its part of the list with one atomic and
      // signs off with a second one, whose result tells the last slice the row's total
      Match* listed = sl.matches + (int64_t)row * LDS::kMatch;
      if (c.tid == 0) sh_base = (int32_t)(uint32_t)atomicAdd(&sl.state[row], (u64)(uint32_t)M);
      block_sync<BLOCK>();
      for (int32_t m = c.tid; m < M && m < LDS::kMatch; m += BLOCK)
        if (sh_base + m < LDS::kMatch) listed[sh_base + m] = s.match[m];
      block_sync<BLOCK>();              // every wave's stores have left the CU
      // (while wave 0 signs off, the others prepare the tables of the walk that rows of
      // 65 .. 1024 matches take: wasted on all slices but the last, which would wait here anyway)
      if (!POOLS || a.pool_mode == CSD_POOL_DAG) walk_tab_clear<BLOCK>(s, c.tid, kWave);
      if (c.tid == 0) {
        // one wave fences for the workgroup (a device-scope fence writes the L2 back: sixteen
        // of them in a row cost more than the scan): list entries before the sign-off, the
        // sign-off before the reads below
        __threadfence();
        const u64 seen = atomicAdd(&sl.state[row], 1ull << 32);
        sh_last = ((uint32_t)(seen >> 32) & (uint32_t)(sl.n - 1)) == (uint32_t)(sl.n - 1);
        sh_total = (int32_t)(uint32_t)seen;   // every slice has reserved before it signs off
        // the next launch starts with an empty list (nobody else touches the word any more)
        if (sh_last) sl.state[row] = ((seen >> 32) + 1ull) << 32;
        __threadfence();
      }
      block_sync<BLOCK>();
      CSD_STAMP(unit, 3, CSD_CLOCK());
      if (!sh_last) return;             // the last slice goes on with all matches of the row
      M = sh_total;
      for (int32_t m = c.tid; m < M && m < LDS::kMatch; m += BLOCK) s.match[m] = listed[m];
      if (c.tid == 0) s.n_match = M;
      block_sync<BLOCK>();
    }
    CSD_STAMP(unit, 4, CSD_CLOCK());
    CSD_STAMP(unit, 9, (unsigned long long)M);
    if (POOLS && M > 0 && a.pool_mode != CSD_POOL_DAG) {
      auto each = [&](auto f) {
        if (M <= LDS::kMatch) {
          for (int32_t m = c.tid; m < M; m += BLOCK) f(s.match[m], m);
        } else {
          auto g = [&](Match found) { f(found, -1); };
          FnSink<decltype(g)> fs{g};
          match_scan<BLOCK, FUZZY, QC>(s, c, fs);
        }
      };
      if (a.pool_mode == CSD_POOL_TREE && M <= kWave) {
        int32_t* windows = reinterpret_cast<int32_t*>(s.table);
        fetch_windows<BLOCK>(s, c, M, L, windows);
        if (c.tid < kWave)
          walk_matches<true>(s, c, M, L, WinInfo{0, M}, windows, a.alpha_q, a.score_mode, o);
      } else if (a.pool_mode == CSD_POOL_TREE) {
        walk_tree<BLOCK>(s, c, WinInfo{M, 0}, M, L, a.alpha_q, ix.status, o, each);
      } else {
        walk_list<BLOCK>(s, c, WinInfo{M, 0}, L, a.alpha_q, o, each);
      }
    } else if (M > 0) {
      // up to a wave's worth of matches: a lane per match; up to a workgroup's worth: a thread
      // per match; else streaming
      bool done = false;
      if (M <= kWave) {
        // one lane of wave 0 per match, no tables: all threads fetch the continuations into
        // windows (laid over the unused table), one (match, layer) instance each.  (More matches
        // per lane do not pay here: with one-edit matching most continuations differ, and a
        // layer then costs one round per match.)
        int32_t* windows = reinterpret_cast<int32_t*>(s.table);
        fetch_windows<BLOCK>(s, c, M, L, windows);
        if (c.tid < kWave) walk_matches(s, c, M, L, WinInfo{0, M}, windows, a.alpha_q, a.score_mode, o);
        done = true;
      } else if (M <= BLOCK) {
        // one thread per match: node weights tabulated first, or layer by layer
        // (the second where the first does not apply or finds too many distinct continuations)
        if (!walk_tab_fits<BLOCK>(M, L, ix.vocab, a.score_mode) ||
            !walk_tab<BLOCK, !INDEXED>(s, c, M, L, a.alpha_q, o, sl.n > 1))
          walk_wide<BLOCK, !INDEXED>(s, c, M, L, a.alpha_q, a.score_mode, o);
        done = true;
      }
      if (!done)
        walk_streaming<BLOCK>(s, c, WinInfo{M, 0}, M, L, a.alpha_q, a.score_mode, ix.status, o, [&](auto f) {
          if (M <= LDS::kMatch) {
            for (int32_t m = c.tid; m < M; m += BLOCK) f(s.match[m], m);
          } else {
            auto g = [&](Match found) { f(found, -1); };
            FnSink<decltype(g)> fs{g};
            match_scan<BLOCK, FUZZY, QC>(s, c, fs);
          }
        });
    }
  }
  CSD_STAMP(unit, 5, CSD_CLOCK());
  write_outputs<BLOCK>(a, row, o, c.tid);
  if (a.targets && c.tid < kWave) {
    int32_t target = c.tid < L ? a.targets[(int64_t)row * L + c.tid] : 0;
    write_accept(a, row, o, target, c.tid);
  }
  CSD_STAMP(unit, 6, CSD_CLOCK());
}

template <int QC, bool POOLS, bool FUZZY>
__global__ __launch_bounds__(kScanBlock) void step_scan_kernel(IndexView ix, StepIn in,
                                                               DraftArgs a, ScanSlices sl) {
  fetch_kernel_arguments<sizeof(IndexView) + sizeof(StepIn) + sizeof(DraftArgs) + sizeof(ScanSlices)>();
  int32_t row, slice = 0;
  if (sl.n == 1) {
    row = xcd_row(ix.P * ix.N);
  } else {                              // XCD x takes rows x, x + 8, ..: a row's slices share an L2
    int32_t idx = (int32_t)(blockIdx.x >> 3);
    slice = idx & (sl.n - 1);
    row = (idx / sl.n) * 8 + (int32_t)(blockIdx.x & 7);
    if (row >= ix.P * ix.N) row = -1;
  }
  if (row < 0) return;
  scan_step<QC, POOLS, FUZZY>(ix, in, a, sl, row, slice);
}

// Index mode.  Per (problem, path) one wave64 runs the front end (matches with
// their continuations in LDS), the DAG and its walk in one of three forms
// (lanes = instances, lanes = matches, LDS tables), outputs and accept; the
// append and the split-phase index insert are done by the same wave (one-edit
// matching) or by a second one (exact matching, see below).
// FUZZY: the index files every position under its gram's variants and matching tolerates
// one edit (Eq. 4).
// QC: compile-time bound (4 or 8) of the index's gram length.
// Two waves per row (on two SIMDs of the CU): the second does the row's append and index
// insert, which the draft does not depend on, so that they leave the critical path of the
// first.  The two never meet at a barrier.
constexpr int step_wave_threads(bool) { return 2 * kWave; }

// The accept-driven loop's stand-in model as the tail of a step (see advance_kernel): the row
// that has just drafted and counted its accepted tokens works out what it appends at the NEXT
// step — those tokens plus the one the model emits itself, from the path's own future — and
// the targets of the next draft, into buffers that the next launch reads (not the ones this
// launch reads: the caller alternates between two sets).
struct NoTail {};
struct LoopTail {
  const int32_t* future_tok;    // [rows][max_len]
  const float* future_prob;     // [rows][max_len] or null
  int32_t* next_tok;            // [rows][n]
  float* next_prob;             // [rows][n] or null
  int32_t* next_cnt;            // [rows]
  int32_t* next_targets;        // [rows][L]
  int32_t* path_len;            // [rows] output: lengths after this step's append
  int32_t n, max_len;
};

// Hands a row's accept length back to the workgroup (see loop_kernel).
struct AcceptTail {
  int32_t* accepted;            // [paths of the problem]
};

// Rows that a wave leaves to a workgroup (replay_leave_kernel): those with more matches than the walks
// with a lane per match take.
struct LeaveTail {
  RestList list;
  int32_t unit;                 // see replay_unit
};

// One decode step of one row by one wave: front end, DAG, walk, outputs, accept, tail.
// APPENDS: the wave also appends the row's tokens and files them in the index (false: another
// wave of the workgroup does, see wave_append).  s: the row's on-chip state.
// MULTI: also compiled for steps of several tokens (POOLS: for these, the tree and list pools and the options).
template <int LCAP, bool POOLS, class LDS, bool FUZZY, int QC, bool APPENDS, class TAIL, bool MULTI = POOLS>
__device__ __forceinline__ void row_step(LDS& s, const IndexView& ix, const StepIn& in,
                                         const DraftArgs& a, const TAIL& tail, int32_t row, int lane) {
  int32_t p;
  Ctx c = make_ctx(ix, in, row, p);
  c.tid = lane;
#ifdef CSD_STAMPS
  c.unit = row;
  if (lane == 0 && row < (1 << 14)) {
    g_stamps[row * kStampSlots + 0] = CSD_CLOCK();
    g_stamps[row * kStampSlots + 6] = 0ull;
  }
#endif
  const int32_t L = a.L;
  int32_t target = (a.targets && c.tid < L) ? a.targets[(int64_t)row * L + c.tid] : 0;
  WinInfo wi;
  InsertTicket ticket;
  VariantTicket tickets;
  bool ticket_used;
  constexpr bool kLeaves = std::is_same<TAIL, LeaveTail>::value;
  int32_t M = FUZZY ? wave_front_end_fuzzy<LCAP, QC, APPENDS, kLeaves ? kWave : INT_MAX>(s, c, ix, p, a.k, L, wi, tickets, ticket_used)
                    : wave_front_end<LCAP, QC, APPENDS, MULTI>(s, c, ix, p, a.k, L, wi, ticket, ticket_used);
  block_sync<kWave>();
#ifdef CSD_STAMPS
  if (lane == 0 && row < (1 << 14)) {
    g_stamps[row * kStampSlots + 1] = CSD_CLOCK();
    g_stamps[row * kStampSlots + 9] = (unsigned long long)M;
  }
#endif
  if (APPENDS && MULTI && !FUZZY && in.n > 1) {
    // a step of several tokens appended by the drafting wave itself (nothing this step's
    // drafts read is written here)
    append_path<true, false, QC>(ix, in, p, c.i, kWave, lane);
  }
  // the loop's tail needs the path's future from its new end on (lane x: x tokens further):
  // requested here, so that the load travels during the walk
  int32_t future_a = 0, future_b = 0;
  float future_p = 0.0f;
  if constexpr (std::is_same<TAIL, LoopTail>::value) {
    const int64_t base = (int64_t)row * tail.max_len;
    const int32_t xa = c.len_i + c.tid, xb = xa + kWave;
    future_a = tail.future_tok[base + (xa < tail.max_len ? xa : 0)];
    future_b = tail.future_tok[base + (xb < tail.max_len ? xb : 0)];
    if (tail.future_prob) future_p = tail.future_prob[base + (xa < tail.max_len ? xa : 0)];
  }
  if (POOLS && (ix.options & 2)) {
    // query back-off: no match, so the query loses its oldest token and the histories are
    // searched again (position by position: the index holds grams of max_query_len tokens only)
    while (M == 0 && c.q > 1) {
      --c.q;
      WaveListSink<LDS> sink{&s, &M, c.tid};
      match_plain<FUZZY>(s, c, sink);
      wi = WinInfo{M, 0};
      if (c.tid == 0) s.n_match = M;
      block_sync<kWave>();
    }
  }
  if constexpr (kLeaves) {
    const int32_t windows = LDS::kWin / (2 * L) + (a.pool_mode == CSD_POOL_DAG ? (int32_t)sizeof(s.table) / (2 * L * (int32_t)sizeof(int32_t)) : 0);
    if (M > kWave || (M > 8 && M > windows)) {           // uniform over the wave
      const uint32_t xcd = blockIdx.x & 7;
      if (lane == 0) *tail.list.unit(xcd, false, atomicAdd(tail.list.count(xcd, false), 1)) = tail.unit;
      return;
    }
  }

  DraftOut o;
  if (POOLS && M > 0 && a.pool_mode != CSD_POOL_DAG) {
    auto each = [&](auto f) {
      if (M <= LDS::kMatch) {
        for (int32_t m = c.tid; m < M; m += kWave) f(s.match[m], m);
      } else {
        auto g = [&](Match found) { f(found, -1); };
        FnSink<decltype(g)> fs{g};
        match_plain<FUZZY>(s, c, fs);
      }
    };
    if (a.pool_mode == CSD_POOL_TREE && M <= kWave && M <= LDS::kWin / (2 * L))
      walk_matches<true>(s, c, M, L, wi, s.win, a.alpha_q, a.score_mode, o);   // one lane per match
    else if (a.pool_mode == CSD_POOL_TREE)
      walk_tree<kWave>(s, c, wi, M, L, a.alpha_q, ix.status, o, each);
    else
      walk_list<kWave>(s, c, wi, L, a.alpha_q, o, each);
  } else if (M > 0 && M <= 8 && (L << lanes_log2(M)) <= kWave) {                   // few matches: no tables
    switch (lanes_log2(M)) {
      case 0: walk_instances<1>(s, c, M, L, wi, a.alpha_q, a.score_mode, o); break;
      case 1: walk_instances<2>(s, c, M, L, wi, a.alpha_q, a.score_mode, o); break;
      case 2: walk_instances<4>(s, c, M, L, wi, a.alpha_q, a.score_mode, o); break;
      default: walk_instances<8>(s, c, M, L, wi, a.alpha_q, a.score_mode, o); break;
    }
  } else if (M > 0 && M <= kWave &&
             (M - LDS::kWin / (2 * L)) * 2 * L * (int32_t)sizeof(int32_t) <= (int32_t)sizeof(s.table)) {
    // one lane per match; with more matches than the layout has windows, the others' windows
    // are laid over the table, which this walk does not use
    walk_matches(s, c, M, L, wi, s.win, a.alpha_q, a.score_mode, o, reinterpret_cast<int32_t*>(s.table),
                 LDS::kWin / (2 * L));
  } else if (kLeaves) {
    // (M is 0)
  } else if (M > 0 && M <= 2 * kWave && M <= LDS::kWin / (2 * L)) {
    walk_matches<false, 2>(s, c, M, L, wi, s.win, a.alpha_q, a.score_mode, o);   // two matches per lane
  } else if (M > 0 && walk_tab_wave_fits<LDS>(M, ix.vocab, a.score_mode) &&
             walk_tab_wave(s, c, wi, M, L, a.alpha_q, o)) {
    // node weights of all layers tabulated first, then the walk
  } else if (M > 0) {
    bool streaming = M > LDS::kMatch;
    if (!streaming) {
      Tier1 t1 = build_dag<kWave>(s, c, M, L, wi, a.alpha_q);
      streaming = s.overflow != 0;
      if (!streaming) walk_dag<kWave, LCAP>(s, c, t1, L, a.alpha_q, a.score_mode, o);
    }
    if (streaming)
      walk_streaming<kWave>(s, c, wi, M, L, a.alpha_q, a.score_mode, ix.status, o, [&](auto f) {
        if (M <= LDS::kMatch) {
          for (int32_t m = c.tid; m < M; m += kWave) f(s.match[m], m);
        } else {
          auto g = [&](Match found) { f(found, -1); };
          FnSink<decltype(g)> fs{g};
          match_plain<FUZZY>(s, c, fs);
        }
      });
  }
#ifdef CSD_STAMPS
  if (lane == 0 && row < (1 << 14)) g_stamps[row * kStampSlots + 5] = CSD_CLOCK();
#endif
  // the posting stores wait on atomics issued long ago: do them before the output stores
  if (ticket_used && FUZZY)
    variants_finish(tickets, const_cast<int32_t*>(c.gram), c.buckets, c.y.pos(c.i, c.len_i - 1),
                    c.tid);
  else if (ticket_used)
    insert_finish(ticket, const_cast<int32_t*>(c.gram), c.buckets,
                  c.y.pos(c.i, c.len_i - 1), c.tid);
  write_outputs<kWave>(a, row, o, c.tid);
  int32_t accepted = 0;
  if (a.targets) accepted = write_accept(a, row, o, target, c.tid);
#ifdef CSD_STAMPS
  if (lane == 0 && row < (1 << 14)) g_stamps[row * kStampSlots + 6] = CSD_CLOCK();
#endif
  if constexpr (std::is_same<TAIL, AcceptTail>::value) {
    if (c.tid == 0) tail.accepted[c.i] = accepted;
  }
  if constexpr (std::is_same<TAIL, LoopTail>::value) {
    const int32_t len = c.len_i;                        // after this step's append
    int32_t grow = accepted + 1;
    grow = grow > tail.n ? tail.n : grow;
    const int32_t room = tail.max_len - len;
    grow = grow < room ? grow : room;
    const int64_t r = row;
    static_assert(CSD_MAX_DRAFT_LEN + 1 <= kWave && 2 * CSD_MAX_DRAFT_LEN < 2 * kWave,
                  "a lane per step token; the targets lie within two waves' worth of the future");
    if (c.tid == 0) {
      tail.next_cnt[r] = grow;
      tail.path_len[r] = len;
    }
    if (c.tid < tail.n) {
      const bool in_path = len + c.tid < tail.max_len;
      tail.next_tok[r * tail.n + c.tid] = in_path ? future_a : 0;
      if (tail.next_prob) tail.next_prob[r * tail.n + c.tid] = in_path ? future_p : 0.0f;
    }
    // target d of the next draft is the future token grow + d places beyond the new end
    const int32_t x = grow + c.tid;
    const int32_t from_a = __shfl(future_a, x & (kWave - 1));
    const int32_t from_b = __shfl(future_b, x & (kWave - 1));
    if (c.tid < L)
      tail.next_targets[r * L + c.tid] = len + x < tail.max_len ? (x < kWave ? from_a : from_b) : -1;
  }
}

// The row of this workgroup: its first wave drafts, a second wave appends.
template <int LCAP, bool POOLS, class LDS, bool FUZZY, int QC, bool MULTI, class TAIL>
__device__ __forceinline__ void step_wave_body(const IndexView& ix, const StepIn& in,
                                               const DraftArgs& a, const TAIL& tail) {
  constexpr bool SPLIT = step_wave_threads(FUZZY) > kWave;
  __shared__ LDS s;
  int32_t row = xcd_row(ix.P * ix.N);
  if (row < 0) return;
  const int lane = (int)(threadIdx.x & (kWave - 1));
  if (SPLIT && __builtin_amdgcn_readfirstlane((int)threadIdx.x) >= kWave) {
    int32_t p;
    Ctx c = make_ctx(ix, in, row, p);
    c.tid = lane;
    if (FUZZY) wave_append_fuzzy(c, ix, p);
    else wave_append<QC, MULTI, std::is_same<LDS, LdsWaveSmall>::value ? 1 : kInsertLanes>(c, ix, in, p);
    return;
  }
  row_step<LCAP, POOLS, LDS, FUZZY, QC, !SPLIT, TAIL, MULTI>(s, ix, in, a, tail, row, lane);
}

// BLOCKS: for an index with home blocks (see Buckets).
template <int LCAP, bool POOLS, class LDS, bool FUZZY, int QC, bool MULTI = POOLS, bool BLOCKS = true>
__global__ __launch_bounds__(step_wave_threads(FUZZY)) void step_wave_kernel(IndexView ix, StepIn in,
                                                                             DraftArgs a) {
  fetch_kernel_arguments<sizeof(IndexView) + sizeof(StepIn) + sizeof(DraftArgs)>();
  if (!BLOCKS) ix.buckets.block = ix.buckets.mask;
  step_wave_body<LCAP, POOLS, LDS, FUZZY, QC, MULTI>(ix, in, a, NoTail{});
}

// The same for launches of thousands of rows (exact matching, drafts of up to 8 tokens), where
// the number of rows resident on a CU bounds the throughput: compiled for eight waves per SIMD
// (at most 64 registers per lane), with the small on-chip layout: sixteen rows per CU.  (Registers by number, of
// which the attribute counts half: asked for by waves the compiler gives a wave 80 scalar registers, eight
// arguments more are spilled and read back all over the kernel; with 102 a SIMD has seven waves.  65536 rows
// from empty histories 81.6 us a step, at full histories 116.4, with 80 81.7 and 123.4, with 102 91 and 137.)
// BLOCKS: see step_wave_kernel.
template <int QC, bool BLOCKS>
__global__ __launch_bounds__(step_wave_threads(false)) __attribute__((amdgpu_num_vgpr(32), amdgpu_num_sgpr(96)))
void step_wave_many_kernel(IndexView ix, StepIn in, DraftArgs a) {
  fetch_kernel_arguments<sizeof(IndexView) + sizeof(StepIn) + sizeof(DraftArgs)>();
  if (!BLOCKS) ix.buckets.block = ix.buckets.mask;
  step_wave_body<8, false, LdsWaveSmall, false, QC, false>(ix, in, a, NoTail{});
}

// One step of the accept-driven loop in one launch: a step of up to L + 1 tokens per path
// (general instantiation, exact matching), then the tail that prepares the next step.
template <int LCAP, int QC, bool POOLS>
__global__ __launch_bounds__(step_wave_threads(false)) void step_loop_kernel(IndexView ix, StepIn in,
                                                                             DraftArgs a,
                                                                             LoopTail tail) {
  fetch_kernel_arguments<sizeof(IndexView) + sizeof(StepIn) + sizeof(DraftArgs) + sizeof(LoopTail)>();
  step_wave_body<LCAP, POOLS, LdsWave, false, QC, true>(ix, in, a, tail);
}

// Many steps per launch (the device-side form of the host loops csd_replay and
// csd_accept_loop, where nothing happens on the host between two steps): one workgroup per
// problem, one wave per path (at most 16), exact matching through the index.  A step's rows
// only read what earlier steps wrote, so one workgroup barrier between steps orders
// everything; no launch, no cold cache and no argument fetch per step.
struct MultiArgs {
  int32_t n_steps, cur;         // cur: which meta buffer holds the paths' ends on entry
  int32_t* meta[2];
  // replay: step t appends tokens[t] (one token per path) and drafts into slice t
  const int32_t* tokens;        // [n_steps][P][N], or null (the accept-driven loop)
  const float* probs;           // [n_steps][P][N] or null
  const int32_t* targets;       // [n_steps][P][N][L] or null
  float* token_scores;          // [n_steps][P][N][L] or null
  float* path_scores;           // [n_steps][P][N] or null
  // accept-driven loop: the two sets of step buffers (see LoopTail); step t reads set t & 1
  int32_t* step_tok[2];
  float* step_prob[2];
  int32_t* step_cnt[2];
  int32_t* step_targets[2];
  const int32_t* future_tok;
  const float* future_prob;
  int32_t* path_len;            // [n_steps][P][N]
  int32_t n;                    // tokens per path and step the loop offers (L + 1)
  // both
  DraftArgs a;                  // outputs of step 0; step t writes slice t
};

template <int LCAP, bool POOLS, int QC, bool LOOP>
__global__ __launch_bounds__(16 * kWave) void step_multi_kernel(IndexView ix, MultiArgs m) {
  __shared__ LdsMulti rows_lds[16];
  const int wave = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & (kWave - 1));
  const int32_t row = (int32_t)blockIdx.x * ix.N + wave;    // the block has N waves
  const int64_t rows = (int64_t)ix.P * ix.N;
  const int64_t L = m.a.L;
  for (int32_t t = 0; t < m.n_steps; ++t) {
    IndexView v = ix;
    v.meta_old = m.meta[(m.cur + t) & 1];
    v.meta_new = m.meta[(m.cur + t + 1) & 1];
    DraftArgs a = m.a;
    a.draft_tokens += t * rows * L;
    a.draft_len += t * rows;
    if (a.accept_len) a.accept_len += t * rows;
    if constexpr (LOOP) {
      const int x = t & 1;
      const StepIn in{m.step_tok[x], m.step_prob[x], m.step_cnt[x], m.n};
      a.targets = m.step_targets[x];
      const LoopTail tail{m.future_tok, m.future_prob, m.step_tok[x ^ 1], m.step_prob[x ^ 1],
                          m.step_cnt[x ^ 1], m.step_targets[x ^ 1], m.path_len + t * rows, m.n, ix.max_len};
      row_step<LCAP, true, LdsMulti, false, QC, true>(rows_lds[wave], v, in, a, tail, row, lane);
    } else {
      const StepIn in{m.tokens + t * rows, m.probs ? m.probs + t * rows : nullptr, nullptr, 1};
      if (a.targets) a.targets += t * rows * L;
      if (a.token_scores) a.token_scores += t * rows * L;
      if (a.path_scores) a.path_scores += t * rows;
      row_step<LCAP, POOLS, LdsMulti, false, QC, true>(rows_lds[wave], v, in, a, NoTail{}, row, lane);
    }
    // what this step wrote (histories, path ends, index, the loop's next input) before what
    // the next step reads: the waves of a workgroup share their CU's vector cache, which is
    // dropped here all the same (index buckets are also written by atomics, which work in
    // the L2)
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  }
}

// A recorded trace (csd_replay): all tokens are known when the call is made, so its steps do not
// wait for each other.  One launch appends the tokens of many steps and notes every path's end as
// it is after each of them; a second one drafts all paths at all those steps side by side, each
// from the ends of its own step: what lies beyond them in the histories and postings is not seen.
// A launch per step leaves most of the chip idle and waits for its slowest row; this is bound by the
// drafts a CU holds at once.  us for reset, append of the past and replay, a launch per step / this:
// 16 paths x 1024 tokens, 64 steps 355 / 22; 64 x 4096, 48 steps 357 / 36; one edit by scan, 16 x 1024, 32 steps 622 / 49; one
// edit through the index, 64 x 4096, 24 steps 686 / 106.  (Many small problems: replay_staged_kernel, one launch for both.)
struct ReplayIn {
  const int32_t* tok;           // [steps][P][N]
  const float* prob;            // [steps][P][N] or null
  int32_t steps;
};

// The append: a workgroup has 2^paths_log2 whole paths of a problem (so that the paths' ends can be
// replaced in place: meta_new may be meta_old), a thread per new position; neighbouring threads
// have neighbouring paths, whose tokens of a step lie side by side.
// step_meta [steps][P][N][meta_stride]: the paths' ends after each step.
template <bool INDEX, bool FUZZY, int QC>
__global__ __launch_bounds__(256) void replay_append_kernel(IndexView ix, ReplayIn in, int32_t* step_meta,
                                                             int32_t paths_log2, int32_t* rest_count) {
  if (blockIdx.x == 0 && threadIdx.x < 16) rest_count[threadIdx.x * kBucketWords] = 0;   // (of the drafts' launches behind this one)
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1);
  const int32_t paths = 1 << paths_log2, groups = (ix.N + paths - 1) >> paths_log2;
  const int32_t p = (int32_t)blockIdx.x / groups, i0 = ((int32_t)blockIdx.x - p * groups) << paths_log2;
  const int32_t i = i0 + (tid & (paths - 1)), at_once = (int32_t)blockDim.x >> paths_log2;
  const bool on = i < ix.N;
  const int64_t rows = (int64_t)ix.P * ix.N, row = (int64_t)p * ix.N + (on ? i : i0);
  int32_t* gram = INDEX ? ix.gram + (int64_t)p * ((int64_t)ix.buckets.mask + 1) * kBucketWords : nullptr;
  uint32_t flags = 0;
  for (int32_t t0 = 0; t0 < in.steps; t0 += at_once) {   // uniform over the workgroup
    const int32_t t = on ? t0 + (tid >> paths_log2) : in.steps;   // (idle: behind the last step)
    NewTokens<QC> x;
    x.load(ix, row, in.tok + row, in.prob ? in.prob + row : nullptr, rows, in.steps, nullptr, t);
    const int32_t cnt = x.count(ix);
    if (x.most() > cnt) flags |= CSD_STATUS_CAPACITY;
    flags |= x.store(ix, in.prob != nullptr, row, cnt);
    if constexpr (INDEX)
      file_positions<FUZZY, QC>(gram, ix.buckets, ix.kmax, x.G, x.filed(ix, cnt), x.pos(ix, i), lane, [] {});
    if (t < in.steps) {
      int32_t* end = step_meta + (t * rows + row) * ix.meta_stride;
      end[0] = x.len + (t < cnt ? t + 1 : cnt);
      for (int32_t a = ix.tail_len; a + 1 < ix.meta_stride; ++a) end[1 + a] = 0;
      if (t < cnt) {
        end[1] = x.token;
#pragma unroll
        for (int a = 0; a < QC; ++a)
          if (a + 1 < ix.tail_len) end[2 + a] = x.G[a];
      } else {                                           // the path was full before
        const int32_t* meta = ix.meta_old + row * ix.meta_stride;
        for (int32_t a = 0; a < ix.tail_len; ++a)
          end[1 + a] = a < cnt ? in.tok[(cnt - 1 - a) * rows + row] : (a < x.len + cnt ? meta[1 + a - cnt] : 0);
      }
    }
  }
  __syncthreads();                                       // the old ends have been read, the new ones noted
  for (int32_t x = tid; x < paths * ix.meta_stride; x += (int32_t)blockDim.x) {
    const int32_t path = i0 + x / ix.meta_stride, w = x % ix.meta_stride;
    if (path < ix.N) {
      const int64_t r = (int64_t)p * ix.N + path;
      ix.meta_new[r * ix.meta_stride + w] = step_meta[((in.steps - 1) * rows + r) * ix.meta_stride + w];
    }
  }
  if (flags) atomicOr(ix.status, flags);
}

// Which (problem, step, path) a workgroup drafts: the steps of a problem lie together, so that an
// XCD's L2 holds the problems that its workgroups are at.  Returns the row, or -1; ix and a become
// those of the step.  (ix.meta_old: step_meta of the append.)
__device__ __forceinline__ int32_t replay_unit(IndexView& ix, DraftArgs& a, int32_t steps, int32_t unit) {
  if (unit < 0) return -1;
  const int32_t per_problem = ix.N * steps, p = unit / per_problem, rest = unit - p * per_problem;
  const int32_t t = rest / ix.N, i = rest - t * ix.N;
  const int64_t before = (int64_t)t * ix.P * ix.N;       // rows of the steps before
  ix.meta_old += before * ix.meta_stride;
  a.draft_tokens += before * a.L;
  a.draft_len += before;
  if (a.token_scores) a.token_scores += before * a.L;
  if (a.path_scores) a.path_scores += before;
  if (a.targets) {
    a.targets += before * a.L;
    a.accept_len += before;
  }
  return p * ix.N + i;
}

template <int LCAP, bool POOLS, class LDS, bool FUZZY, int QC>
__global__ __launch_bounds__(kWave) void replay_wave_kernel(IndexView ix, int32_t steps, DraftArgs a) {
  __shared__ LDS s;
  const int32_t row = replay_unit(ix, a, steps, xcd_row(ix.P * ix.N * steps));
  if (row < 0) return;
  row_step<LCAP, POOLS, LDS, FUZZY, QC, false>(s, ix, StepIn{nullptr, nullptr, nullptr, 0}, a, NoTail{}, row,
                                               (int)threadIdx.x);
}

// The rows that are left to a wave of their own, in one launch of workgroups that hold either four waves
// with the small layout or one with the large: the rows with few matches take the former (what counts is
// how many are under way), those with many, whose hundreds of matches take 19 us instead of 92, the
// latter.  An XCD's workgroups are split between its two lists by the room that their rows take, so that
// both are done at once.  Where thousands of rows are left (paths that agree in most tokens) all take the
// small layout, in twice as many workgroups as the chip holds at once.  us, the two launches that this was
// before (the small layout for lists of more than 1024 rows, then the large for all others) / this:
// 1024 problems x 16 paths x 24 steps, 8000 rows left, 4.7 + 68 / 46; 64 problems x 48 steps, 1000 rows,
// 3.8 + 22.7 / 21; the whole replay where the paths agree in all but 20 %, 5 %, 2 % of their tokens: 1024 problems
// 157, 315, 374 / 147, 269, 310, 64 problems 46, 73, 81 / 38, 66, 74.  Left to itself the compiler takes 182
// registers (252, 256 for drafts of up to 16, 32 tokens) for the two layouts' code, two waves a SIMD: 1024
// problems 73 / 68.  Held to more waves it spills (29, 133, 58 registers; the launches before: none) and is the
// faster all the same: the whole replay of 1024 problems, paths of few matches, agreeing in all but 5 %, drafts
// of 8: 280, 318 before, 204, 287 at three waves, 198, 266 at four; of 16: 315, 435 / 280, 378 at two, 272, 340 at
// three; of 32: 820, 720 / 577, 631 at one, 442, 495 at two.
// A wave takes many rows, one after the other.  It reads the arguments anew for each (kept over the
// loop beside the row's own they were spilled, 500 instructions a row), and requests the next row's
// unit before this one's work (two round trips a row).
struct RestArgs {
  IndexView ix;
  int32_t steps;
  DraftArgs a;
  RestList list;
};
constexpr int32_t kFewRest = 1024;     // rows of a list
constexpr int32_t kRestTurn = 128;   // workgroups of an XCD that are under way at once (of twice as many)
struct LdsWaveRest : LdsWaveSmall {};  // (four buckets of a chain are read up front: most of these rows have long ones)
__device__ __forceinline__ const RestArgs& rest_arguments() {
  auto* kernarg = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kernarg));
  return *(const RestArgs*)kernarg;
}
// The rows x, x + stride .. of `count`, of which the first `few` are of the list of rows with few matches.
template <int LCAP, int QC, class LDS>
__device__ __forceinline__ void rest_rows(LDS& s, int32_t x, int32_t stride, int32_t few, int32_t count, int lane) {
  auto unit_of = [&](int32_t x) {      // (any unit behind the last)
    const RestList list = rest_arguments().list;
    const bool many = x >= few;
    return *list.unit(blockIdx.x & 7, many, x < count ? (many ? x - few : x) : 0);
  };
  if (x >= count) return;
  int32_t next = unit_of(x);
  while (x < count) {
    const int32_t unit = __builtin_amdgcn_readfirstlane(next);
    x += stride;
    next = unit_of(x);
    const RestArgs& args = rest_arguments();
    IndexView v = args.ix;
    DraftArgs b = args.a;
    const int32_t row = replay_unit(v, b, args.steps, unit);
    row_step<LCAP, false, LDS, false, QC, false>(s, v, StepIn{nullptr, nullptr, nullptr, 0}, b, NoTail{}, row, lane);
    block_sync<kWave>();
  }
}
template <int LCAP, int QC>
__global__ __launch_bounds__(4 * kWave) __attribute__((amdgpu_waves_per_eu(LCAP <= 8 ? 4 : LCAP <= 16 ? 3 : 2)))
void replay_rest_kernel(RestArgs) {
  constexpr int kWaves = 4;
  __shared__ union Layouts {
    LdsWaveRest small[kWaves];
    LdsWave large;
  } s;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = (int)(threadIdx.x & (kWave - 1));
  const int32_t nth = (int32_t)(blockIdx.x >> 3);
  int32_t few, many;
  {
    const RestList list = rest_arguments().list;
    few = __builtin_amdgcn_readfirstlane(*list.count(blockIdx.x & 7, false));
    many = __builtin_amdgcn_readfirstlane(*list.count(blockIdx.x & 7, true));
  }
  if (few + many == 0) return;                           // (the same in all waves of the XCD's workgroups)
  if (rest_arguments().list.readers) {                   // uniform over the launch
    // each wave has read the counters for itself: thread 0 signs off for all four behind the last of them (else
    // the XCD's last reader zeroes them before a late wave, whose rows would stay as they are)
    __syncthreads();
    if (threadIdx.x == 0) {
      const RestList list = rest_arguments().list;
      int32_t* readers = list.readers + (blockIdx.x & 7) * kBucketWords;
      if (atomicAdd(readers, 1) == (int32_t)(gridDim.x >> 3) - 1) *readers = *list.count(blockIdx.x & 7, false) = *list.count(blockIdx.x & 7, true) = 0;
    }
  }
  // (a row of the large layout takes the room of four; the large ones are spread over the workgroups'
  // numbers, so that those under way first are of both kinds)
  int32_t groups = 2 * kRestTurn, large = 0, before = 0;
  if (many <= kFewRest) {
    groups = few > kFewRest ? 2 * kRestTurn : kRestTurn;
    if (nth >= groups) return;
    large = (groups * kWaves * many + few + kWaves * many - 1) / (few + kWaves * many);
    large = large < many ? large : many;
    large = few > 0 && large >= groups ? groups - 1 : large;
    before = nth * large / groups;                       // workgroups below this one that take the large layout
    if ((nth + 1) * large / groups > before) {
      if (wave == 0) rest_rows<LCAP, QC>(s.large, few + before, large, few, few + many, lane);
      return;
    }
  }
  rest_rows<LCAP, QC>(s.small[wave], (nth - before) * kWaves + wave, (groups - large) * kWaves, few,
                      many <= kFewRest ? few : few + many, lane);
}

// One edit through the index, many drafts: most rows have few matches and are done by a wave, on a small
// layout so that all of them start at once; the few with more than 64, which set the time (front end
// 25 us, walk 60), are listed, each XCD's apart, for workgroups that look up with all waves and walk like
// the scan.
template <int LCAP, int QC>
__global__ __launch_bounds__(kWave) void replay_leave_kernel(IndexView ix, int32_t steps, DraftArgs a, RestList list) {
  fetch_kernel_arguments<sizeof(IndexView) + sizeof(int32_t) + sizeof(DraftArgs) + sizeof(RestList)>();
  __shared__ LdsWaveLeave s;
  const int32_t unit = xcd_row(ix.P * ix.N * steps), row = replay_unit(ix, a, steps, unit);
  if (row < 0) return;
  row_step<LCAP, true, LdsWaveLeave, true, QC, false>(s, ix, StepIn{nullptr, nullptr, nullptr, 0}, a, LeaveTail{list, unit}, row,
                                                      (int)threadIdx.x);
}

template <int QC, bool POOLS>
__global__ __launch_bounds__(kScanBlock) void replay_left_kernel(IndexView ix, int32_t steps, DraftArgs a, RestList list) {
  const uint32_t xcd = blockIdx.x & 7;
  const int32_t count = __builtin_amdgcn_readfirstlane(*list.count(xcd, false));
  for (int32_t x = (int32_t)(blockIdx.x >> 3); x < count; x += (int32_t)(gridDim.x >> 3)) {   // uniform over the workgroup
    IndexView v = ix;
    DraftArgs b = a;
    const int32_t row = replay_unit(v, b, steps, __builtin_amdgcn_readfirstlane(*list.unit(xcd, false, x)));
    scan_step<QC, POOLS, true, LdsScan, true>(v, StepIn{nullptr, nullptr, nullptr, 0}, b, ScanSlices{1, nullptr, nullptr}, row, 0);
    __syncthreads();
  }
}

template <int QC, bool POOLS, bool FUZZY>
__global__ __launch_bounds__(kScanBlock) void replay_scan_kernel(IndexView ix, int32_t steps, DraftArgs a) {
  // (the early request keeps the arguments in registers, which the kernels for edits and queries beyond four
  // tokens do not have: 53 of a lane's spilled instead of 16, 4 x 256, 24 steps 17.5 / 21.8 us; one edit,
  // queries of three, 16 x 1024, 40 steps 45.1 / 46.6 without; exact, of three 42.4 / 41.5 without, of five 29.2 / 28.6)
  if (FUZZY == (QC <= 4)) fetch_kernel_arguments<sizeof(IndexView) + sizeof(int32_t) + sizeof(DraftArgs)>();
  const int32_t row = replay_unit(ix, a, steps, xcd_row(ix.P * ix.N * steps));
  if (row < 0) return;
  scan_step<QC, POOLS, FUZZY>(ix, StepIn{nullptr, nullptr, nullptr, 0}, a, ScanSlices{1, nullptr, nullptr}, row, 0);
}

// The same with two rows a CU (LdsScanPair, 64 registers a lane): the scan of one, bound by instruction
// issue, beside the walk of the other, a chain of LDS round trips.  us, replay of 32 steps with one edit,
// one row a CU / two: 16 x 1024 positions 57 / 46, 8 problems (24 steps) 215 / 145, 16 problems (12
// steps) 249 / 161, edge scoring 65 / 52; scan_pairs says where it loses.  Three things made up the
// step: two rows (57 / 52), the wave's candidates pooled (49), two spans in flight and not four,
// which spilled less (46).
template <int QC, bool FUZZY>
__global__ __launch_bounds__(kScanBlock) __attribute__((amdgpu_waves_per_eu(8, 8)))
void replay_scan_pair_kernel(IndexView ix, int32_t steps, DraftArgs a) {
  fetch_kernel_arguments<sizeof(IndexView) + sizeof(int32_t) + sizeof(DraftArgs)>();
  const int32_t row = replay_unit(ix, a, steps, xcd_row(ix.P * ix.N * steps));
  if (row < 0) return;
  scan_step<QC, false, FUZZY, LdsScanPair>(ix, StepIn{nullptr, nullptr, nullptr, 0}, a, ScanSlices{1, nullptr, nullptr}, row, 0);
}

static __global__ __launch_bounds__(256) void accept_kernel(int64_t rows, int32_t L,
                                                     const int32_t* draft_tokens,
                                                     const int32_t* draft_len,
                                                     const int32_t* targets, int32_t* accept_len) {
  int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= rows) return;
  int32_t n = draft_len[r];
  n = n < 0 ? 0 : (n > L ? L : n);
  int32_t a = 0;
  while (a < n && draft_tokens[r * L + a] == targets[r * L + a]) ++a;
  accept_len[r] = a;
}

// The stand-in model of the accept-driven loop: what the model samples for a
// path is the path's own future.  Per row: the step's input — the tokens the
// previous step settled (its accepted draft tokens plus the one token the model
// emits itself), i.e. the next n of the path's future with a count, clipped at
// max_len — and the targets the coming draft will be checked against, the L
// future tokens behind them (-1 beyond the end).
static __global__ __launch_bounds__(256) void advance_kernel(int64_t rows, int32_t max_len, int32_t n,
                                                      int32_t L, const int32_t* meta,
                                                      int32_t meta_stride, const int32_t* settled,
                                                      const int32_t* future_tok,
                                                      const float* future_prob, int32_t* step_tok,
                                                      float* step_prob, int32_t* step_cnt,
                                                      int32_t* targets, int32_t* path_len) {
  int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= rows) return;
  int32_t len = meta[r * meta_stride];
  int32_t grow = (settled ? settled[r] : 0) + 1;
  grow = grow < 1 ? 1 : (grow > n ? n : grow);
  int32_t room = max_len - len;
  grow = grow < room ? grow : room;
  step_cnt[r] = grow;
  path_len[r] = len + grow;
  const int32_t* ft = future_tok + r * max_len;
  for (int32_t t = 0; t < n; ++t) {
    bool in = len + t < max_len;
    step_tok[r * n + t] = in ? ft[len + t] : 0;
    if (step_prob) step_prob[r * n + t] = in ? future_prob[r * max_len + len + t] : 0.0f;
  }
  for (int32_t d = 0; d < L; ++d) {
    int32_t t = len + grow + d;
    targets[r * L + d] = t < max_len ? ft[t] : -1;
  }
}

// advance_kernel and append_kernel in one launch (index mode): one wave per row works out the
// row's step input, writes it where the draft launch behind it finds the targets, and appends it.
// The path's end is replaced in place (nobody else reads it).
template <bool FUZZY, int QC>
__global__ __launch_bounds__(kWave) void advance_append_kernel(
    IndexView ix, int32_t n, int32_t L, const int32_t* settled, const int32_t* future_tok,
    const float* future_prob, int32_t* step_tok, float* step_prob, int32_t* step_cnt,
    int32_t* targets, int32_t* path_len) {
  fetch_kernel_arguments<sizeof(IndexView) + 2 * sizeof(int32_t) + 9 * sizeof(void*)>();
  const int64_t r = blockIdx.x;
  const int tid = threadIdx.x;
  const int32_t max_len = ix.max_len;
  const int32_t len = ix.meta_old[r * ix.meta_stride];
  int32_t grow = (settled ? settled[r] : 0) + 1;
  grow = grow < 1 ? 1 : (grow > n ? n : grow);
  const int32_t room = max_len - len;
  grow = grow < room ? grow : room;
  if (tid == 0) {
    step_cnt[r] = grow;
    path_len[r] = len + grow;
  }
  const int32_t* ft = future_tok + r * max_len;
  for (int32_t t = tid; t < n; t += kWave) {
    bool in = len + t < max_len;
    step_tok[r * n + t] = in ? ft[len + t] : 0;
    if (step_prob) step_prob[r * n + t] = in ? future_prob[r * max_len + len + t] : 0.0f;
  }
  for (int32_t d = tid; d < L; d += kWave) {
    int32_t t = len + grow + d;
    targets[r * L + d] = t < max_len ? ft[t] : -1;
  }
  __syncthreads();                      // the step input is read back below
  const int32_t p = (int32_t)r / ix.N;
  append_path<true, FUZZY, QC>(ix, StepIn{step_tok, step_prob, step_cnt, n}, p, (int32_t)r - p * ix.N, kWave, tid);
}

// Plain copy of n 16-byte words: the known-size kernel that hardware traffic
// counters are calibrated against.
static __global__ __launch_bounds__(256) void copy_kernel(const uint4* __restrict__ src,
                                                   uint4* __restrict__ dst, int64_t n) {
  int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t x = (int64_t)blockIdx.x * 256 + threadIdx.x; x < n; x += stride) dst[x] = src[x];
}

// ---- debug dumps ------------------------------------------------------------

// Scan mode: marks every match of every row in a bitmap [rows][words].
static __global__ __launch_bounds__(kScanBlock) void dump_match_bits_scan_kernel(IndexView ix, StepIn in,
                                                                          int32_t k, uint32_t* bits,
                                                                          int32_t words) {
  __shared__ LdsScan s;
  int32_t row = xcd_row(ix.P * ix.N);
  if (row < 0) return;
  int32_t p;
  Ctx c = make_ctx(ix, in, row, p);   // in.n == 0: nothing is being appended
  int32_t old_i = c.y.old_len(c.i);
  c.len_i = old_i;
  load_query(c, k, old_i);
  cache_lens<kScanBlock>(s, c.y, c.tid);
  block_sync<kScanBlock>();
  if (c.q <= 0) return;
  BitmapSink sink{bits + (int64_t)row * words};
  match_scan_any<kScanBlock>(s, c, sink);
}

// Index mode: the matches as the step kernel's own front end finds them.
template <bool FUZZY>
__global__ __launch_bounds__(kWave) void dump_match_bits_wave_kernel(IndexView ix, StepIn in,
                                                                     int32_t k, uint32_t* bits,
                                                                     int32_t words) {
  __shared__ LdsWave s;
  int32_t row = xcd_row(ix.P * ix.N);
  if (row < 0) return;
  int32_t p;
  Ctx c = make_ctx(ix, in, row, p);   // in.n == 0: nothing is being appended
  WinInfo wi;
  InsertTicket ticket;
  VariantTicket tickets;
  bool ticket_used;
  int32_t M = FUZZY ? wave_front_end_fuzzy<8>(s, c, ix, p, k, 1, wi, tickets, ticket_used)
                    : wave_front_end<8, CSD_MAX_QUERY_LEN, true, true>(s, c, ix, p, k, 1, wi, ticket, ticket_used);
  block_sync<kWave>();
  BitmapSink sink{bits + (int64_t)row * words};
  if (M <= LdsWave::kMatch) {
    for (int32_t m = c.tid; m < M; m += kWave) sink.push(c.y, true, s.match[m]);
  } else if (c.q > 0) {
    match_plain<FUZZY>(s, c, sink);
  }
}

// counts[row] = number of set bits of the row (one workgroup per row)
static __global__ __launch_bounds__(256) void count_bits_kernel(const uint32_t* bits, int32_t words,
                                                         int32_t* counts) {
  __shared__ int total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  const uint32_t* b = bits + (int64_t)blockIdx.x * words;
  int n = 0;
  for (int32_t w = threadIdx.x; w < words; w += 256) n += __popc(b[w]);
  atomicAdd(&total, n);
  __syncthreads();
  if (threadIdx.x == 0) counts[blockIdx.x] = total;
}

// off[0] = 0, off[r+1] = off[r] + max(counts[r], 0); *bad = 1 if any count < 0
static __global__ void offsets_kernel(const int32_t* counts, int32_t rows, int32_t* off, int32_t* bad) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  int32_t acc = 0, any_bad = 0;
  off[0] = 0;
  for (int32_t r = 0; r < rows; ++r) {
    int32_t n = counts[r];
    if (n < 0) { any_bad = 1; n = 0; }
    acc += n;
    off[r + 1] = acc;
  }
  *bad = any_bad;
}

// Expands each row's bitmap into ascending (j, e) pairs (one wave per row).
static __global__ __launch_bounds__(64) void expand_bits_kernel(const uint32_t* bits, int32_t words,
                                                         int32_t max_len, const int32_t* off,
                                                         int32_t* out_je, int64_t cap) {
  const uint32_t* b = bits + (int64_t)blockIdx.x * words;
  int64_t base = off[blockIdx.x];
  int lane = threadIdx.x;
  for (int32_t w0 = 0; w0 < words; w0 += 64) {
    int32_t w = w0 + lane;
    uint32_t x = w < words ? b[w] : 0u;
    int n = __popc(x);
    int incl = n;                                     // inclusive prefix sum over lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    int64_t at = base + incl - n;
    while (x) {
      int bit = __ffs(x) - 1;
      x &= x - 1;
      int32_t pos = w * 32 + bit;
      if (at < cap) {
        out_je[2 * at] = pos / max_len;
        out_je[2 * at + 1] = pos % max_len;
      }
      ++at;
    }
    base += __shfl(incl, 63);
  }
}

// Scan mode: builds the tier-1 DAG tables of a row exactly as step_scan_kernel
// does and writes the edge entries, sorted by key, to tmp rows of kDumpStride
// entries.  counts[row] = number of edges, or -1 if the row's DAG does not fit
// the table as a whole.
static __global__ __launch_bounds__(kScanBlock) void dump_edge_rows_scan_kernel(
    IndexView ix, StepIn in, int32_t k, int32_t L, u64* tmp_keys, u64* tmp_vals, int32_t* counts) {
  constexpr int BLOCK = kScanBlock;
  __shared__ LdsScan s;
  __shared__ int n_edges;
  int32_t row = xcd_row(ix.P * ix.N);
  if (row < 0) return;
  int32_t p;
  Ctx c = make_ctx(ix, in, row, p);   // in.n == 0: nothing is being appended
  int32_t old_i = c.y.old_len(c.i);
  c.len_i = old_i;
  load_query(c, k, old_i);
  cache_lens<BLOCK>(s, c.y, c.tid);
  if (c.tid == 0) { s.n_match = 0; n_edges = 0; }
  block_sync<BLOCK>();
  if (c.q <= 0) { if (c.tid == 0) counts[row] = 0; return; }
  ListSink<LdsScan> sink{&s};
  match_scan_any<BLOCK>(s, c, sink);
  block_sync<BLOCK>();
  int32_t M = s.n_match;
  if (M == 0) { if (c.tid == 0) counts[row] = 0; return; }
  if (M > LdsScan::kMatch) { if (c.tid == 0) counts[row] = -1; return; }
  Tier1 t1 = build_dag<BLOCK>(s, c, M, L, WinInfo{M, 0}, 0u);
  if (s.overflow) { if (c.tid == 0) counts[row] = -1; return; }
  emit_sorted_edges<BLOCK>(s, t1.region * (uint32_t)L, c.tid, &n_edges,
                           tmp_keys + (int64_t)row * kDumpStride, tmp_vals + (int64_t)row * kDumpStride);
  block_sync<BLOCK>();
  if (c.tid == 0) counts[row] = n_edges;
}

// Index mode: front end and DAG build of the step kernel itself.
template <int LCAP, bool FUZZY>
__global__ __launch_bounds__(kWave) void dump_edge_rows_wave_kernel(IndexView ix, StepIn in,
                                                                    int32_t k, int32_t L,
                                                                    u64* tmp_keys, u64* tmp_vals,
                                                                    int32_t* counts) {
  __shared__ LdsWave s;
  __shared__ int n_edges;
  int32_t row = xcd_row(ix.P * ix.N);
  if (row < 0) return;
  int32_t p;
  Ctx c = make_ctx(ix, in, row, p);   // in.n == 0: nothing is being appended
  if (c.tid == 0) n_edges = 0;
  WinInfo wi;
  InsertTicket ticket;
  VariantTicket tickets;
  bool ticket_used;
  int32_t M = FUZZY ? wave_front_end_fuzzy<LCAP>(s, c, ix, p, k, L, wi, tickets, ticket_used)
                    : wave_front_end<LCAP, CSD_MAX_QUERY_LEN, true, true>(s, c, ix, p, k, L, wi, ticket, ticket_used);
  block_sync<kWave>();
  if (M == 0) { if (c.tid == 0) counts[row] = 0; return; }
  if (M > LdsWave::kMatch) { if (c.tid == 0) counts[row] = -1; return; }
  Tier1 t1 = build_dag<kWave>(s, c, M, L, wi, 0u);
  if (s.overflow) { if (c.tid == 0) counts[row] = -1; return; }
  emit_sorted_edges<kWave>(s, t1.region * (uint32_t)L, c.tid, &n_edges,
                           tmp_keys + (int64_t)row * kDumpStride, tmp_vals + (int64_t)row * kDumpStride);
  block_sync<kWave>();
  if (c.tid == 0) counts[row] = n_edges;
}

static __global__ __launch_bounds__(256) void scatter_edges_kernel(const u64* tmp_keys,
                                                            const u64* tmp_vals,
                                                            const int32_t* off, int32_t* out_duv,
                                                            uint64_t* out_cs, int64_t cap) {
  int32_t row = blockIdx.x;
  int64_t base = off[row];
  int32_t n = off[row + 1] - off[row];
  for (int32_t x = threadIdx.x; x < n; x += 256) {
    int64_t at = base + x;
    if (at >= cap) break;
    u64 key = tmp_keys[(int64_t)row * kDumpStride + x];
    u64 val = tmp_vals[(int64_t)row * kDumpStride + x];
    out_duv[3 * at] = (int32_t)(key >> 58);
    out_duv[3 * at + 1] = (int32_t)key_u(key);
    out_duv[3 * at + 2] = (int32_t)key_v(key);
    out_cs[2 * at] = cs_count(val);
    out_cs[2 * at + 1] = cs_sum(val);
  }
}

}  // namespace csd
