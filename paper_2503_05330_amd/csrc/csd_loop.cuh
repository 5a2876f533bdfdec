// csd — the accept-driven loop in one launch: a workgroup per problem, sixteen lanes per path.
#pragma once

#include "csd_kernels.cuh"

namespace csd {

constexpr int kLoopLanes = 16;         // lanes of a path: a row of DPP moves
constexpr int kLoopPaths = 32;         // most paths of a problem (eight waves of four)
constexpr int kLoopMatches = 64;       // most matches of a row that its sixteen lanes draft (four a lane in registers)
constexpr uint32_t kLoopChain = 9;     // buckets of a chain that they look through: the first, and four at a time

// What the loop's steps may append is known when the call is made: each path's own future.  It goes
// to the histories behind the paths' ends beforehand (what lies there is not seen, see append and
// replay), so that a step has no histories to write and all that it reads of them is settled.
// A workgroup has the same 256 cells of every row_groups-th path.
static __global__ __launch_bounds__(256) void loop_fill_kernel(IndexView ix, const int32_t* future_tok,
                                                               const float* future_prob, int32_t ahead, int32_t chunks,
                                                               int32_t row_groups) {
  const int32_t first = (int32_t)blockIdx.x / chunks, t = ((int32_t)blockIdx.x - first * chunks) * 256 + (int32_t)threadIdx.x;
  for (int32_t row = first; row < ix.P * ix.N; row += row_groups) {
    const int32_t len = ix.meta_old[(int64_t)row * ix.meta_stride];
    if (t >= ahead || t >= ix.max_len - len) continue;
    const int64_t at = (int64_t)row * ix.max_len + len + t;
    ix.tok[at] = future_tok[at];
    ix.pq[at] = future_prob ? quantize_prob(future_prob[at]) : 65536u;
  }
}

struct LoopArgs {
  IndexView ix;
  int32_t steps;
  int32_t* targets;             // [rows][L] scratch, for the rows that a wave drafts
  int32_t* path_len;            // [steps][rows]
  DraftArgs a;                  // outputs of step 0; step t writes slice t
};

// A barrier behind which everything that the workgroup has stored is in the L2 (a workgroup's own fence waits
// for LDS alone, since its waves share a vector cache; the buckets are read past it).
__device__ __forceinline__ void memory_barrier() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The kernel's arguments, read anew: what is done with them here is not kept over the code around
// (of which there is not much room in scalar registers).
__device__ __forceinline__ const LoopArgs& loop_arguments() {
  auto* kernarg = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kernarg));
  return *(const LoopArgs*)kernarg;
}

// The steps of csd_accept_loop, one after the other.  A launch per step is bound by its latency:
// dispatch, then three round trips on caches that are cold at every launch, 6.6 us at 16 x 1024.
// Here a step's chain is the query's bucket, the postings' tokens, the matches' continuations and the
// walk, in caches that stay warm, and two barriers of the workgroup; the paths' ends and newest tokens
// are in LDS, the positions that the step itself appends are matched from a list of their hashes
// there, their claims travel during the look-up and the walk, and the outputs of a step behind the next
// one's barrier.  4.1 us a step (top to bucket 0.45, claims 0.2, look-up 0.8, postings 0.15, walk up to
// 1.7, the wait for the slowest wave's); one wave issues an instruction every 7 cycles here, so the
// instructions of the chain count.  With a wave per path (step_multi_kernel) the four SIMDs of the one
// CU had 1500 instructions a row and step to issue, 14 us; with sixteen lanes a path they have four
// waves of a few hundred.
// A row with up to sixteen matches is walked by group_walk, one with up to sixty-four by lanes_walk.  A row
// with more of them, a chain of more than kLoopChain buckets or a path shorter than a gram is drafted by a
// wave on the layout of a launch per step, behind a barrier, when the step's postings are in the
// index: code apart from the steps' (inlined into their loop it spilled their registers, 5.6 us a step).
// us a call, a launch per step / this (queries of three, drafts of eight, 48 steps): 1 problem of 16 paths
// x 1024 tokens 360 / 208, of 4 x 256 (24 steps) 161 / 81; 64 problems 543 / 253, 1024 of 16 x 512 (24
// steps) 2319 / 435; 24 paths x 1024 392 / 248, 64 problems of 32 x 512 (24 steps) 463 / 153.  Paths of
// different lengths that agree in all but 5 %, 2 % of their tokens: 16 x 1024 456 / 319, 455 / 323, 24 x 1024
// 481 / 423, 472 / 439.  Each gram twice, four times, six times in each path: 16 x 1024 458 / 359, 474 / 425,
// 526 / 474, 24 x 1024 503 / 445, 550 / 526, 692 / 1112; 64 times (24 steps) 16, 24 x 1024 2250 / 5270,
// 5270 / 19900: where most rows have more than sixty-four matches a few waves (as many as have room for that
// layout) draft them in turn.  (With sixteen matches and three buckets as the bounds, and the chains of full
// buckets followed one by one, 16 x 1024 with each gram twice, four times took 779, 1019, and 24 x 1024, all but
// 2 % equal, 737.)
// Exact matching through the index, DAG pool, queries of kmax = K tokens.
template <int LCAP, int WAVES, int K, bool BLOCKS>
__global__ __launch_bounds__(WAVES * kWave) void loop_kernel(LoopArgs m) {
  constexpr int G = kLoopLanes, kPaths = WAVES * kWave / G, BLOCK = WAVES * kWave;
  constexpr int kWide = WAVES < 4 ? WAVES : (WAVES == 4 ? 4 : 3);   // waves that draft the rows left (what the LDS has room for)
  constexpr int kBefore = 4;                             // tokens before a path's end that are kept
  constexpr int kOwn = (2 * LCAP + kBefore + 1 + G - 1) / G;   // words of a path's window that a lane has
  static_assert(kLoopChain + 4 <= kNear, "buckets of a gram's home block");
  static_assert(K >= 2 && K <= kBefore, "a gram's tokens in one load");
  __shared__ LdsWave wide[kWide];
  __shared__ int32_t own_all[kPaths][kOwn * G];          // tokens from kBefore before a path's end on, up to 2 L behind it
  __shared__ int2 fresh[kPaths * (LCAP + 1)];            // the step's new positions: packed, hash of the gram before them
  __shared__ int2 ends[kPaths];                          // lengths before and after the step's append
  __shared__ uint32_t found_all[kPaths][kLoopMatches];   // matches
  __shared__ int32_t draft_all[kPaths][LCAP], accepted_by_wave[kPaths];
  __shared__ int32_t n_fresh[2], n_crowded[2];           // (a step clears the next one's)
  __shared__ uint8_t crowded[kPaths];
  const IndexView& ix = m.ix;
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), sub = lane & (G - 1);
  const int32_t path = tid / G, p = (int32_t)blockIdx.x, N = ix.N, L = m.a.L;
  const bool on = path < N;
  const int64_t rows = (int64_t)ix.P * N;
  UnitRow u;
  u.i = path;
  u.first = p * N;
  u.row = u.first + (on ? path : 0);
  u.tok = ix.tok + (int64_t)u.first * ix.max_len;
  u.pq = ix.pq + (int64_t)u.first * ix.max_len;
  u.lens = nullptr;
  u.buckets = (int64_t)p * ((int64_t)ix.buckets.mask + 1);
  int32_t* gram = ix.gram + u.buckets * kBucketWords;
  const Buckets buckets{ix.buckets.mask, BLOCKS ? ix.buckets.block : ix.buckets.mask};
  const int32_t* history = ix.tok + (int64_t)u.row * ix.max_len;
  int32_t* own = own_all[path];
  uint32_t* found = found_all[path];
  auto group_bits = [&](bool x) { return (uint32_t)(wave_ballot(x) >> (lane & ~(G - 1))) & ((1u << G) - 1u); };
  int32_t window[kOwn];
  auto request_window = [&](int32_t end) {
#pragma unroll
    for (int x = 0; x < kOwn; ++x) {
      const int32_t t = end - kBefore + sub + x * G;
      window[x] = history[t < 0 ? 0 : (t < ix.max_len ? t : ix.max_len - 1)];
    }
  };
  auto keep_window = [&](int32_t end) {                  // (-1 beyond max_len: what no draft can meet)
#pragma unroll
    for (int x = 0; x < kOwn; ++x) own[sub + x * G] = end - kBefore + sub + x * G < ix.max_len ? window[x] : -1;
    block_sync<kWave>();                                 // (a path's lanes are of one wave)
  };
  int32_t old = ix.meta_old[(int64_t)u.row * ix.meta_stride];
  int32_t cnt = on && old < ix.max_len ? 1 : 0;          // tokens of this step
  if (tid < 2) n_fresh[tid] = n_crowded[tid] = 0;
  request_window(old);
  keep_window(old);
  lds_barrier<BLOCK>();
  uint32_t flags = 0;
  // outputs of the step before
  int32_t out_tok = 0, out_n = 0, accepted = 0;
  bool out_drafted = false;
  auto store_outputs = [&](int32_t t, int32_t len) {
    const int64_t row = t * rows + u.row;
    if (on && out_drafted) {
      if (sub < L) m.a.draft_tokens[row * L + sub] = out_tok;
      if (sub == 0) {
        m.a.draft_len[row] = out_n;
        m.a.accept_len[row] = accepted;
      }
    }
    if (on && sub == 0) m.path_len[row] = len;
  };
  bool leave = false;
  auto advance = [&]() {                                 // to what the next step appends
    const int32_t room = ix.max_len - (old + cnt);
    int32_t grow = accepted < L ? accepted + 1 : L + 1;
    grow = grow < room ? grow : room;
    old += cnt;
    cnt = on ? grow : 0;
    keep_window(old);
  };
  for (int32_t step = 0;;) {
    int32_t n_left = 0;
    while (step < m.steps) {                             // uniform over the workgroup, as n_left
      const int parity = step & 1;
      const int32_t now = old + cnt;
      int32_t Q[K], G0[K];
#pragma unroll
      for (int a = 0; a < K; ++a) Q[a] = own[kBefore - 1 + cnt - a];
      const GramHash gh = gram_hash_of(Q, K);
      // ---- round trip 1: the query's first bucket, past the CU's own cache (slots are claimed in the L2);
      // all postings of the steps before are there
      auto bucket = [&](uint32_t r) {
        return __hip_atomic_load(gram + (int64_t)gram_near(gh, r, buckets) * kBucketWords + sub, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
      };
      int32_t next = bucket(0);
      request_window(now);
      // the step's new positions, a lane each (drafts of sixteen tokens: one may go round again)
      auto gram_before = [&](int32_t t, int32_t (&g)[K]) {
#pragma unroll
        for (int a = 0; a < K; ++a) g[a] = own[kBefore - 1 + (t < cnt ? t : 0) - a];
      };
      auto filed = [&](int32_t t) { return t < cnt && old + t >= K; };
      auto packed = [&](int32_t t) { return (path << ix.eshift) | (old + t); };
      auto list = [&](int32_t t, const int32_t (&g)[K]) {
        const int32_t token = own[kBefore + (t < cnt ? t : 0)];
        flags |= t < cnt && (token < 0 || token >= ix.vocab) ? CSD_STATUS_TOKEN_RANGE : 0u;
        if (filed(t)) fresh[atomicAdd(&n_fresh[parity], 1)] = int2{packed(t), (int32_t)gram_hash_of(g, K).h};
      };
      gram_before(sub, G0);
      list(sub, G0);
      if (LCAP >= G && wave_ballot(sub + G < cnt) != 0) {
        int32_t g[K];
        gram_before(sub + G, g);
        list(sub + G, g);
      }
      if (sub == 0) ends[path] = int2{old, now};
      lds_barrier<BLOCK>();                              // the list, the ends
      if (tid == 0) n_fresh[parity ^ 1] = n_crowded[parity ^ 1] = 0;   // (everybody has read them, nobody adds to them before the next barrier)
      if (step > 0) store_outputs(step - 1, old);
      const bool is_short = now < K;
      bool looking = on && !is_short;
      int32_t M = 0;
      leave = is_short;
      // ---- round trip 2: a candidate's gram (with the continuations of all candidates it takes 1.9 us
      // instead of 1.1: the four waves share one cache that looks up a line a cycle)
      auto verify = [&](auto n, const bool (&one)[n()], const int32_t (&words)[n()], bool is_new) {
        bool cand[n()];
        int2 end[n()];
        Run4 r[n()];
#pragma unroll
        for (int x = 0; x < n(); ++x) {
          const int32_t j = words[x] >> ix.eshift, e = words[x] & ((1 << ix.eshift) - 1);
          cand[x] = one[x] && words[x] >= 0 && j != path && j < N;
          end[x] = ends[cand[x] ? j : 0];
          cand[x] = cand[x] && (is_new || e < end[x].x);   // (newer postings may be in flight: those are in the list)
          const int32_t cell = cand[x] ? (int32_t)__umul24((uint32_t)j, (uint32_t)ix.max_len) + e : K;
          r[x] = *reinterpret_cast<const Run4*>(u.tok + cell - K);
        }
#pragma unroll
        for (int x = 0; x < n(); ++x)
#pragma unroll
          for (int y = 0; y < K; ++y) consume_here(r[x].x[y]);
#pragma unroll
        for (int x = 0; x < n(); ++x) {
          int32_t differ = 0;
#pragma unroll
          for (int y = 0; y < K; ++y) differ |= r[x].x[y] ^ Q[K - 1 - y];
          const bool hit = cand[x] && differ == 0;
          const uint32_t hits = group_bits(hit);
          const int32_t to = M + (int32_t)__popc(hits & ((1u << sub) - 1u)), rem = end[x].y - (words[x] & ((1 << ix.eshift) - 1));
          if (hit && to < kLoopMatches) found[to] = (uint32_t)words[x] | (uint32_t)(rem < L ? rem : L) << 25;
          M += (int32_t)__popc(hits);
        }
      };
      auto look_up = [&]() {
        // four of the list's positions a lane at once (as a loop of one, every turn was a round trip in LDS)
        const int32_t listed = __builtin_amdgcn_readfirstlane(n_fresh[parity]);
        for (int32_t x0 = 0; x0 < listed; x0 += 4 * G) {
          int2 f[4];
#pragma unroll
          for (int y = 0; y < 4; ++y) f[y] = fresh[x0 + y * G + sub < listed ? x0 + y * G + sub : 0];
          uint32_t cands = 0;
#pragma unroll
          for (int y = 0; y < 4; ++y)
            cands |= looking && x0 + y * G + sub < listed && f[y].y == (int32_t)gh.h && f[y].x >> ix.eshift != path ? 1u << y : 0u;
          if (wave_ballot(cands != 0) != 0)
#pragma unroll
            for (int y = 0; y < 4; ++y) verify(std::integral_constant<int, 1>{}, {(cands >> y & 1u) != 0}, {f[y].x}, true);
        }
        constexpr int kAhead = 4;                        // buckets of a chain that are looked through together
        int32_t words[kAhead];
        auto request = [&](uint32_t r) {
#pragma unroll
          for (int x = 0; x < kAhead; ++x) words[x] = bucket(r + x);
        };
        auto count_of = [&](int32_t word) { return (int32_t)dpp_move<0x150>((uint32_t)word); };   // (the group's first lane has it)
        const int32_t count = count_of(next);
        const bool has_some = looking && sub >= 1 && sub - 1 < count;
        looking = looking && count >= kBucketSlots && ix.buckets.mask > 0;
        if (wave_ballot(looking) != 0) request(1);       // (in flight while the bucket before is looked through)
        verify(std::integral_constant<int, 1>{}, {has_some}, {next}, false);
        for (uint32_t r = 1; wave_ballot(looking) != 0; r += kAhead) {   // uniform over the wave
          int32_t these[kAhead];
          bool one[kAhead];
#pragma unroll
          for (int x = 0; x < kAhead; ++x) { these[x] = words[x]; consume_here(these[x]); }
#pragma unroll
          for (int x = 0; x < kAhead; ++x) {
            const int32_t filled = count_of(these[x]);
            one[x] = looking && sub >= 1 && sub - 1 < filled;
            looking = looking && filled >= kBucketSlots && r + x < ix.buckets.mask;
          }
          leave = leave || (looking && r + kAhead >= kLoopChain);
          looking = looking && !leave;
          if (wave_ballot(looking) != 0) request(r + kAhead);
          verify(std::integral_constant<int, kAhead>{}, one, these, false);
        }
      };
      Filing<K> filing;
      filing.claim(gram, buckets, K, G0, filed(sub), packed(sub));
      look_up();
      filing.settle();
      if (LCAP >= G && wave_ballot(sub + G < cnt) != 0) {
        int32_t g[K];
        gram_before(sub + G, g);
        file_positions<false, K>(gram, buckets, K, g, filed(sub + G), packed(sub + G), lane, [] {});
      }
      // ---- the walk, by as many lanes of a path as the wave's paths have matches
      leave = on && (leave || M > kLoopMatches);
      block_sync<kWave>();
      const bool drafts = on && !leave, walks = drafts && M > 0;
      int32_t n = 0;
      if (wave_ballot(walks) != 0) {                     // uniform over the wave
        const uint32_t match = walks && sub < M ? found[sub] : 0u;
        auto chosen = [&](auto layer, bool going, const Cand& best) {
          if (sub == 0) draft_all[path][layer() - 1] = best.v;
          n = going ? layer() : n;
        };
        auto walk = [&](auto lanes, auto edge) {
          int32_t v[1][LCAP], pr[1][LCAP];
          read_windows<LCAP, 1>(ix, u, {match}, v, pr);
          group_walk<lanes(), LCAP, edge()>(m.a, match, v[0], pr[0], walks, chosen);
        };
        auto weighed = [&](auto edge) {
          auto several = [&](auto n) {                   // matches a lane
            uint32_t matches[n()];
#pragma unroll
            for (int x = 0; x < n(); ++x) matches[x] = walks && sub + x * G < M ? found[sub + x * G] : 0u;
            int32_t v[n()][LCAP], pr[n()][LCAP];
            read_windows<LCAP, n()>(ix, u, matches, v, pr);
            lanes_walk<n(), LCAP, edge()>(m.a, matches, v, pr, walks, chosen);
          };
          if (wave_ballot(walks && M > 4) == 0) walk(std::integral_constant<int, 4>{}, edge);
          else if (wave_ballot(walks && M > 8) == 0) walk(std::integral_constant<int, 8>{}, edge);
          else if (wave_ballot(walks && M > G) == 0) walk(std::integral_constant<int, G>{}, edge);
          else if (wave_ballot(walks && M > 2 * G) == 0) several(std::integral_constant<int, 2>{});
          else several(std::integral_constant<int, kLoopMatches / G>{});
        };
        if (m.a.score_mode == 0) weighed(std::false_type{});
        else weighed(std::true_type{});
      }
      filing.finish();
      n = (int32_t)dpp_move<0x150>((uint32_t)n);
      block_sync<kWave>();                               // the draft's tokens
      const int32_t drafted = draft_all[path][sub < LCAP ? sub : 0];
      const uint32_t stops = group_bits(!(sub < n && drafted == own[kBefore + cnt + (sub < L ? sub : 0)])) | 1u << G;
      accepted = (int32_t)__ffs(stops) - 1;
      out_tok = sub < n ? drafted : -1;
      out_n = n;
      out_drafted = drafts;
      if (leave && sub == 0) crowded[atomicAdd(&n_crowded[parity], 1)] = (uint8_t)path;
      memory_barrier();                                  // the step's postings are in the L2
      n_left = __builtin_amdgcn_readfirstlane(n_crowded[parity]);
      if (n_left > 0) break;
      advance();
      ++step;
    }
    if (n_left == 0) {
      if (step > 0) store_outputs(step - 1, old);
      break;
    }
    // ---- rows that are left to a wave
    {
      const LoopArgs& args = loop_arguments();
      const IndexView& in_place = args.ix;
      int32_t t = tid;
      consume_here(t);
      const int32_t wave = __builtin_amdgcn_readfirstlane(t >> 6), now = old + cnt;
      if (on && sub <= in_place.tail_len)
        in_place.meta_new[(int64_t)u.row * in_place.meta_stride + sub] = sub == 0 ? now : (sub <= now ? own[kBefore + cnt - sub] : 0);
      if (leave && sub < args.a.L) args.targets[(int64_t)u.row * args.a.L + sub] = own[kBefore + cnt + sub];
      memory_barrier();                                  // ends and targets are in memory, as the step's postings are
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      for (int32_t x = wave; wave < kWide && x < n_left; x += kWide) {
        const LoopArgs& again = loop_arguments();
        IndexView v = again.ix;
        v.meta_old = v.meta_new;
        DraftArgs b = again.a;
        const int64_t before = step * ((int64_t)v.P * v.N);
        b.draft_tokens += before * b.L;
        b.draft_len += before;
        b.accept_len += before;
        b.targets = again.targets;
        const int32_t row = (int32_t)blockIdx.x * v.N + __builtin_amdgcn_readfirstlane((int)crowded[x]);
        row_step<LCAP, false, LdsWave, false, 4, false>(wide[wave], v, StepIn{nullptr, nullptr, nullptr, 0}, b,
                                                        AcceptTail{accepted_by_wave}, row, t & (kWave - 1));
        block_sync<kWave>();
      }
      __syncthreads();
      accepted = leave ? accepted_by_wave[path] : accepted;
    }
    advance();
    ++step;
  }
  if (on && sub <= ix.tail_len)
    ix.meta_new[(int64_t)u.row * ix.meta_stride + sub] = sub == 0 ? old : (sub <= old ? own[kBefore - sub] : 0);
  if (flags) atomicOr(ix.status, flags);
}

// As many waves as the paths need, since the LDS of four has room for one workgroup a CU.  us, this / four
// waves up to sixteen paths (24 steps): 1024 problems of 4 x 256 110 / 318, 1024 of 8 x 256 202 / 359, 64 of
// 8 x 512 104 / 103, 1 of 4 x 256 82 / 85.
template <int LCAP, int K>
void launch_loop_kernel(const LoopArgs& m, hipStream_t st) {
  auto of = [&](auto waves, auto blocks) {
    constexpr int WAVES = waves();
    loop_kernel<LCAP, WAVES, K, blocks()><<<(uint32_t)m.ix.P, WAVES * kWave, 0, st>>>(m);
  };
  const std::integral_constant<int, 4> four;
  const std::integral_constant<int, 8> eight;
  if (m.ix.buckets.mask > m.ix.buckets.block) {          // (of few problems: the LDS has room)
    if (m.ix.N <= 16) of(four, std::true_type{});
    else of(eight, std::true_type{});
  } else if (m.ix.N <= 4) of(std::integral_constant<int, 1>{}, std::false_type{});
  else if (m.ix.N <= 8) of(std::integral_constant<int, 2>{}, std::false_type{});
  else if (m.ix.N <= 16) of(four, std::false_type{});
  else of(eight, std::false_type{});
}

}  // namespace csd
