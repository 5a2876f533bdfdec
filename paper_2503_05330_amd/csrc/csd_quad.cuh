// csd — drafts of rows with few matches, four or eight lanes per row: for launches of many
// thousand drafts (a replay's steps side by side), which are bound by the instructions that all
// rows issue.
#pragma once

#include "csd_common.cuh"
#include "csd_index.cuh"

namespace csd {

constexpr int kQuadRows = kWave / 4;   // rows of a wave with a quad of lanes each

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
// x of another lane of a group of G, each of them for one R = 1 .. G - 1: lane ^ R, or (G = 16) the lane
// that a rotation by R brings here
template <int G, int R>
__device__ __forceinline__ uint32_t group_other(uint32_t x) {
  static_assert((G == 2 || G == 4 || G == 8 || G == 16) && R >= 1 && R < G, "a pair, a quad, half a DPP row or a whole one");
  if constexpr (G == 16) return dpp_move<0x120 + R>(x);
  constexpr int kFlip = R < 4 ? R : 7 - R;               // within a quad; R >= 4: behind the half row's mirror (^ 7)
  constexpr int kQuad = kFlip == 1 ? 0xB1 : kFlip == 2 ? 0x4E : 0x1B;
  if constexpr (R >= 4) x = dpp_move<0x141>(x);
  return kFlip == 0 ? x : dpp_move<kQuad>(x);
}
// f(a lane move), so that every lane of the group ends with what all of them have, for operations
// that may meet a value twice
template <int CTRL>
struct DppMove {
  __device__ __forceinline__ uint32_t operator()(uint32_t x) const { return dpp_move<CTRL>(x); }
};
template <int G, class F>
__device__ __forceinline__ void group_stages(F&& f) {
  f(DppMove<0xB1>{});                                    // lane ^ 1
  if constexpr (G >= 4) f(DppMove<0x4E>{});              // ^ 2
  if constexpr (G >= 8) f(DppMove<0x141>{});             // the half row's mirror
  if constexpr (G >= 16) f(DppMove<0x140>{});            // the row's
}

struct __attribute__((packed, aligned(4))) Run4 { int32_t x[4]; };   // four words at any of them

// The draft of a lane's unit (see replay_unit): where its data lies.
struct UnitRow {
  int32_t i, row, first;        // path; row among all steps' rows; the problem's first row at this step
  const int32_t *tok, *lens;    // the problem's histories; its paths' ends at this step
  const uint32_t* pq;
  int64_t buckets;              // the problem's first bucket
  UnitRow() = default;
  __device__ __forceinline__ UnitRow(const IndexView& ix, uint32_t steps, uint32_t unit) {
    const uint32_t N = (uint32_t)ix.N;
    const uint32_t p = unit / (N * steps), in_problem = unit - p * (N * steps), t = in_problem / N;
    i = (int32_t)(in_problem - t * N);
    first = (int32_t)(t * (uint32_t)ix.P * N + p * N);
    row = first + i;
    const int64_t cells = (int64_t)(p * N) * ix.max_len;
    tok = ix.tok + cells;
    pq = ix.pq + cells;
    lens = ix.meta_old + (int64_t)first * ix.meta_stride;
    buckets = (int64_t)p * ((int64_t)ix.buckets.mask + 1);
  }
  // the path's length and newest tokens (newest first)
  template <int QC>
  __device__ __forceinline__ int32_t end(const IndexView& ix, int32_t (&Q)[QC]) const {
    const int32_t* meta = lens + i * ix.meta_stride;
    const int4 m0 = *reinterpret_cast<const int4*>(meta);
    const int4 m1 = QC > 3 ? *reinterpret_cast<const int4*>(meta + (ix.kmax > 3 ? 4 : 0)) : int4{0, 0, 0, 0};
    const int32_t tail[8] = {m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w, QC > 7 ? meta[ix.kmax > 7 ? 8 : 0] : 0};
#pragma unroll
    for (int x = 0; x < QC; ++x) Q[x] = tail[x];
    return m0.x;
  }
};

template <int QC>
__device__ __forceinline__ GramHash gram_hash_of(const int32_t (&Q)[QC], int32_t kmax) {
  uint32_t acc = kGramSeed;
#pragma unroll
  for (int x = 0; x < QC; ++x)
    if (x < kmax) acc = gram_hash_add(acc, Q[x]);
  return gram_hash_end(acc, kmax);
}

// Files the new position of each lane (see file_positions) in three parts: the claims on the first buckets
// of the chains, the fill counts of the next four where those were full, and the claims there.  What lies
// between them (the look-up and the walk of a loop's step) has their round trips.  K: compile-time bound of kmax.
template <int K>
struct Filing {
  static constexpr int kAhead = 4;
  int32_t* gram = nullptr;
  Buckets buckets{0u, 0u};
  GramHash gh{0u, 1u};
  int32_t pos = 0, claimed = kBucketSlots;
  bool open = false;            // no slot yet
  int32_t fill[kAhead];
  __device__ __forceinline__ void look(uint32_t r) {
    if (!open) return;
#pragma unroll
    for (int x = 0; x < kAhead; ++x)
      fill[x] = __hip_atomic_load(gram_bucket(gram, gh, r + x, buckets), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ void claim(int32_t* table, Buckets of_problem, int32_t kmax, const int32_t (&G)[K], bool mine, int32_t packed) {
    gram = table;
    buckets = of_problem;
    gh = gram_hash_of(G, kmax);
    pos = packed;
    open = mine;
    claimed = kBucketSlots;
    if (mine) claimed = atomicAdd(gram_bucket_near(gram, gh, 0, buckets), 1);
  }
  __device__ __forceinline__ void settle() {
    if (claimed < kBucketSlots) {
      gram_bucket_near(gram, gh, 0, buckets)[1 + claimed] = pos;
      open = false;
    }
    if (wave_ballot(open) != 0) look(1);
  }
  __device__ __forceinline__ void finish() {             // (what finds no slot in a full index is dropped)
    const uint32_t turns = gram_turns(buckets);
    for (uint32_t r = 1; r < turns && wave_ballot(open) != 0; r += kAhead) {   // uniform over the wave
      if (r > 1) look(r);
      uint32_t room = 0;
#pragma unroll
      for (int x = 0; x < kAhead; ++x) room |= open && fill[x] < kBucketSlots && r + x < turns ? 1u << x : 0u;
      while (wave_ballot(room != 0) != 0) {
        if (room != 0) {
          int32_t* b = gram_bucket(gram, gh, r + (uint32_t)__ffs(room) - 1u, buckets);
          const int32_t c = atomicAdd(b, 1);
          if (c < kBucketSlots) b[1 + c] = pos;
          open = c >= kBucketSlots;
          room = open ? room & (room - 1u) : 0u;
        }
      }
    }
  }
};

// A posting of a bucket: what it takes to verify it, loaded without a branch (an idle one reads the
// problem's first cell).
template <int QC>
struct Posting {
  bool cand;
  int32_t e, len, gram[QC];
  __device__ __forceinline__ void load(const IndexView& ix, const UnitRow& u, bool is_one, int32_t word) {
    const int32_t j = word >> ix.eshift;
    e = word & ((1 << ix.eshift) - 1);
    cand = is_one && word >= 0 && j != u.i && j < ix.N;
    len = u.lens[cand ? j * ix.meta_stride : 0];
    const int32_t* at = u.tok + (cand ? (int32_t)__umul24((uint32_t)j, (uint32_t)ix.max_len) + e - ix.kmax : 0);
#pragma unroll
    for (int y = 0; y < QC; y += 4) {
      const Run4 r = *reinterpret_cast<const Run4*>(at + y);
#pragma unroll
      for (int z = 0; z < 4; ++z) gram[y + z] = r.x[z];
    }
  }
  // (several postings' loads are in flight before the first is looked at: left to itself the
  // compiler loads behind the comparisons)
  __device__ __forceinline__ void arrive() {
    consume_here(len);
#pragma unroll
    for (int y = 0; y < QC; ++y) consume_here(gram[y]);
  }
  __device__ __forceinline__ bool hit(const int32_t (&Q)[QC], int32_t kmax) const {
    int32_t differ = 0;                                  // gram: oldest token first
#pragma unroll
    for (int y = 0; y < QC; ++y) differ |= y < kmax ? gram[y] ^ pick(Q, kmax - 1 - y) : 0;
    return cand && e < len && differ == 0;
  }
  // position and layers that the match reaches, in one word
  __device__ __forceinline__ uint32_t packed(int32_t word, int32_t L) const {
    return (uint32_t)word | (uint32_t)(len - e < L ? len - e : L) << 25;
  }
};

// The continuations of S matches (as packed above; 0: none) from the problem's histories in memory.
template <int LCAP, int S>
__device__ __forceinline__ void read_windows(const IndexView& ix, const UnitRow& u, const uint32_t (&match)[S],
                                             int32_t (&v)[S][LCAP], int32_t (&pr)[S][LCAP]) {
#pragma unroll
  for (int x = 0; x < S; ++x) {
    const int32_t pos = (int32_t)(match[x] & ((1u << 25) - 1u));
    const int32_t cell = (int32_t)__umul24((uint32_t)(pos >> ix.eshift), (uint32_t)ix.max_len) +
                         (pos & ((1 << ix.eshift) - 1));
#pragma unroll
    for (int d = 0; d < LCAP; d += 4) {
      const Run4 r = *reinterpret_cast<const Run4*>(u.tok + cell + d);
      const Run4 s = *reinterpret_cast<const Run4*>(u.pq + cell + d);
#pragma unroll
      for (int z = 0; z < 4; ++z) {
        v[x][d + z] = r.x[z];
        pr[x][d + z] = s.x[z];
      }
    }
  }
#pragma unroll
  for (int x = 0; x < S; ++x)
#pragma unroll
    for (int d = 0; d < LCAP; ++d) {
      consume_here(v[x][d]);
      consume_here(pr[x][d]);
    }
}

// The greedy walk of a row from its matches, one per lane of its group (`match`: as packed above; 0:
// none; v, pr: its continuation): layer by layer Eq. 5's sums and the greedy rule (as in
// walk_instances) by exchanges within the group.  going: the same in a group's lanes.
// EDGE: edges are weighed, not nodes (score_mode 1; asked at every exchange of every layer it was a
// branch each).  chosen(layer, going, best): the layer's choice, where going.
template <int G, int LCAP, bool EDGE, class CHOSEN>
__device__ __forceinline__ void group_walk(const DraftArgs& a, uint32_t match, const int32_t (&v)[LCAP],
                                           const int32_t (&pr)[LCAP], bool going, CHOSEN&& chosen) {
  constexpr int kCount = 24;                             // count (<= 16) above the probability sum (<= 2^20)
  const int32_t rem = (int32_t)(match >> 25);            // (at most L)
  int32_t cur = 0;
  static_for<1, LCAP + 1>([&](auto layer) {
    constexpr int d = layer();
    constexpr bool kByEdge = EDGE && d > 1;
    if (wave_ballot(going) == 0) return;                 // uniform over the wave; so from the layer behind L on
    const bool alive = d <= rem;
    const uint32_t vd = (uint32_t)v[d - 1], ud = d > 1 ? (uint32_t)v[d > 1 ? d - 2 : 0] : 0u;
    const bool from_cur = alive && going && (d == 1 || (int32_t)ud == cur);
    // the lanes with the same token (score_mode 1: with the same predecessor too)
    const uint32_t own = alive ? (1u << kCount) + (uint32_t)pr[d - 1] : 0u;
    uint32_t cs = own;
    // (the moves are made before the comparisons: in a lane that a condition rules out, a move
    // delivers nothing to the others)
    static_for<1, G>([&](auto r) {
      const uint32_t other_v = group_other<G, r()>(vd), other = group_other<G, r()>(own);
      bool same_node = other_v == vd;
      if constexpr (kByEdge) {
        const uint32_t other_u = group_other<G, r()>(ud);
        same_node = same_node && other_u == ud;
      }
      cs += same_node ? other : 0u;
    });
    // the heaviest weight, then the lowest token that has it
    const u64 weight = weight_key(pack_cs(cs >> kCount, cs & ((1u << kCount) - 1u)), a.alpha_q);
    u64 key = from_cur ? weight : 0ull;
    group_stages<G>([&](auto other) {
      const uint32_t lo = other((uint32_t)key), hi = other((uint32_t)(key >> 32));
      const u64 theirs = ((u64)hi << 32) | lo;
      key = theirs > key ? theirs : key;
    });
    int32_t token = from_cur && weight == key ? (int32_t)vd : INT_MAX;
    group_stages<G>([&](auto other) {
      const int32_t theirs = (int32_t)other((uint32_t)token);
      token = theirs < token ? theirs : token;
    });
    going = going && token != INT_MAX;                   // else a leaf: no edge leaves cur
    cur = token;
    chosen(layer, going, Cand{key, token});
  });
}

// group_walk for rows of seventeen to sixty-four matches, S of them a lane of the sixteen: in each layer the
// tokens that follow the last choice are taken up one after the other, the lowest first, each with what all
// lanes have of it, until those left could not outweigh the heaviest together.  (Every lane against every other, as there, is 4 S times the exchanges of sixteen
// matches; here it is as many rounds as there are different tokens, few where the paths agree.)
template <int S, int LCAP, bool EDGE, class CHOSEN>
__device__ __forceinline__ void lanes_walk(const DraftArgs& a, const uint32_t (&match)[S], const int32_t (&v)[S][LCAP],
                                           const int32_t (&pr)[S][LCAP], bool going, CHOSEN&& chosen) {
  constexpr int kCount = 24;                             // count (<= 64) above the probability sum (<= 2^22)
  static_assert(S <= 4, "the sums of a layer in one word");
  int32_t cur = 0;
  static_for<1, LCAP + 1>([&](auto layer) {
    constexpr int d = layer();
    if (wave_ballot(going) == 0) return;                 // uniform over the wave; so from the layer behind L on
    uint32_t own[S];
    int32_t left[S];                                     // successors of the last choice that are still to be taken up
#pragma unroll
    for (int x = 0; x < S; ++x) {
      const bool alive = d <= (int32_t)(match[x] >> 25);
      const bool from_cur = alive && going && (d == 1 || v[x][d > 1 ? d - 2 : 0] == cur);
      own[x] = (EDGE ? from_cur : alive) ? (1u << kCount) + (uint32_t)pr[x][d - 1] : 0u;
      left[x] = from_cur ? v[x][d - 1] : INT_MAX;
    }
    uint32_t rest = 0;                                   // what the layer's tokens that are not taken up yet have in all
#pragma unroll
    for (int x = 0; x < S; ++x) rest += own[x];
    auto weight = [&](uint32_t cs) { return weight_key(pack_cs(cs >> kCount, cs & ((1u << kCount) - 1u)), a.alpha_q); };
    auto lowest_and_sum = [&](uint32_t& sum) {
      int32_t token = left[0];
#pragma unroll
      for (int x = 1; x < S; ++x) token = left[x] < token ? left[x] : token;
      group_stages<16>([&](auto other) {
        const int32_t theirs = (int32_t)other((uint32_t)token);
        token = theirs < token ? theirs : token;
        sum += other(sum);                               // (each stage brings other lanes' sums)
      });
      return token;
    };
    int32_t token = lowest_and_sum(rest);
    Cand best = cand_none();
    while (wave_ballot(token != INT_MAX && (best.v == INT_MAX || weight(rest) > best.key)) != 0) {   // uniform over the wave
      uint32_t cs = 0;
#pragma unroll
      for (int x = 0; x < S; ++x) {
        cs += v[x][d - 1] == token ? own[x] : 0u;
        left[x] = left[x] == token ? INT_MAX : left[x];
      }
      const int32_t next = lowest_and_sum(cs);
      const u64 key = weight(cs);
      if (token != INT_MAX && (best.v == INT_MAX || key > best.key)) best = Cand{key, token};
      rest -= token != INT_MAX ? cs : 0u;
      token = next;
    }
    going = going && best.v != INT_MAX;                  // else a leaf: no edge leaves cur
    cur = best.v;
    chosen(layer, going, best);
  });
}

// A draft as a group of lanes has it: lane `sub` keeps the choices of the layers sub * kKept + 1 and on.
template <int G, int LCAP>
struct GroupDraft {
  static constexpr int kKept = (LCAP + G - 1) / G;
  int32_t tok[kKept], n = 0;
  u64 key[kKept], key_sum = 0;
  __device__ __forceinline__ GroupDraft() {
#pragma unroll
    for (int x = 0; x < kKept; ++x) {
      tok[x] = -1;
      key[x] = 0;
    }
  }
  __device__ __forceinline__ void choose(int32_t d, bool going, const Cand& best, int sub) {
    n = going ? d : n;
    key_sum += going ? best.key : 0ull;
#pragma unroll
    for (int x = 0; x < kKept; ++x) {
      const bool keep = going && sub * kKept + x == d - 1;
      tok[x] = keep ? best.v : tok[x];
      key[x] = keep ? best.key : key[x];
    }
  }
  // the outputs of the rows with `write` (n and key_sum: of the group's first lane)
  __device__ __forceinline__ void store(const DraftArgs& a, int64_t row, bool write, int sub, const int32_t (&target)[kKept]) const {
    const int32_t L = a.L;
    int32_t same = 0;                                    // of this lane's layers, from its first on
    bool all = true;
#pragma unroll
    for (int x = 0; x < kKept; ++x) {
      const int32_t d = sub * kKept + x;
      all = all && d < n && target[x] == tok[x];
      same += all ? 1 : 0;
      if (write && d < L) {
        a.draft_tokens[row * L + d] = tok[x];
        if (a.token_scores) a.token_scores[row * L + d] = key_to_score(key[x]);
      }
    }
    if (a.targets) {                                     // the first layer that differs
      uint32_t stop = all ? (uint32_t)LCAP : (uint32_t)(sub * kKept + same);
      group_stages<G>([&](auto move) {
        const uint32_t other = move(stop);
        stop = other < stop ? other : stop;
      });
      if (write && sub == 0) a.accept_len[row] = (int32_t)stop < n ? (int32_t)stop : n;
    }
    if (write && sub == 0) {
      a.draft_len[row] = n;
      if (a.path_scores) a.path_scores[row] = key_to_score(key_sum);
    }
  }
};

// The draft of a row whose matches, one a lane, are in the histories in memory, and its outputs.
template <int G, int LCAP, bool EDGE>
__device__ __forceinline__ void group_draft(const IndexView& ix, const DraftArgs& a, const UnitRow& u, uint32_t match,
                                            bool write, int sub, const int32_t (&target)[(LCAP + G - 1) / G]) {
  int32_t v[1][LCAP], pr[1][LCAP];
  read_windows<LCAP, 1>(ix, u, {match}, v, pr);
  GroupDraft<G, LCAP> draft;
  group_walk<G, LCAP, EDGE>(a, match, v[0], pr[0], write,
                            [&](auto layer, bool going, const Cand& best) { draft.choose(layer(), going, best, sub); });
  draft.store(a, u.row, write, sub, target);
}

// The targets of the layers that this lane keeps.
template <int G, int LCAP>
__device__ __forceinline__ void load_targets(const DraftArgs& a, const UnitRow& u, int sub,
                                             int32_t (&target)[(LCAP + G - 1) / G]) {
  constexpr int kKept = (LCAP + G - 1) / G;
#pragma unroll
  for (int x = 0; x < kKept; ++x) {
    const int32_t d = sub * kKept + x;
    target[x] = a.targets ? a.targets[(int64_t)u.row * a.L + (d < a.L ? d : 0)] : 0;
  }
}

// The first of this workgroup's `per_block` units: XCD x takes a contiguous range of the units.
__device__ __forceinline__ uint32_t block_units(uint32_t per_block) {
  return ((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3)) * per_block;
}

// One draft per quad of lanes, sixteen per wave: exact matching through the index, DAG pool, query
// of kmax tokens.  A lane takes four words of the row's first bucket, verifies its postings against
// the histories, and the row's matches (at most four) go to a lane each.  No tables, no loop over
// matches, and a wave's scalar instructions are shared by sixteen rows: with a wave per row those
// kept the scalar unit busiest (539 scalar and 350 vector instructions a row; here 20 and 54).
// What is left: four dependent round trips, whose loads gather 64 lines each.  Rows whose bucket is full (their chain may
// go on), that have more than four matches or fewer tokens than a gram are left to the next
// kernel: bit 4 r of rest[w] is row r of wave w.  (A list of them with one counter took 12 ns per
// wave, the rate of atomics on one address, and its order spread a problem's rows over all L2s.)
// ix.meta_old and a are those of the first step.
template <int LCAP, int QC, bool EDGE>
__global__ __launch_bounds__(256) void replay_quad_kernel(IndexView ix, int32_t steps, DraftArgs a, u64* rest) {
  __shared__ uint32_t found[256];                        // [row of the workgroup][4] matches
  const int tid = (int)threadIdx.x, lane = tid & (kWave - 1), sub = tid & 3;
  const uint32_t unit = block_units(4 * kQuadRows) + (uint32_t)(tid >> 2);
  const bool on = unit < (uint32_t)(ix.P * ix.N * steps);
  const UnitRow u(ix, (uint32_t)steps, on ? unit : 0u);
  // ---- round trip 1: the path's end
  int32_t Q[QC], target[LCAP / 4];
  const int32_t len = u.end(ix, Q);
  load_targets<4, LCAP>(a, u, sub, target);
  // ---- round trip 2: the first bucket of the query
  const int64_t bucket = u.buckets + (gram_hash_of(Q, ix.kmax).h & ix.buckets.mask);
  const int4 w4 = *reinterpret_cast<const int4*>(ix.gram + bucket * kBucketWords + 4 * sub);
  const int32_t word[4] = {w4.x, w4.y, w4.z, w4.w};
  const int32_t count = (int32_t)dpp_move<0x00>((uint32_t)word[0]);
  bool leave = len < ix.kmax || count >= kBucketSlots;   // to the next kernel
  // ---- round trip 3: every posting's gram and its path's length
  Posting<QC> post[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int32_t slot = 4 * sub + x - 1;
    post[x].load(ix, u, !leave && slot >= 0 && slot < count, word[x]);
  }
  uint32_t hits = 0;
#pragma unroll
  for (int x = 0; x < 4; ++x) post[x].arrive();
#pragma unroll
  for (int x = 0; x < 4; ++x) hits |= post[x].hit(Q, ix.kmax) ? 1u << x : 0u;
  // the row's matches, one per lane
  const uint32_t mine = __popc(hits);
  const uint32_t n0 = dpp_move<0x00>(mine), n1 = dpp_move<0x55>(mine), n2 = dpp_move<0xAA>(mine), n3 = dpp_move<0xFF>(mine);
  const int32_t M = (int32_t)(n0 + n1 + n2 + n3);
  leave = leave || M > 4;
  uint32_t to = (sub > 0 ? n0 : 0u) + (sub > 1 ? n1 : 0u) + (sub > 2 ? n2 : 0u);
#pragma unroll
  for (int x = 0; x < 4; ++x)
    if (hits >> x & 1u) {
      if (to < 4) found[(tid & ~3) + to] = post[x].packed(word[x], a.L);
      ++to;
    }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // (a row's lanes are of one wave)
  // ---- round trip 4: the matches' continuations; walk, outputs
  group_draft<4, LCAP, EDGE>(ix, a, u, !leave && sub < M ? found[tid] : 0u, on && !leave, sub, target);
  const u64 left = wave_ballot(on && leave && sub == 0);
  if (lane == 0 && on) rest[unit / kQuadRows] = left;
}

// Rows for the kernels with a wave per row: a list per XCD, of the units that it has drafted from its
// L2 already, the rows with few matches from the front on, the others from the back (of a staged replay, which
// lists only those, from the front: the last XCD's part may be larger than its rows).
struct RestList {
  static constexpr int kSet = 16 * kBucketWords;         // a counter for each list, a line apart (an atomic takes one 12 ns)
  static constexpr int kCounters = 2 * kSet + 8 * kBucketWords;
  int32_t* counts;              // zeroed by the launch before the one that lists
  int32_t* units;               // [8][capacity]
  int32_t capacity;             // units of an XCD
  int32_t* readers;             // or null.  A line for each XCD: workgroups that have read its counters, of which
                                //   the last zeroes them and this, for the next launch that lists
  // words: of the workspace, all counters and then the units.  staged: the second set of counters, which nobody
  // zeroes beforehand
  static RestList in(int32_t* words, bool staged, int32_t capacity) {
    return RestList{words + (staged ? kSet : 0), words + kCounters, capacity, staged ? words + 2 * kSet : nullptr};
  }
  __device__ __forceinline__ int32_t* count(uint32_t xcd, bool many) const { return counts + (2 * xcd + many) * kBucketWords; }
  __device__ __forceinline__ int32_t* unit(uint32_t xcd, bool many, int32_t nth) const {
    return units + (int32_t)xcd * capacity + (many && !readers ? capacity - 1 - nth : nth);
  }
};
constexpr int32_t kRestPad = 8 * 256;  // units by which the lists of all XCDs may exceed the drafts

// The same with eight lanes per row, for the rows that replay_quad_kernel has left: the first
// buckets of the query's chain, up to eight matches.  A workgroup pools the rows that WAVES waves of
// that kernel have left (one in eight, most of them because their first bucket is full), and its
// waves take eight each.  A turn is a chain of five to nine round trips, so what counts is one
// turn for most waves and all of them resident at once: 1024 problems x 24 steps 74 us with the rows
// of four waves pooled, 60 with those of sixteen.  It lists the rows with more matches or a
// longer chain for the kernels with a wave per row (one reservation: atomics on one address take 12 ns
// each).  A chain is followed to its end, or for kLongChain buckets, also when the row's matches
// are too many: it tells the rows with more than few_matches, which that kernel may draft with
// another layout (any serves any row), and where the chain goes on those that had more than eight so far.
// 1024 problems x 24 steps leave 8000 of 393000 rows: 4130 whose chain has ended (3180 with 9 .. 16
// matches, 950 up to 30, 18 more) and 3920 with longer chains (2320 with up to eight so far, 1120, 470).
constexpr int32_t few_matches(int32_t L) { return L <= 24 ? 30 : 24; }   // (what the small layout has windows for)
constexpr uint32_t kLongChain = 3;     // buckets after which the wave per row, which reads four at once, takes over
template <int WAVES, int LCAP, int QC, bool EDGE>
__global__ __launch_bounds__(256) void replay_eight_kernel(IndexView ix, int32_t steps, DraftArgs a, const u64* rest,
                                                           RestList list) {
  constexpr int G = 8, kWaves = 4, kRows = WAVES * kQuadRows;   // rows of the workgroup
  static_assert(kLongChain <= kNear, "buckets of a gram's home block");
  static_assert(WAVES <= kWave && kRows <= 256, "a lane per wave of the other kernel, a byte per row");
  __shared__ uint32_t found_all[kWaves][kWave];          // [row of the turn][8] matches
  __shared__ uint8_t todo[kRows], left[2][kRows];        // left: few matches, many
  __shared__ int32_t n_todo, n_left[2], list_at[2];
  const int lane = (int)threadIdx.x & (kWave - 1), wave = (int)threadIdx.x >> 6, sub = lane & (G - 1);
  uint32_t* found = found_all[wave];
  const uint32_t units = (uint32_t)(ix.P * ix.N * steps), first = block_units(kRows);
  if (wave == 0) {                                       // the rows' numbers, one after the other
    u64 rows = 0;
    if (lane < WAVES && first + (uint32_t)(lane * kQuadRows) < units) rows = rest[first / kQuadRows + lane];
    int32_t at = 0, total = 0;
#pragma unroll
    for (int x = 0; x < WAVES; ++x) {
      const int32_t n = __builtin_amdgcn_readlane((int)__popcll(rows), x);
      at = lane == x ? total : at;
      total += n;
    }
    for (; rows; rows &= rows - 1) todo[at++] = (uint8_t)(lane * kQuadRows + (((int)__ffsll((long long)rows) - 1) >> 2));
    if (lane == 0) {
      n_todo = total;
      n_left[0] = n_left[1] = 0;
    }
  }
  __syncthreads();
  const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane(n_todo);
  for (uint32_t turn = (uint32_t)(wave * (kWave / G)); turn < total; turn += kWaves * (kWave / G)) {   // uniform over the wave
    const uint32_t nth = turn + (uint32_t)(lane / G);
    const bool on = nth < total;
    const uint32_t which = todo[on ? nth : turn];
    const UnitRow u(ix, (uint32_t)steps, first + which);
    int32_t Q[QC], target[(LCAP + G - 1) / G];
    const int32_t len = u.end(ix, Q);
    load_targets<G, LCAP>(a, u, sub, target);
    const GramHash gh = gram_hash_of(Q, ix.kmax);
    const bool is_short = len < ix.kmax;                 // no gram to look up: scanned for
    bool leave = is_short;
    int32_t M = 0;
    bool looking = on && !leave;                         // the same in a group's lanes
    auto bucket = [&](uint32_t r) {
      const int64_t b = u.buckets + gram_near(gh, r, ix.buckets);
      return *reinterpret_cast<const int2*>(ix.gram + b * kBucketWords + 2 * sub);
    };
    int2 next = bucket(0);
    for (uint32_t r = 0; wave_ballot(looking) != 0; ++r) {   // uniform over the wave
      const int2 w = next;
      next = bucket(r + 1);                              // (in flight while this one is looked through)
      const int32_t word[2] = {w.x, w.y}, count = __shfl(w.x, lane & ~(G - 1));
      Posting<QC> post[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const int32_t slot = 2 * sub + x - 1;
        post[x].load(ix, u, looking && slot >= 0 && slot < count, word[x]);
      }
#pragma unroll
      for (int x = 0; x < 2; ++x) post[x].arrive();
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const bool hit = post[x].hit(Q, ix.kmax);
        const uint32_t hits = (uint32_t)(wave_ballot(hit) >> (lane & ~(G - 1))) & ((1u << G) - 1u);
        const int32_t to = M + (int32_t)__popc(hits & ((1u << sub) - 1u));
        if (hit && to < G) found[(lane & ~(G - 1)) + to] = post[x].packed(word[x], a.L);
        M += (int32_t)__popc(hits);
      }
      const bool goes_on = count >= kBucketSlots && r < ix.buckets.mask;
      leave = leave || (looking && goes_on && r + 1 >= kLongChain);
      looking = looking && goes_on && !leave;
    }
    const bool many = is_short || M > (leave ? G : few_matches(a.L));   // (leave: the chain goes on)
    leave = leave || M > G;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (LDS of this wave alone)
    group_draft<G, LCAP, EDGE>(ix, a, u, on && !leave && sub < M ? found[lane] : 0u, on && !leave, sub, target);
    if (on && leave && sub == 0) left[many][atomicAdd(&n_left[many], 1)] = (uint8_t)which;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // (the next turn's matches go to the same cells)
  }
  __syncthreads();
  const uint32_t xcd = blockIdx.x & 7;                   // (see block_units)
  if (threadIdx.x < 2 && n_left[threadIdx.x] > 0)
    list_at[threadIdx.x] = atomicAdd(list.count(xcd, threadIdx.x != 0), n_left[threadIdx.x]);
  __syncthreads();
  for (int m = 0; m < 2; ++m)
    for (int x = (int)threadIdx.x; x < n_left[m]; x += 256)
      *list.unit(xcd, m != 0, list_at[m] + x) = (int32_t)(first + left[m][x]);
}

}  // namespace csd
