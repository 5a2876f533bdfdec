// csd — the incrementally updated n-gram hash index (the "dynamic draft pool"
// of the Method section made searchable) and the append of a step's tokens.
//
// One table of 64-byte buckets [count, 15 postings] per problem, for grams of
// length kmax (the configured maximum query length; shorter queries, which a
// decode loop only issues while a path is shorter than kmax, are matched by
// scan).  A posting (j, e) — "the kmax tokens before index e of path j" — is
// stored under the hash of those tokens when token e is appended, so a query
// finds its matches (Eq. 3) without scanning histories.  Bucket r of a gram's
// probe sequence is (h + r * step) mod n_buckets with an odd step.  In an index with home blocks (see Buckets)
// the first kNear are the home block's, by the same step (a workgroup that has the block in LDS files nearly
// every posting there, whatever else is appended meanwhile), and then the sequence goes through the whole
// table, so that a frequent gram fills kNear buckets of one block.  An insert goes into the first bucket of the sequence that is
// not full, so a lookup may stop at the first bucket that is not full.  Hash collisions are harmless:
// every posting is verified against the history before it counts.
#pragma once

#include "csd_common.cuh"

namespace csd {

struct GramHash {
  uint32_t h, step;
};
// The hash folds the gram's tokens newest first, so the hashes of all gram
// lengths that end at one position come from one pass over the tokens.
constexpr uint32_t kGramSeed = 0x243F6A88u;
__device__ __forceinline__ uint32_t gram_hash_add(uint32_t acc, int32_t token) {
  acc = (acc + (uint32_t)token) * 0x9E3779B1u;
  return acc ^ (acc >> 15);
}
__device__ __forceinline__ GramHash gram_hash_end(uint32_t acc, int g) {
  uint32_t x = acc ^ ((uint32_t)g * 0x85EBCA6Bu);
  uint32_t h = x * 0xC2B2AE35u;
  h ^= h >> 16;
  uint32_t step = ((x * 0x27D4EB2Fu) >> 7) | 1u;
  return GramHash{h, step};
}
// Bucket r of a gram's sequence (step is odd).  Of the first kNear ones, and where there are no home blocks of all:
constexpr uint32_t kNear = 32;
__device__ __forceinline__ uint32_t gram_near(GramHash gh, uint32_t r, Buckets t) {
  return ((gh.h & ~t.block) | ((gh.h + r * gh.step) & t.block)) & t.mask;
}
// What precedes the way through the whole table: the near buckets, where there are others.
__device__ __forceinline__ uint32_t gram_ahead(Buckets t) { return t.mask > t.block ? kNear : 0u; }
// Behind them: through the whole table by the odd step.  (The near buckets come again then: an insert finds them full, a
// look-up passes them, see gram_again.  Few instructions, as in every row's way: block after block, with the home block's
// last, it was seven, and thousands of rows a launch took 4 % longer.)
__device__ __forceinline__ uint32_t gram_far(GramHash gh, uint32_t r, Buckets t) {
  return (gh.h + (r - gram_ahead(t)) * gh.step) & t.mask;
}
__device__ __forceinline__ uint32_t gram_index(GramHash gh, uint32_t r, Buckets t) {
  return r < kNear ? gram_near(gh, r, t) : gram_far(gh, r, t);
}
// Turns of a sequence, in which every bucket comes, also where more is filed than there are positions (see
// file_positions_own).
__device__ __forceinline__ uint32_t gram_turns(Buckets t) { return t.mask + 1u + gram_ahead(t); }
// Whether the bucket of turn r came before: one of the home block that is among the first kNear of the block's own order.
__device__ __forceinline__ bool gram_again(GramHash gh, uint32_t r, Buckets t) {
  return r >= kNear && t.mask > t.block && ((r - kNear) & t.block) < kNear && ((gram_far(gh, r, t) ^ gh.h) & t.mask) <= t.block;
}
__device__ __forceinline__ int32_t* gram_bucket(int32_t* tbl, GramHash gh, uint32_t r,
                                                Buckets tb) {
  return tbl + (int64_t)gram_index(gh, r, tb) * kBucketWords;
}
// (where r is known to be small: the other half is code on the way of every launch, 0.3 us of small ones)
__device__ __forceinline__ int32_t* gram_bucket_near(int32_t* tbl, GramHash gh, uint32_t r, Buckets tb) {
  return tbl + (int64_t)gram_near(gh, r, tb) * kBucketWords;
}

// Word `sub` of bucket r0 + grp of a gram's sequence, for a look-up by batches of four buckets (r0: the batch's first,
// uniform over the wave).  A bucket that came before is as one without postings that goes on; with SELECT the caller
// passes over it.
// SELECT: near or far without a branch, where registers are short (step_wave_many_kernel, 65536 rows 82.5 us, 92 with the
// branch, whose other side needs a few at once); else the usual one alone on the way (64 x 4096, a step 6.7 us, 6.9
// without).  Where the kernel is compiled for an index without home blocks none of it is left.
template <bool SELECT = false>
__device__ __forceinline__ int32_t gram_word(const int32_t* tbl, GramHash gh, uint32_t r0, int grp, int sub, Buckets tb) {
  uint32_t r = r0 + (uint32_t)grp;
  if (SELECT || (__builtin_constant_p(tb.mask > tb.block) && tb.mask <= tb.block))
    return tbl[(int64_t)gram_index(gh, r, tb) * kBucketWords + sub];
  if (__builtin_expect(r0 + 4u <= kNear, 1)) return tbl[(int64_t)gram_near(gh, r, tb) * kBucketWords + sub];
  consume_here(r);                                      // (else what follows is prepared ahead of the caller's loop)
  consume_here(gh.h);
  consume_here(gh.step);
  int32_t word = sub == 0 ? kBucketSlots : -1;
  if (!gram_again(gh, r, tb)) word = tbl[(int64_t)gram_index(gh, r, tb) * kBucketWords + sub];
  return word;
}

// General insert, by one whole wave: reads the fill counts of the sequence's buckets from r0 on, the first few and then
// 64 per round trip, and claims a slot in the first one that is not full.  Bounded by the table size; the
// tables hold more slots than there are positions.
// (The first few: of the rows whose first bucket is full most find one of the next open; 64 at once fetched as many
// lines, 4096 problems at full history 129 us a step for 123.)
constexpr uint32_t kInsertFirst = 4;
__device__ __forceinline__ void gram_insert_from(int32_t* tbl, Buckets tb, GramHash gh,
                                                 uint32_t r0, int32_t pos, int lane) {
  const uint32_t turns = gram_turns(tb), few = turns < kInsertFirst ? turns : kInsertFirst;
  while (r0 < turns) {                                  // uniform over the wave
    const uint32_t r = r0 + lane, end = r0 < few ? few : turns;
    const uint32_t at = gram_index(gh, r, tb);
    bool open = r < end && tbl[(int64_t)at * kBucketWords] < kBucketSlots;
    u64 m = wave_ballot(open);
    while (m) {
      int first = (int)__ffsll((long long)m) - 1;
      int32_t* b = tbl + (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)at, first) * kBucketWords;
      int32_t c = 0;
      if (lane == 0) c = atomicAdd(b, 1);
      c = __builtin_amdgcn_readfirstlane(c);
      if (c < kBucketSlots) {
        if (lane == 0) b[1 + c] = pos;
        return;
      }
      m &= m - 1;                                       // filled up meanwhile: next open bucket
    }
    r0 = r0 < few ? few : r0 + kWave;
  }
}

// Split-phase insert of ONE new position by one wave, so that its two memory
// round trips overlap the lookup's: lanes 0..3 look at the first four buckets of
// the gram's sequence (sixteen were no faster and fetched twelve more lines per row).
// (With thousands of rows per launch the step is bound by what all rows together issue and
// fetch, not by one row's latency: there only the first bucket is looked at up front, LANES = 1.)
constexpr int kInsertLanes = 4;     // buckets of the chain whose fill counts are read up front
struct InsertTicket {
  GramHash gh;
  int32_t fill;                 // fill count of bucket `lane` of the sequence (lanes < LANES)
  int32_t lanes;                // LANES: buckets looked at up front
  int32_t first;                // first open bucket among those looked at, or -1
  int32_t claimed;              // lane 0: slot the atomic returned, or kBucketSlots
  bool live;                    // the position has kmax tokens before it
};

// Phase 1: hash of the gram that ends just before the new position (tail[a] =
// a-th token before it) and the fill-count loads (not waited for here).
template <int QC, int LANES = kInsertLanes>
__device__ __forceinline__ InsertTicket insert_begin(int32_t* gram, Buckets tb, int32_t kmax,
                                                     const int32_t (&tail)[kTailCap],
                                                     int32_t n_before, int lane) {
  static_assert(LANES >= 1 && (LANES & (LANES - 1)) == 0, "a power of two of buckets");
  InsertTicket t;
  t.lanes = LANES;
  uint32_t acc = kGramSeed;
#pragma unroll
  for (int a = 1; a <= QC; ++a)
    if (a <= kmax) acc = gram_hash_add(acc, tail[a - 1]);
  t.gh = gram_hash_end(acc, kmax);
  t.live = kmax <= n_before;
  t.first = -1;
  t.claimed = kBucketSlots;
  uint32_t r = (uint32_t)(lane & (LANES - 1));          // every lane loads: no branch, no early wait
  t.fill = gram_bucket_near(gram, t.gh, r <= tb.mask ? r : 0u, tb)[0];
  return t;
}

// Phase 2: lane 0 claims a slot in the first open bucket.
__device__ __forceinline__ void insert_claim(InsertTicket& t, int32_t* gram, Buckets tb,
                                             int lane) {
  consume_here(t.fill);
  bool open = t.live && lane < t.lanes && (uint32_t)lane <= tb.mask && t.fill < kBucketSlots;
  u64 m = wave_ballot(open);
  t.first = m ? (int32_t)__ffsll((long long)m) - 1 : -1;
  if (t.live && lane == 0 && t.first >= 0)
    t.claimed = atomicAdd(gram_bucket_near(gram, t.gh, (uint32_t)t.first, tb), 1);
}

// Phase 3: store the posting; if the buckets looked at were full (or the last
// slot was lost in a race) take the general insert.
__device__ __forceinline__ void insert_finish(const InsertTicket& t, int32_t* gram, Buckets tb,
                                              int32_t pos, int lane) {
  if (!t.live) return;
  int32_t claimed = __builtin_amdgcn_readfirstlane(t.claimed);
  if (claimed < kBucketSlots) {
    if (lane == 0) gram_bucket_near(gram, t.gh, (uint32_t)t.first, tb)[1 + claimed] = pos;
    return;
  }
  gram_insert_from(gram, tb, t.gh, t.first < 0 ? (uint32_t)t.lanes : (uint32_t)t.first, pos,
                   lane);
}

// ---------------------------------------------------------------- one-edit matching (Eq. 4) through the index
//
// Variant v of a gram G[0 .. kmax) (newest token first): v = 0 is the gram
// itself, v >= 1 the gram without G[v-1].  Two strings within one edit of each
// other share a variant (delete the substituted token from both; delete the
// extra token from the longer one), so a position whose kmax-gram is filed
// under all its kmax + 1 variants is found by looking up the query's variants.
// The converse does not hold, and a position can be found several times:
// candidates are verified and de-duplicated by the matcher.
// A posting of the variant index carries the number of the variant it was
// filed under above the packed position (which needs at most 25 bits): chains
// of different variants can share a bucket, and the matcher must tell them apart.
constexpr int kVariantShift = 26;
__device__ __forceinline__ int32_t variant_posting(int32_t pos, int32_t v) {
  return pos | (v << kVariantShift);
}

template <int SIZE>
__device__ __forceinline__ GramHash variant_hash(const int32_t (&G)[SIZE], int32_t kmax, int32_t v) {
  constexpr int kMost = SIZE < CSD_MAX_QUERY_LEN ? SIZE : CSD_MAX_QUERY_LEN;
  uint32_t acc = kGramSeed;
#pragma unroll
  for (int a = 0; a < kMost; ++a)
    if (a < kmax && a != v - 1) acc = gram_hash_add(acc, G[a]);
  return gram_hash_end(acc, v == 0 ? kmax : kmax - 1);
}
// Variant v >= 2 is the same string as variant v - 1 when the two dropped tokens are equal.
template <int SIZE>
__device__ __forceinline__ bool variant_is_new(const int32_t (&G)[SIZE], int32_t v) {
  return v < 2 || pick(G, v - 1) != pick(G, v - 2);
}

// Split-phase insert of ONE new position under its variants: the four groups
// of 16 lanes take variants 0..3 (fill counts of the first 16 buckets of each
// chain in one round trip, one slot claim per group); further variants
// (kmax >= 4) and groups whose quick claim failed use the general insert.
struct VariantTicket {
  GramHash gh;                  // of this lane's group's variant
  int32_t fill;                 // fill count of bucket (lane & 15) of that chain
  int32_t first;                // first open bucket among those looked at, or -1
  int32_t claimed;              // group leader: slot the atomic returned, or kBucketSlots
  bool live;                    // this group has a variant to file
  bool any;                     // the position has kmax tokens before it
};

__device__ __forceinline__ VariantTicket variants_begin(int32_t* gram, Buckets tb, int32_t kmax,
                                                        const int32_t (&tail)[kTailCap],
                                                        int32_t n_before, int lane) {
  VariantTicket t;
  const int32_t v = lane >> 4;
  t.gh = variant_hash(tail, kmax, v);
  t.any = kmax <= n_before;
  t.live = t.any && v <= kmax && variant_is_new(tail, v);
  t.first = -1;
  t.claimed = kBucketSlots;
  uint32_t r = (uint32_t)(lane & 15);                   // every lane loads: no branch, no early wait
  t.fill = gram_bucket_near(gram, t.gh, r <= tb.mask ? r : 0u, tb)[0];
  return t;
}

__device__ __forceinline__ void variants_claim(VariantTicket& t, int32_t* gram, Buckets tb,
                                               int lane) {
  consume_here(t.fill);
  bool open = t.live && (uint32_t)(lane & 15) <= tb.mask && t.fill < kBucketSlots;
  uint32_t mine = (uint32_t)(wave_ballot(open) >> (lane & 48)) & 0xFFFFu;   // this group's 16 lanes
  t.first = mine ? (int32_t)__ffs(mine) - 1 : -1;
  if (t.live && (lane & 15) == 0 && t.first >= 0)
    t.claimed = atomicAdd(gram_bucket_near(gram, t.gh, (uint32_t)t.first, tb), 1);
}

// Variants beyond the four the groups take (kmax >= 4): the general insert.
__device__ __forceinline__ void variants_beyond_four(const VariantTicket& t, int32_t* gram,
                                                     Buckets tb, int32_t kmax,
                                                     const int32_t (&tail)[kTailCap], int32_t pos,
                                                     int lane) {
  if (!t.any) return;
  for (int32_t v = 4; v <= kmax; ++v)
    if (variant_is_new(tail, v))
      gram_insert_from(gram, tb, variant_hash(tail, kmax, v), 0u, variant_posting(pos, v), lane);
}

__device__ __forceinline__ void variants_finish(const VariantTicket& t, int32_t* gram, Buckets tb,
                                                int32_t pos, int lane) {
  if (!t.any) return;
  bool stored = t.live && (lane & 15) == 0 && t.claimed < kBucketSlots;
  if (stored) gram_bucket_near(gram, t.gh, (uint32_t)t.first, tb)[1 + t.claimed] = variant_posting(pos, lane >> 4);
  int32_t retry = (t.live && !stored) ? 1 : 0;          // meaningful on the group leaders
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (__shfl(retry, 16 * g) == 0) continue;           // uniform over the wave
    GramHash gh{(uint32_t)__shfl((int)t.gh.h, 16 * g), (uint32_t)__shfl((int)t.gh.step, 16 * g)};
    int32_t first = __shfl(t.first, 16 * g);
    gram_insert_from(gram, tb, gh, first < 0 ? 16u : (uint32_t)first, variant_posting(pos, g), lane);
  }
}

// Files the position of each lane of a wave (`mine`: the lane has one; G: the tokens before it,
// newest first) in the index: under its gram, or (FUZZY) under every variant of it.  The slot
// claims of all lanes and variants are atomics on the first buckets of their chains, in flight
// together, without a look at the fill counts before: at most 8 of a bucket's 15 slots are taken
// on average when a problem's histories are full, so few claims miss.  Those go on as claims in
// the next kFileNear buckets, a lane at a time for itself, and what is left then (the long chain of
// a frequent gram) is the whole wave's.  meanwhile(): called while the first claims are in flight.
// LOOK: the fill counts are looked at before all the same (see launch_append).
constexpr uint32_t kFileNear = 4;
template <bool FUZZY, int QC, bool LOOK = false, class MEANWHILE>
__device__ __forceinline__ void file_positions(int32_t* gram, Buckets tb, int32_t kmax,
                                               const int32_t (&G)[QC], bool mine, int32_t pos, int lane,
                                               MEANWHILE&& meanwhile) {
  constexpr int kVariants = FUZZY ? QC + 1 : 1;
  uint32_t todo = 0;                                     // variants of this lane that have no slot yet
  int32_t claimed[kVariants];
  uint32_t at[kVariants];                                // first bucket of the variant's chain
#pragma unroll
  for (int v = 0; v < kVariants; ++v) {
    bool live = mine && v <= kmax;
    if (v >= 2) live = live && G[v - 1] != G[v - 2];     // (else the same string as variant v - 1)
    at[v] = variant_hash(G, kmax, v).h & tb.mask;
    claimed[v] = kBucketSlots;
    todo |= live ? 1u << v : 0u;
  }
  uint32_t claims = todo;
  if (LOOK) {
#pragma unroll
    for (int v = 0; v < kVariants; ++v)
      claims &= gram[(int64_t)at[v] * kBucketWords] < kBucketSlots ? ~0u : ~(1u << v);
    consume_here(claims);
  }
#pragma unroll
  for (int v = 0; v < kVariants; ++v)
    if (claims >> v & 1u) claimed[v] = atomicAdd(gram + (int64_t)at[v] * kBucketWords, 1);
  meanwhile();
#pragma unroll
  for (int v = 0; v < kVariants; ++v)
    if (claimed[v] < kBucketSlots) {                     // (never without a claim)
      gram[(int64_t)at[v] * kBucketWords + 1 + claimed[v]] = FUZZY ? variant_posting(pos, v) : pos;
      todo &= ~(1u << v);
    }
  while (__builtin_expect(wave_ballot(todo != 0) != 0, 0)) {   // uniform over the wave (unlikely: the code behind it stays near)
    const int32_t v = todo != 0 ? (int32_t)__ffs(todo) - 1 : 0;
    const GramHash gh = variant_hash(G, kmax, v);
    const int32_t posting = FUZZY ? variant_posting(pos, v) : pos;
    bool open = todo != 0;
    // (all their fill counts at once: one after the other each was a round trip)
    int32_t fill[kFileNear];
    if (open) {
#pragma unroll
      for (uint32_t x = 0; x < kFileNear; ++x) fill[x] = gram[(int64_t)gram_near(gh, x + 1u, tb) * kBucketWords];
    }
#pragma unroll
    for (uint32_t x = 0; x < kFileNear; ++x) {
      if (!open || fill[x] >= kBucketSlots || x + 1u > tb.mask) continue;
      int32_t* b = gram + (int64_t)gram_near(gh, x + 1u, tb) * kBucketWords;
      const int32_t c = atomicAdd(b, 1);
      if (c < kBucketSlots) {
        b[1 + c] = posting;
        open = false;
      }
    }
    u64 left = wave_ballot(open);
    while (left) {                                       // those were full, too
      const int t = (int)__ffsll((long long)left) - 1;
      left &= left - 1;
      const GramHash g{(uint32_t)__builtin_amdgcn_readlane((int)gh.h, t),
                       (uint32_t)__builtin_amdgcn_readlane((int)gh.step, t)};
      gram_insert_from(gram, tb, g, kFileNear + 1u, __builtin_amdgcn_readlane(posting, t), lane);
    }
    todo &= todo - 1u;                                   // 0 stays 0
  }
}

// The same where one workgroup files all new positions of a problem: `fill` holds the fill counts
// of the problem's buckets in LDS, slots are claimed there, and the postings go to `slots` (bucket
// b's from word 16 b + 1 on), in memory or in LDS too.  A lane has W consecutive positions: `tok`
// are the QC tokens before the first of them, oldest first, and the W at the positions, `filed` has
// a bit per position, `pos` is the first one's packed (path, index).
template <bool FUZZY, int QC, int W>
__device__ __forceinline__ void file_positions_own(int32_t* slots, int32_t* fill, Buckets tb, int32_t kmax,
                                                   const int32_t (&tok)[QC + W], uint32_t filed, int32_t pos) {
  // positions that claim together: all of a lane's (one gram each), or one (its variants)
  constexpr int kTogether = FUZZY ? 1 : W, kVariants = FUZZY ? QC + 1 : 1, kClaims = kTogether * kVariants;
#pragma unroll
  for (int x0 = 0; x0 < W; x0 += kTogether) {
    GramHash gh[kClaims];
    int32_t posting[kClaims], claimed[kClaims];
    uint32_t todo = 0;
#pragma unroll
    for (int y = 0; y < kClaims; ++y) {
      const int x = x0 + (FUZZY ? 0 : y), v = FUZZY ? y : 0;
      int32_t G[QC];
#pragma unroll
      for (int a = 0; a < QC; ++a) G[a] = tok[QC + x - 1 - a];
      bool live = (filed >> x & 1u) != 0 && v <= kmax;
      if (v >= 2) live = live && G[v - 1] != G[v - 2];   // (else the same string as variant v - 1)
      gh[y] = variant_hash(G, kmax, v);
      posting[y] = FUZZY ? variant_posting(pos + x, v) : pos + x;
      todo |= live ? 1u << y : 0u;
    }
#pragma unroll
    for (int y = 0; y < kClaims; ++y) {
      claimed[y] = kBucketSlots;
      if (todo >> y & 1u) claimed[y] = atomicAdd(&fill[gh[y].h & tb.mask], 1);
    }
#pragma unroll
    for (int y = 0; y < kClaims; ++y)
      if (claimed[y] < kBucketSlots) {                   // (never without a claim)
        slots[(gh[y].h & tb.mask) * kBucketWords + 1 + claimed[y]] = posting[y];
        todo &= ~(1u << y);
      }
    // first bucket full: on along the chain, once through all buckets at most (the table holds more
    // slots than positions, but positions may have been filed twice: a launch that leaves the paths'
    // new ends in the other buffer, captured and replayed; their postings are dropped when it is full)
    if (wave_ballot(todo != 0) == 0) continue;
#pragma unroll
    for (int y = 0; y < kClaims; ++y) {
      bool looking = (todo >> y & 1u) != 0;
      const uint32_t turns = gram_turns(tb), home = gh[y].h & tb.mask & ~tb.block;
      uint32_t turn = gh[y].h + gh[y].step;
      for (uint32_t r = 1; r < turns && wave_ballot(looking) != 0; ++r, turn += gh[y].step) {   // uniform over the wave
        uint32_t b = home | (turn & tb.block);
        if (__builtin_expect(tb.mask > tb.block && r >= kNear, 0)) b = gram_far(gh[y], r, tb);
        if (looking) {
          int32_t c = fill[b];                           // (a full bucket is passed without an atomic)
          if (c < kBucketSlots) c = atomicAdd(&fill[b], 1);
          if (c < kBucketSlots) {
            slots[b * kBucketWords + 1 + c] = posting[y];
            looking = false;
          }
        }
      }
    }
  }
}

// What the step appends to a path: its tokens t .. t + 63 (one per lane) with the tokens before
// each, the path's length and the number of tokens it takes.  Everything lies at an address that
// the kernel's arguments give (a new position's gram runs through the step's own tokens and the
// old tail, which the meta row holds), so all loads are in flight together.
// QC: compile-time bound (4 or 8) of the index's gram length; 0: no index.
template <int QC>
struct NewTokens {
  int32_t t, token, len, want, offered;
  float prob;
  int32_t G[QC > 0 ? QC : 1];
  __device__ __forceinline__ void load(const IndexView& ix, const StepIn& in, int64_t row, int32_t t_lane) {
    load(ix, row, in.tok + row * in.n, in.prob ? in.prob + row * in.n : nullptr, 1, in.n,
         in.counts ? in.counts + row : nullptr, t_lane);
  }
  // st, sp: the row's first new token and its probability (or null); `stride`: from one to the next
  __device__ __forceinline__ void load(const IndexView& ix, int64_t row, const int32_t* st, const float* sp,
                                       int64_t stride, int32_t n, const int32_t* count_of_row, int32_t t_lane) {
    const int32_t* meta = ix.meta_old + row * ix.meta_stride;
    t = t_lane;
    const int32_t tt = t < n ? t : 0;
    token = st[tt * stride];
    prob = sp ? sp[tt * stride] : 1.0f;
#pragma unroll
    for (int a = 0; a < QC; ++a) {
      const int32_t back = a < ix.kmax ? a : 0;            // (words beyond the gram are not used)
      G[a] = *(tt > back ? st + (tt - 1 - back) * stride : meta + 1 + (back - tt));
    }
    want = count_of_row ? *count_of_row : n;
    offered = n;
    len = meta[0];
  }
  __device__ __forceinline__ int32_t most() const { return want < 0 ? 0 : (want > offered ? offered : want); }
  __device__ __forceinline__ int32_t count(const IndexView& ix) const {
    const int32_t room = ix.max_len - len;
    return most() < room ? most() : room;
  }
  __device__ __forceinline__ bool mine(int32_t cnt) const { return t < cnt; }
  __device__ __forceinline__ bool filed(const IndexView& ix, int32_t cnt) const {
    return t < cnt && len + t >= ix.kmax;
  }
  __device__ __forceinline__ int32_t pos(const IndexView& ix, int32_t i) const { return (i << ix.eshift) | (len + t); }
  // token and quantised probability to the history; returns the status bits to raise
  __device__ __forceinline__ uint32_t store(const IndexView& ix, bool probs, int64_t row, int32_t cnt) const {
    if (!mine(cnt)) return 0u;
    ix.tok[row * ix.max_len + len + t] = token;
    ix.pq[row * ix.max_len + len + t] = probs ? quantize_prob(prob) : 65536u;
    return (token < 0 || token >= ix.vocab) ? CSD_STATUS_TOKEN_RANGE : 0u;
  }
};

// The path's new meta row (word 0 = length, word 1 + a = a-th token from the new end) after cnt new
// tokens, a word per lane of one wave, into the rows `to` that nobody reads meanwhile.
__device__ __forceinline__ void store_end(const IndexView& ix, const StepIn& in, int64_t row, int32_t len,
                                          int32_t cnt, int32_t* to, int lane) {
  if (lane > ix.tail_len) return;
  const int32_t* st = in.tok + row * in.n;
  const int32_t* meta = ix.meta_old + row * ix.meta_stride;
  const int32_t a = lane - 1;
  int32_t w = len + cnt;
  if (lane > 0) w = a < cnt ? st[cnt - 1 - a] : (a < len + cnt ? meta[1 + a - cnt] : 0);
  to[row * ix.meta_stride + lane] = w;
}
// The same in two halves, for an end that is replaced in place: no branch between them, so a lane's
// word is stored behind all lanes' loads.
__device__ __forceinline__ int32_t end_word(const IndexView& ix, const StepIn& in, int64_t row, int32_t len,
                                            int32_t cnt, int lane) {
  const int32_t a = lane - 1;
  const bool tail = a >= 0 && a < ix.tail_len, fresh = tail && a < cnt, kept = tail && !fresh && a < len + cnt;
  const int32_t token = in.tok[row * in.n + (fresh ? cnt - 1 - a : 0)];
  const int32_t before = ix.meta_old[row * ix.meta_stride + (kept ? 1 + a - cnt : 0)];
  return lane == 0 ? len + cnt : (fresh ? token : (kept ? before : 0));
}
__device__ __forceinline__ void store_end_word(const IndexView& ix, int64_t row, int32_t word, int lane) {
  if (lane <= ix.tail_len) ix.meta_new[row * ix.meta_stride + lane] = word;
}

// The same with four consecutive tokens per lane (t a multiple of 4), for the kernel whose work is
// bound by the instructions it issues: 16-byte loads and stores (at 4-byte alignment), one address.
template <int QC>
struct NewTokens4 {
  int32_t t, len, want, offered;
  int32_t tok[QC + 4];          // tokens t - QC .. t + 3
  float prob[4];
  struct __attribute__((packed, aligned(4))) Word4 { int32_t x[4]; };
  __device__ __forceinline__ void load(const IndexView& ix, const StepIn& in, int64_t row, int32_t t_first,
                                       int lane) {
    const int32_t n = in.n;
    const int32_t* st = in.tok + row * n;
    const int32_t* meta = ix.meta_old + row * ix.meta_stride;
    t = t_first + 4 * lane;
    if (t + 4 <= n) {
      const Word4 w = *reinterpret_cast<const Word4*>(st + t);
#pragma unroll
      for (int x = 0; x < 4; ++x) tok[QC + x] = w.x[x];
      if (in.prob) {
        const Word4 q = *reinterpret_cast<const Word4*>(in.prob + row * n + t);
#pragma unroll
        for (int x = 0; x < 4; ++x) prob[x] = __int_as_float(q.x[x]);
      }
    } else {                                             // the row's end: nothing behind it is read
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        tok[QC + x] = st[t + x < n ? t + x : n - 1];
        if (in.prob) prob[x] = in.prob[row * n + (t + x < n ? t + x : n - 1)];
      }
    }
    if (t >= QC && t <= n) {
#pragma unroll
      for (int b = 0; b < QC; b += 4) {
        const Word4 w = *reinterpret_cast<const Word4*>(st + t - QC + b);
#pragma unroll
        for (int x = 0; x < 4; ++x) tok[b + x] = w.x[x];
      }
    } else {                                             // the row's start: before it lies the old tail
#pragma unroll
      for (int x = 0; x < QC; ++x) {
        const int32_t at = t - QC + x, back = -1 - at;
        tok[x] = at >= 0 ? st[at < n ? at : n - 1] : meta[1 + (back < ix.kmax ? back : 0)];
      }
    }
    want = in.counts ? in.counts[row] : n;
    offered = n;
    len = meta[0];
  }
  __device__ __forceinline__ int32_t most() const { return want < 0 ? 0 : (want > offered ? offered : want); }
  __device__ __forceinline__ int32_t count(const IndexView& ix) const {
    const int32_t room = ix.max_len - len;
    return most() < room ? most() : room;
  }
  __device__ __forceinline__ uint32_t filed(const IndexView& ix, int32_t cnt) const {   // bit x: position t + x
    const int32_t last = cnt - t < 4 ? cnt - t : 4, first = ix.kmax - len - t;
    const uint32_t below = last > 0 ? (1u << last) - 1u : 0u;
    return first <= 0 ? below : (first < 4 ? below & ~((1u << first) - 1u) : 0u);
  }
  __device__ __forceinline__ int32_t pos(const IndexView& ix, int32_t i) const { return (i << ix.eshift) | (len + t); }
  __device__ __forceinline__ uint32_t store(const IndexView& ix, const StepIn& in, int64_t row, int32_t cnt) const {
    if (t >= cnt) return 0u;
    int32_t* to = ix.tok + row * ix.max_len + len + t;
    uint32_t* to_pq = ix.pq + row * ix.max_len + len + t;
    Word4 w, q;
    uint32_t flags = 0;
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      w.x[x] = tok[QC + x];
      q.x[x] = in.prob ? (int32_t)quantize_prob(prob[x]) : 65536;
      if (t + x < cnt && (w.x[x] < 0 || w.x[x] >= ix.vocab)) flags = CSD_STATUS_TOKEN_RANGE;
    }
    if (t + 4 <= cnt) {
      *reinterpret_cast<Word4*>(to) = w;
      *reinterpret_cast<Word4*>(to_pq) = q;
    } else {
#pragma unroll
      for (int x = 0; x < 4; ++x)
        if (t + x < cnt) {
          to[x] = w.x[x];
          to_pq[x] = (uint32_t)q.x[x];
        }
    }
    return flags;
  }
};

// Stores a share of what a step appends to path i of problem p: tokens, quantised probabilities
// and postings of the step's tokens t_first + tid, then every t_stride-th.  Called by whole waves,
// tid counting the threads that share the work.  `head`: this share raises the status bit of a full
// path.  at_end(end, tokens taken): called once by every wave, when all that it needs of the path's
// old end has arrived; `end` is the new one (end_word).
template <bool INDEX, bool FUZZY, int QC, bool LOOK = false, class AT_END>
__device__ __forceinline__ void append_positions(const IndexView& ix, const StepIn& in, int32_t p,
                                                 int32_t i, int32_t t_first, int32_t t_stride,
                                                 bool head, int tid, AT_END&& at_end) {
  const int64_t row = (int64_t)p * ix.N + i;
  const int lane = tid & (kWave - 1);
  int32_t* gram = INDEX ? ix.gram + (int64_t)p * ((int64_t)ix.buckets.mask + 1) * kBucketWords : nullptr;
  uint32_t flags = 0;
  int32_t t0 = t_first + (tid - lane), cnt;
  do {                                                   // uniform over the wave
    NewTokens<INDEX ? QC : 0> x;
    x.load(ix, in, row, t0 + lane);
    cnt = x.count(ix);
    const bool last = t0 + t_stride >= cnt;
    int32_t end = 0;
    if (last) end = end_word(ix, in, row, x.len, cnt, lane);
    if (head && tid == 0 && t0 == 0 && x.most() > cnt) flags |= CSD_STATUS_CAPACITY;
    flags |= x.store(ix, in.prob != nullptr, row, cnt);
    auto sign_off = [&]() {
      if (!last) return;
      consume_here(end);
      at_end(end, cnt);
    };
    if constexpr (INDEX) {
#pragma unroll
      for (int a = 0; a < QC; ++a) consume_here(x.G[a]);
      file_positions<FUZZY, QC, LOOK>(gram, ix.buckets, ix.kmax, x.G, x.filed(ix, cnt), x.pos(ix, i), lane, sign_off);
    } else {
      sign_off();
    }
    t0 += t_stride;
  } while (t0 < cnt);
  if (flags) atomicOr(ix.status, flags);
}

// ... the whole of it, by the waves of one workgroup.  The new end goes to meta_new: a row that
// nobody reads in this launch, or, for one wave, over the old one.
template <bool INDEX, bool FUZZY, int QC>
__device__ __forceinline__ void append_path(const IndexView& ix, const StepIn& in, int32_t p, int32_t i,
                                            int32_t threads, int tid) {
  append_positions<INDEX, FUZZY, QC>(ix, in, p, i, 0, threads, true, tid, [&](int32_t end, int32_t) {
    if (tid < kWave) store_end_word(ix, (int64_t)p * ix.N + i, end, tid);   // uniform over the wave
  });
}

}  // namespace csd
