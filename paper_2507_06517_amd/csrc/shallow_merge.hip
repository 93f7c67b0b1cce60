// Greedy highest-degree codebook construction (Alg. 1, Eq. 11-13) on the neighbour lists.
#include "shallow.h"

namespace spindle {
namespace {

// ---------------------------------------------------------------- greedy merge
// Exact parallel form of the loop of Alg. 1.  With key(v) = (degree among remaining
// tokens, lower index first), the sequential loop always takes the remaining token of
// largest key.  A token whose key is the largest within two hops cannot lose a
// neighbour before it is taken itself (whoever removed one would be within two hops and
// would have needed a larger key), and tokens taken meanwhile are three or more hops away,
// so they do not touch its neighbourhood.  Each round therefore takes every two-hop
// maximum at once; sorting all picks by their key at pick time (which strictly decreases
// along the sequential loop) restores the codebook order.
//
// A round has three phases:
//   one-hop   m1[v] = largest key in v's closed neighbourhood; v is a candidate if it is its own
//   two-hop   a candidate whose neighbours' m1 never exceed its key is picked: its remaining
//             neighbours get its position as their slot and leave the next round's live bits
//   update    keys of tokens that left become 0, those that stay count the neighbours still
//             there (Eq. 13): one population count per word of their list
// The first kGridRounds rounds, where most tokens are still there, run as grid-wide kernels (one launch
// per phase): a wave takes 32 consecutive positions, eight lanes per row, and what it finds goes out
// as the 32 bits of its positions (live, candidate, picked), so that no list has to be built and no
// counter is shared: same-address atomics cost about 40 ns each here.  Neighbours stand close to each
// other in the sorted order, so the 64-byte reads of 16 keys at a time mostly hit the caches.
// The remaining rounds run in one 1024-thread workgroup per problem with keys and live bits in LDS,
// separated by workgroup barriers only.  Bound by the latency of a row's words and what they point at:
// two grid rounds of 16 problems of 32768 tokens take 0.09 ms (0.165 ms with single neighbours, lists of
// remaining tokens and counters), of 64 such problems with half of the tokens isolated 0.24 (0.55) ms.
constexpr int kMergeThreads = 1024;
constexpr int kSegW = 8;                 // lanes that share one row
constexpr int kGridRounds = 2;           // live[] holds the bits of one round more
// Up to here the workgroup per problem runs all rounds: six launches less, and no more than eight rows per lane segment
// and phase.  f16, us per call with and without the grid rounds, clusters and half isolated: one head of 512
// tokens 68, 88 and 55, 73; 8 of 1024 95, 125 and 81, 115; 8 of 1536 114, 163 and 111, 170; 8 of 2048 129, 178 and 132, 196.
constexpr int kTailOnly = 1024;
constexpr int kPhaseThreads = 256;
constexpr int kKeysInLds = 36 * 1024;   // tokens whose keys fit in LDS next to the live bits

struct Row {
  const uint32_t *w;
  int n;            // words
  bool dense;       // the bits of all half tiles in order instead of words
};

__device__ __forceinline__ Row row_at(const ShallowParams &p, size_t base, const uint32_t *lists, int v) {
  const uint2 info = p.rows[base + v];
  return Row{lists + info.x, (int)(info.y & ~kDenseRow), (info.y & kDenseRow) != 0};
}

// Word i of a row: half tile << 16 | bits.
__device__ __forceinline__ uint32_t word_at(const Row &r, int i) {
  return r.dense ? ((uint32_t)i << 16) | reinterpret_cast<const uint16_t *>(r.w)[i] : r.w[i];
}

// f(word) for words i, i + 8, ... of a row that have bits, four loads in flight.
template <typename F>
__device__ __forceinline__ void for_words(const Row &r, int i, F f) {
  for (; i < r.n; i += 4 * kSegW) {
    uint32_t x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = i + j * kSegW;
      x[j] = k >= r.n ? 0u : r.dense ? reinterpret_cast<const uint16_t *>(r.w)[k] : r.w[k];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (x[j] & 0xFFFFu) f(r.dense ? (uint32_t)(i + j * kSegW) << 16 | x[j] : x[j]);
  }
}

// Largest of the 16 values of the half tile that the bits select (and m).
__device__ __forceinline__ uint32_t masked_max(const uint32_t *a, uint32_t word, uint32_t m) {
  const u4 *q = reinterpret_cast<const u4 *>(a + (word >> 16) * 16);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const u4 x = q[i];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t y = x[j] & (uint32_t)__builtin_amdgcn_sbfe((int)word, 4 * i + j, 1);
      m = y > m ? y : m;
    }
  }
  return m;
}

// The bits of `word` that are set in the bit array `live` (one bit per position).
__device__ __forceinline__ uint32_t still(const uint32_t *live, uint32_t word) {
  return word & 0xFFFFu & (live[word >> 17] >> ((word >> 12) & 16));
}

// Largest of the values in LDS that the bits `rem` of the word select (and m).  One at a time where no lane of the wave
// has more than a few: a late round of a dense graph, or neighbours all over the sequence (16 problems of 8192
// tokens with a tenth of all pairs adjacent: the remaining rounds 13.7 -> 10.7 ms together with four loads in flight per row).
__device__ __forceinline__ uint32_t selected_max(const uint32_t *a, uint32_t word, uint32_t rem, uint32_t m) {
  if (__any(__popc(rem) > 4)) return masked_max(a, (word & 0xFFFF0000u) | rem, m);
  const uint32_t *q = a + (word >> 16) * 16;
  for (; rem; rem &= rem - 1) {
    const uint32_t y = q[__builtin_ctz(rem)];
    m = y > m ? y : m;
  }
  return m;
}

// Lane exchanges inside an 8-lane segment by DPP (no LDS round trip): the two quad
// permutations, then the mirror of the eight lanes, which pairs each lane with one of the
// other quad.
static_assert(kSegW == 8, "the segment reductions are written for eight lanes");
__device__ __forceinline__ uint32_t seg_xchg(uint32_t v, int step) {
  return step == 0 ? (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false)     // quad_perm [1,0,3,2]
         : step == 1 ? (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false)   // quad_perm [2,3,0,1]
                     : (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false); // row_half_mirror
}
__device__ __forceinline__ uint32_t seg_max(uint32_t v) {   // over a segment, result in every lane
#pragma unroll
  for (int step = 0; step < 3; ++step) {
    const uint32_t x = seg_xchg(v, step);
    v = x > v ? x : v;
  }
  return v;
}
__device__ __forceinline__ int seg_sum(int v) {             // over a segment, result in every lane
#pragma unroll
  for (int step = 0; step < 3; ++step) v += (int)seg_xchg((uint32_t)v, step);
  return v;
}

// Largest of the values in memory that the words of a row select (and m), for a segment whose lanes have a word each: a
// quad takes its four words one after the other, each lane 16 of the 64 bytes, so that a load of the wave touches 16 lines
// and not 64 (one-hop maxima of 128 problems of 8192 tokens in clusters of 128, both rounds: 90 us with a word per lane, 60 now;
// the largest key of every half tile and whose it is, asked first, takes 50 there and half as long again in small calls).
// Steps without a bit in any lane's word are left out by the callers: rows that hold the bits of all half tiles are mostly empty where
// a graph has several clusters (4 problems of 8192 tokens in two, both rounds, 208 us with such steps, 167 now; in one, 295, 255).
__device__ __forceinline__ uint32_t quad_max(const uint32_t *a, uint32_t word, uint32_t m) {
  const int piece = lane_id() & 3;
  uint32_t w[4];
  u4 q[4];
  w[0] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0x00, 0xF, 0xF, true);   // quad_perm [i,i,i,i]
  w[1] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0x55, 0xF, 0xF, true);
  w[2] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0xAA, 0xF, 0xF, true);
  w[3] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)word, 0xFF, 0xF, 0xF, true);
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = *reinterpret_cast<const u4 *>(reinterpret_cast<const char *>(a) + ((w[i] >> 16) * 64u + piece * 16u));
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int bits = (int)(w[i] >> (4 * piece));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t y = q[i][j] & (uint32_t)__builtin_amdgcn_sbfe(bits, j, 1);
      m = y > m ? y : m;
    }
  }
  return m;
}

// Bit s of the result: `on` of segment s (0..7), given in the segment's first lane.
__device__ __forceinline__ uint32_t seg_bits(bool on) {
  const unsigned long long m = __ballot(on && (lane_id() & (kSegW - 1)) == 0);
  // bits 0, 8, 16, ... gathered by a multiplication (each half of 32 bits has four of them)
  const uint32_t lo = (uint32_t)m & 0x01010101u, hi = (uint32_t)(m >> 32) & 0x01010101u;
  return ((lo * 0x10204080u) >> 28 & 0xFu) | (((hi * 0x10204080u) >> 28 & 0xFu) << 4);
}

// ---------------------------------------------------------------- grid rounds
// Wave index within a problem = word of the bit arrays = 32 positions; pass k of 4 takes positions
// 8 k .. 8 k + 7 of it, one per segment.
// (Eight waves per SIMD: 128 problems of 8192 tokens in clusters, both rounds 90 us; with the registers for six, the next word
// on its way and dense rows by a half tile per lane 97, and 16 problems of 32768 similar tokens 4.5 ms, not 3.35.)
__global__ __launch_bounds__(kPhaseThreads, 8) void merge_onehop(ShallowParams p, int round) {
  const int ut = blockIdx.y, W = (int)blockIdx.x * (kPhaseThreads / kWave) + (int)(threadIdx.x >> 6);
  if (W >= p.T) return;
  const int lane = lane_id(), seg = lane / kSegW, sl = lane & (kSegW - 1);
  const uint32_t live = __builtin_amdgcn_readfirstlane(p.live[round][(size_t)ut * p.T + W]);
  uint32_t *cand = reinterpret_cast<uint32_t *>(p.cand + (size_t)ut * p.n);
  if (live == 0) {
    if (lane == 0) cand[W] = 0;
    return;
  }
  const size_t base = (size_t)ut * p.n;
  const uint32_t *key = p.key + (size_t)ut * p.n32, *lists = p.lists + base * p.list_row;
  uint32_t *m1 = p.m1 + (size_t)ut * p.n32;
  Row r[4];
  uint32_t w0[4], own[4];
  bool on[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    on[k] = (live >> (8 * k + seg)) & 1;
    const int v = on[k] ? W * kTile + 8 * k + seg : W * kTile;
    r[k] = row_at(p, base, lists, v);
    own[k] = key[v];
  }
  // (a token without neighbours needs none of its words)
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (!on[k] || own[k] >> 16 == 1) r[k].n = 0;
    w0[k] = sl < r[k].n ? word_at(r[k], sl) : 0;
  }
  uint32_t bits = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    uint32_t m = quad_max(key, w0[k], own[k]);        // a token is its own neighbour
    for (int i = sl + kSegW; __any(i < r[k].n); i += kSegW) {
      const uint32_t w = i < r[k].n ? word_at(r[k], i) : 0;
      if (__any(w & 0xFFFFu)) m = quad_max(key, w, m);
    }
    m = seg_max(m);
    if (on[k] && sl == 0) m1[W * kTile + 8 * k + seg] = m;
    bits |= seg_bits(on[k] && m == own[k]) << (8 * k);
  }
  if (lane == 0) cand[W] = bits;
}

__global__ __launch_bounds__(kPhaseThreads, 8) void merge_twohop(ShallowParams p, int round) {
  const int ut = blockIdx.y, W = (int)blockIdx.x * (kPhaseThreads / kWave) + (int)(threadIdx.x >> 6);
  if (W >= p.T) return;
  const int lane = lane_id(), seg = lane / kSegW, sl = lane & (kSegW - 1);
  const size_t base = (size_t)ut * p.n;
  const uint32_t cand = __builtin_amdgcn_readfirstlane(reinterpret_cast<const uint32_t *>(p.cand + base)[W]);
  uint32_t *picked = p.picked + (size_t)ut * p.T + W;
  if (cand == 0) {
    if (round == 0 && lane == 0) *picked = 0;
    return;
  }
  const uint32_t *key = p.key + (size_t)ut * p.n32, *m1 = p.m1 + (size_t)ut * p.n32;
  const uint32_t *lists = p.lists + base * p.list_row, *live = p.live[round] + (size_t)ut * p.T;
  uint32_t *next[2] = {p.live[1] + (size_t)ut * p.T, p.live[2] + (size_t)ut * p.T};
  int *slot = p.slot + base;
  // tokens without neighbours are picked as they are, a lane each
  const int v = W * kTile + (lane & 31);
  const uint32_t kv = cand >> (lane & 31) & 1 ? key[v] : 0u;
  const bool alone = lane < kTile && kv >> 16 == 1;
  if (alone) {
    p.pick_key[base + v] = kv;
    slot[v] = v;
  }
  uint32_t bits = (uint32_t)__ballot(alone);
  if (bits && lane == 0) {
    if (round == 0) atomicAnd(next[0] + W, ~bits);
    atomicAnd(next[1] + W, ~bits);
  }
  const uint32_t rest = cand & ~bits;
  for (int k = 0; k < 4; ++k) {
    if (((rest >> (8 * k)) & 0xFFu) == 0) continue;   // wave-uniform
    const bool on = (rest >> (8 * k + seg)) & 1;
    const int u = on ? W * kTile + 8 * k + seg : W * kTile;
    Row r = row_at(p, base, lists, u);
    if (!on) r.n = 0;
    const uint32_t ku = key[u];
    uint32_t m = 0;
    auto here = [&](uint32_t w) { return (w & 0xFFFF0000u) | still(live, w); };   // neighbours still there at the start of the round
    for (int i = sl; __any(i < r.n); i += kSegW) {
      const uint32_t w = here(i < r.n ? word_at(r, i) : 0);
      if (__any(w & 0xFFFFu)) m = quad_max(m1, w, m);
    }
    const bool pick = on && seg_max(m) == ku;
    bits |= seg_bits(pick) << (8 * k);
    if (pick) {
      if (sl == 0) p.pick_key[base + u] = ku;
      for (int i = sl; i < r.n; i += kSegW) {
        const uint32_t w = word_at(r, i);
        uint32_t rem = still(live, w);
        if (rem == 0) continue;
        const uint32_t clear = ~(rem << ((w >> 12) & 16));
        if (round == 0) atomicAnd(next[0] + (w >> 17), clear);
        atomicAnd(next[1] + (w >> 17), clear);
        do {
          slot[(w >> 16) * 16 + __builtin_ctz(rem)] = u;
          rem &= rem - 1;
        } while (rem);
      }
    }
  }
  if (lane == 0) *picked = (round == 0 ? 0u : *picked) | bits;
}

__global__ __launch_bounds__(kPhaseThreads) void merge_update(ShallowParams p, int round) {
  const int ut = blockIdx.y, W = (int)blockIdx.x * (kPhaseThreads / kWave) + (int)(threadIdx.x >> 6);
  if (W >= p.T) return;
  const int lane = lane_id(), seg = lane / kSegW, sl = lane & (kSegW - 1);
  const uint32_t *next = p.live[round + 1] + (size_t)ut * p.T;
  const uint32_t was = __builtin_amdgcn_readfirstlane(p.live[round][(size_t)ut * p.T + W]);
  const uint32_t now = __builtin_amdgcn_readfirstlane(next[W]);
  if (was == 0) return;
  const size_t base = (size_t)ut * p.n;
  uint32_t *key = p.key + (size_t)ut * p.n32 + W * kTile;
  const uint32_t *lists = p.lists + base * p.list_row;
  if (lane < kTile && ((was & ~now) >> lane & 1)) key[lane] = 0;
  if (now == 0) return;
  Row r[4];
  uint32_t w0[4], own[4];
  bool on[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    on[k] = (now >> (8 * k + seg)) & 1;
    r[k] = row_at(p, base, lists, on[k] ? W * kTile + 8 * k + seg : W * kTile);
    own[k] = on[k] ? key[8 * k + seg] : 0;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) w0[k] = on[k] && sl < r[k].n ? word_at(r[k], sl) : 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    int c = __popc(still(next, w0[k]));
    if (on[k]) for_words(r[k], sl + kSegW, [&](uint32_t w) { c += __popc(still(next, w)); });
    c = seg_sum(c);
    if (on[k] && sl == 0) key[8 * k + seg] = ((uint32_t)c << 16) | (own[k] & 0xFFFFu);
  }
}

// ---------------------------------------------------------------- remaining rounds
// State of one problem in the workgroup: keys in LDS (or global memory), bits in LDS.
struct Tail {
  const uint32_t *lists;
  uint32_t *key, *live, *next, *picked;
  int *n_cand, *n_dying;
  int seg, sl;
};
constexpr int kTailSegs = kMergeThreads / kSegW;

__device__ __forceinline__ void tail_onehop(const ShallowParams &p, size_t base, const Tail &w, uint32_t *m1,
                                            const int *alive, int nalive) {
  int *cand = p.cand + base;
  for (int i0 = 0; i0 < nalive; i0 += 4 * kTailSegs) {
    Row r[4];
    int vv[4];
    bool on[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = i0 + k * kTailSegs + w.seg;
      on[k] = i < nalive;
      vv[k] = on[k] ? alive[i] : 0;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = row_at(p, base, w.lists, vv[k]);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t own = on[k] ? w.key[vv[k]] : 0;
      uint32_t m = own;
      if (on[k])
        for_words(r[k], w.sl, [&](uint32_t x) {
          const uint32_t rem = still(w.live, x);
          if (rem) m = selected_max(w.key, x, rem, m);
        });
      m = seg_max(m);
      if (on[k] && w.sl == 0) {
        m1[vv[k]] = m;
        if (m == own) cand[atomicAdd(w.n_cand, 1)] = vv[k];
      }
    }
  }
}

__device__ __forceinline__ void tail_twohop(const ShallowParams &p, size_t base, const Tail &w,
                                            const uint32_t *m1, int ncand) {
  const int *cand = p.cand + base;
  int *slot = p.slot + base, *dying = p.dying + base;
  for (int i0 = w.seg; i0 < ncand; i0 += kTailSegs) {
    const int u = cand[i0];
    const Row r = row_at(p, base, w.lists, u);
    const uint32_t ku = w.key[u];
    uint32_t m = 0;
    for_words(r, w.sl, [&](uint32_t x) {
      const uint32_t rem = still(w.live, x);
      if (rem) m = selected_max(m1, x, rem, m);
    });
    if (seg_max(m) != ku) continue;
    if (w.sl == 0) {
      p.pick_key[base + u] = ku;
      atomicOr(&w.picked[u >> 5], 1u << (u & 31));
    }
    for (int i = w.sl; i < r.n; i += kSegW) {
      const uint32_t x = word_at(r, i);
      uint32_t rem = still(w.live, x);
      if (rem == 0) continue;
      atomicAnd(&w.next[x >> 17], ~(rem << ((x >> 12) & 16)));
      int at = atomicAdd(w.n_dying, __popc(rem));
      do {
        const int v = (int)(x >> 16) * 16 + __builtin_ctz(rem);
        rem &= rem - 1;
        slot[v] = u;
        dying[at++] = v;
      } while (rem);
    }
  }
}

// ---------------------------------------------------------------- codebook order
// Codebook order: the picks of a problem sorted by decreasing key at pick time, i.e. by decreasing
// degree and among equal degrees by increasing token.  One workgroup per problem lists the picks in token
// order as degree << 16 | position, then a least-significant-digit radix sort of the degrees: at most two
// stable passes of 8 bits that ping-pong between two arrays left free by the merge; a pass whose digit all
// picks share is left out (degrees below 256: one pass).  In a pass every wave owns a run of the items:
// it counts their digits, and after one sum over waves and digits places them, 64 at a time, lanes with the
// same digit finding each other with eight ballots.
// Bound by latency, one workgroup per problem: as a kernel of its own on arrays in memory 43 us for 2 problems of
// 32768 rows, 88 for one layer of 16 x 32768 beside two others, 12 for 512 tokens.  It is the end of
// shallow_merge, whose LDS is free by then: with the launch before it gone and the picks in LDS a call of 512 to
// 4096 tokens takes 5 us less.
__device__ __forceinline__ unsigned long long same_digit(int d, bool on) {
  unsigned long long peers = __ballot(on);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const unsigned long long m = __ballot((d >> bit) & 1);
    peers &= ((d >> bit) & 1) ? m : ~m;
  }
  return peers;
}

struct RankLds {
  int before[1024];                                  // picked tokens in front of 64 consecutive ones
  int place[kMergeThreads / kWave][256];             // next output position of a digit of a wave's items
  int wsum[kMergeThreads / kWave];
  int alike;
};

// `room` words behind `l` are free: picks that fit there twice are sorted in LDS.
__device__ __forceinline__ void rank_picks(const ShallowParams &p, int ut, const uint32_t *picked, RankLds &l, int room) {
  constexpr int kWaves = kMergeThreads / kWave, kAtOnce = 4;
  int *before = l.before, *wsum = l.wsum;
  auto &place = l.place;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, n = p.n;
  const size_t base = (size_t)ut * n;
  int *cnt = p.counters + (size_t)ut * kCounters;
  before[tid] = 0;
  __syncthreads();
  // thread t takes tokens t, t + 1024, ..., eight loads in flight (loops kept short: with all trips unrolled the
  // instruction fetches of a cold kernel cost more than the loads)
  constexpr int kLoads = 8;
  auto is_picked = [&](int tok, int v) { return tok < n && (picked[v >> 5] >> (v & 31) & 1u); };
#pragma unroll 1
  for (int t0 = tid; t0 - tid < n; t0 += kLoads * kMergeThreads) {
    int v[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) v[i] = t0 + i * kMergeThreads < n ? (int)p.iperm[base + t0 + i * kMergeThreads] : 0;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const unsigned long long mk = __ballot(is_picked(t0 + i * kMergeThreads, v[i]));
      if (lane == 0) before[min(1023, (t0 + i * kMergeThreads) >> 6)] = __popcll(mk);
    }
  }
  __syncthreads();
  int P = 0;
  {
    const int own = before[tid];
    int incl = own;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int x = __shfl_up(incl, o);
      if (lane >= o) incl += x;
    }
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    for (int q = 0; q < kWaves; ++q) {
      if (q < wave) incl += wsum[q];
      P += wsum[q];
    }
    before[tid] = incl - own;
  }
  if (tid == 0) {
    cnt[C_PICKS] = P;
    p.n_codes[ut / p.U][ut % p.U] = P < p.cap ? P : p.cap;
    if (p.n_found[ut / p.U]) p.n_found[ut / p.U][ut % p.U] = P;
  }
  __syncthreads();
  const bool in_lds = 2 * P <= room;
  uint32_t *src = in_lds ? reinterpret_cast<uint32_t *>(&l + 1) : p.m1 + (size_t)ut * p.n32;
  uint32_t *dst = in_lds ? src + P : p.key + (size_t)ut * p.n32;
#pragma unroll 1
  for (int t0 = tid; t0 - tid < n; t0 += kLoads * kMergeThreads) {
    int v[kLoads];
    uint32_t k[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) v[i] = t0 + i * kMergeThreads < n ? (int)p.iperm[base + t0 + i * kMergeThreads] : 0;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) k[i] = is_picked(t0 + i * kMergeThreads, v[i]) ? p.pick_key[base + v[i]] : 0u;
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int tok = t0 + i * kMergeThreads;
      const bool on = k[i] != 0;                     // (a token's key at pick time counts itself)
      const unsigned long long mk = __ballot(on);
      if (on) src[before[tok >> 6] + __popcll(mk & ((1ull << lane) - 1ull))] = (k[i] & 0xFFFF0000u) | (uint32_t)v[i];
    }
  }
  const int run = (((P + kWaves - 1) / kWaves) + 63) & ~63;      // items per wave
  const int s_begin = min(P, wave * run), s_end = min(P, s_begin + run);
  volatile int *mine = place[wave];
#pragma unroll 1
  for (int shift = 16; shift < 32; shift += 8) {
    for (int i = tid; i < kWaves * 256; i += kMergeThreads) (&place[0][0])[i] = 0;
    if (tid == 0) l.alike = 0;
    __syncthreads();
#pragma unroll 1
    for (int s0 = s_begin; s0 < s_end; s0 += 64 * kAtOnce) {
      uint32_t k[kAtOnce];
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        const int s = s0 + 64 * q + lane;
        k[q] = s < s_end ? src[s] : 0u;
      }
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        const bool on = s0 + 64 * q + lane < s_end;
        const int d = 255 - (int)((k[q] >> shift) & 255u);        // larger degrees first
        const unsigned long long peers = same_digit(d, on);
        if (on && lane == __builtin_ctzll(peers)) mine[d] = mine[d] + __popcll(peers);
        __builtin_amdgcn_wave_barrier();
      }
    }
    __syncthreads();
    int total = 0, incl = 0;
    if (tid < 256) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) total += place[w][tid];
      incl = total;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int x = __shfl_up(incl, o);
        if (lane >= o) incl += x;
      }
      if (lane == kWave - 1) wsum[wave] = incl;
      if (total == P) l.alike = 1;
    }
    __syncthreads();
    if (l.alike) {                                  // this digit orders nothing (no picks: likewise)
      __syncthreads();
      continue;
    }
    if (tid < 256) {
      int at = incl - total;
      for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const int c = place[w][tid];
        place[w][tid] = at;
        at += c;
      }
    }
    __syncthreads();
#pragma unroll 1
    for (int s0 = s_begin; s0 < s_end; s0 += 64 * kAtOnce) {
      uint32_t k[kAtOnce];
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        const int s = s0 + 64 * q + lane;
        k[q] = s < s_end ? src[s] : 0u;
      }
#pragma unroll
      for (int q = 0; q < kAtOnce; ++q) {
        const bool on = s0 + 64 * q + lane < s_end;
        const int d = 255 - (int)((k[q] >> shift) & 255u);
        const unsigned long long peers = same_digit(d, on);
        const int at = mine[d];
        __builtin_amdgcn_wave_barrier();
        if (on) {
          dst[at + __popcll(peers & ((1ull << lane) - 1ull))] = k[q];
          if (lane == __builtin_ctzll(peers)) mine[d] = at + __popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
    __syncthreads();
    uint32_t *x = src;
    src = dst;
    dst = x;
  }
#pragma unroll 1
  for (int r0 = 0; r0 < P; r0 += kAtOnce * kMergeThreads) {
    int v[kAtOnce], tok[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) v[q] = r0 + q * kMergeThreads + tid < P ? (int)(src[r0 + q * kMergeThreads + tid] & 0xFFFFu) : 0;
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) tok[q] = (int)p.perm[base + v[q]];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const int r = r0 + q * kMergeThreads + tid;
      if (r < P) {
        p.rank[base + v[q]] = r;
        p.rank_vert[base + r] = tok[q];              // from here on tokens again
      }
    }
  }
}

#define MERGE_TICK(k)                          \
  if (tid == 0) {                              \
    const long long now_ = wall_clock64();     \
    cnt[6 + (k)] += (int)(now_ - tick_);       \
    tick_ = now_;                              \
  }

__global__ __launch_bounds__(kMergeThreads) void shallow_merge(ShallowParams p, int first_round, int lds_words) {
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ int sh_n[3];                     // alive, candidates, dying
  __shared__ int wsum[kMergeThreads / kWave];
  const int ut = blockIdx.x, n = p.n, T = p.T, tid = threadIdx.x;
  const int lane = lane_id(), wave = tid >> 6;
  const size_t base = (size_t)ut * n;
  const bool keys_in_lds = n <= kKeysInLds;
  int *cnt = p.counters + (size_t)ut * kCounters;
  uint32_t *gkey = p.key + (size_t)ut * p.n32, *m1 = p.m1 + (size_t)ut * p.n32;
  const int T4 = (T + 3) & ~3;
  Tail w;
  w.lists = p.lists + base * p.list_row;
  w.picked = lds;
  w.live = lds + T4;
  w.next = w.live + T4;
  w.key = keys_in_lds ? w.next + T4 : gkey;
  w.n_cand = &sh_n[1]; w.n_dying = &sh_n[2];
  w.seg = tid / kSegW; w.sl = tid & (kSegW - 1);
  int *alive = p.alive + base;
  const int *dying = p.dying + base;
  long long tick_ = 0;
  if (tid == 0) tick_ = wall_clock64();

  // tokens left after the grid rounds, as a list
  const uint32_t *glive = p.live[first_round] + (size_t)ut * T;
  if (tid < 3) sh_n[tid] = 0;
  for (int i = tid; i < T; i += kMergeThreads) w.picked[i] = first_round > 0 ? p.picked[(size_t)ut * T + i] : 0u;
  for (int w0 = 0; w0 < T; w0 += kMergeThreads) {
    const int i = w0 + tid;
    uint32_t bits = i < T ? glive[i] : 0;
    if (i < T) w.live[i] = w.next[i] = bits;
    int incl = __popc(bits);
    const int mine = incl;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int x = __shfl_up(incl, o);
      if (lane >= o) incl += x;
    }
    __syncthreads();                                  // wsum of the trip before has been read
    if (lane == kWave - 1) wsum[wave] = incl;
    __syncthreads();
    int at = sh_n[0] + incl - mine;
    for (int q = 0; q < wave; ++q) at += wsum[q];
    for (; bits; bits &= bits - 1) alive[at++] = i * 32 + __builtin_ctz(bits);
    __syncthreads();
    if (tid == kMergeThreads - 1) sh_n[0] = at;
  }
  __syncthreads();
  if (sh_n[0] > 0 && keys_in_lds) {
    const u4 *src = reinterpret_cast<const u4 *>(gkey);
    for (int i = tid; i < p.n32 / 4; i += kMergeThreads) reinterpret_cast<u4 *>(w.key)[i] = src[i];
  }
  __syncthreads();
  MERGE_TICK(0)

  // every round removes at least the token of largest key, so n rounds always suffice;
  // the bound only guards against a workspace overwritten under the running call
  int round = first_round;
  for (; round <= n + kGridRounds; ++round) {
    const int nalive = sh_n[0];
    if (nalive == 0) break;
    tail_onehop(p, base, w, m1, alive, nalive);
    __syncthreads();
    MERGE_TICK(2)
    tail_twohop(p, base, w, m1, sh_n[1]);
    __syncthreads();
    MERGE_TICK(4)
    const int ndying = sh_n[2];
    for (int i = tid; i < ndying; i += kMergeThreads) w.key[dying[i]] = 0;
    __syncthreads();
    if (tid < 3) sh_n[tid] = 0;
    // survivors, compacted in place (each wave appends its survivors with one LDS atomic;
    // the write index never passes the read index of a later chunk because chunks are
    // consumed by all waves in lock step)
    for (int i0 = 0; i0 < nalive; i0 += kMergeThreads) {
      const int i = i0 + tid;
      const int v = i < nalive ? alive[i] : -1;
      const bool live = v >= 0 && w.key[v] != 0;
      __syncthreads();
      const unsigned long long mk = __ballot(live);
      int at = 0;
      if (lane == 0 && mk) at = atomicAdd(&sh_n[0], __popcll(mk));
      at = __shfl(at, 0);
      if (live) alive[at + __popcll(mk & ((1ull << lane) - 1ull))] = v;
      __syncthreads();
    }
    MERGE_TICK(0)
    // degrees of the survivors (Eq. 13): subtract at the neighbours of the tokens that left,
    // or recount at the tokens that stayed, whichever list is shorter
    const int nleft = nalive - ndying;
    if (ndying <= nleft) {
      for (int i0 = w.seg; i0 < ndying; i0 += kTailSegs) {
        const Row r = row_at(p, base, w.lists, dying[i0]);
        for_words(r, w.sl, [&](uint32_t x) {
          for (uint32_t rem = still(w.next, x); rem; rem &= rem - 1)
            atomicSub(&w.key[(x >> 16) * 16 + __builtin_ctz(rem)], 1u << 16);
        });
      }
    } else {
      for (int i0 = w.seg; i0 < nleft; i0 += kTailSegs) {
        const int v = alive[i0];
        const Row r = row_at(p, base, w.lists, v);
        int c = 0;
        for_words(r, w.sl, [&](uint32_t x) { c += __popc(still(w.next, x)); });
        c = seg_sum(c);
        if (w.sl == 0) w.key[v] = ((uint32_t)c << 16) | (w.key[v] & 0xFFFFu);
      }
    }
    for (int i = tid; i < T; i += kMergeThreads) w.live[i] = w.next[i];
    __syncthreads();
    MERGE_TICK(6)
  }
  if (tid == 0) cnt[C_ROUNDS] = round;
  MERGE_TICK(8)
  if (sh_n[0] != 0) return;                          // construction did not finish: n_codes stays -1
  RankLds &l = *reinterpret_cast<RankLds *>(w.live);
  rank_picks(p, ut, w.picked, l, lds_words - T4 - (int)(sizeof(RankLds) / sizeof(uint32_t)));
}

}  // namespace

spindle_status launch_merge(const ShallowParams &p, hipStream_t st) {
  const int n = p.n;
  const dim3 pg((unsigned)((p.T + kPhaseThreads / kWave - 1) / (kPhaseThreads / kWave)), p.UT);
  const int first_round = n <= kTailOnly ? 0 : kGridRounds;
  for (int round = 0; round < first_round; ++round) {
    ProfScope ps("shallow_merge_grid", st);
    hipLaunchKernelGGL(merge_onehop, pg, dim3(kPhaseThreads), 0, st, p, round);
    hipLaunchKernelGGL(merge_twohop, pg, dim3(kPhaseThreads), 0, st, p, round);
    hipLaunchKernelGGL(merge_update, pg, dim3(kPhaseThreads), 0, st, p, round);
  }
  // LDS: bits picked, live and next, keys; afterwards, in the place of all but the first, the codebook order's arrays
  // and the picks twice, as far as two blocks per compute unit allow or the keys took that much anyway
  const size_t T4 = (size_t)((p.T + 3) & ~3), rank = T4 + sizeof(RankLds) / sizeof(uint32_t);
  size_t words = 3 * T4 + (n <= kKeysInLds ? (size_t)p.n32 : 0);
  const size_t want = rank + 2 * (size_t)n, half = 78 * 1024 / sizeof(uint32_t);
  if (words < want) words = want <= half ? want : (words < half ? half : words);
  static LdsLimit lim_merge;                              // raised once per device to the largest size in use
  if (spindle_status e = allow_lds(lim_merge, reinterpret_cast<const void *>(&shallow_merge),
                                   (kKeysInLds + 3 * (kKeysInLds / 32 + 4)) * sizeof(uint32_t))) return e;
  { ProfScope ps("shallow_merge", st);
  hipLaunchKernelGGL(shallow_merge, dim3(p.UT), dim3(kMergeThreads), words * sizeof(uint32_t), st, p, first_round, (int)words); }
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}

}  // namespace spindle
