// Outputs and the codebook cap (Alg. 1; Eq. 4 for the re-pointed tokens).
#include "mma.h"
#include "shallow.h"

namespace spindle {
namespace {

// References (Eq. 12, renumbered in codebook order) and codebook entries (Eq. 11), grid-wide.  A
// thread takes a token's reference, a group of lanes with 16 bytes each (16 lanes; 32 for fp32) an entry
// row.  Bound by latency, three dependent loads per reference and two per entry, so a block takes 32
// entries in a few trips and four references per thread at once; a problem's blocks share an XCD's L2.  Where a
// block for every 1024 tokens walked its entries one row per wave at a time and every wave updated the counter
// of cut tokens: 64 problems of 32768 tokens with 4096 entries 225 -> 59 us, 2 of 32768 37 -> 9 us, one of 512
// tokens with 128 entries 27 -> 7 us.
constexpr int kEmitThreads = 256;

// Factor that takes a row of magnitude m to its unit vector x 2^10 (0 for a zero row).
__device__ __forceinline__ float unit_factor(double m) { return (float)(m > 0.0 ? (double)kUnitScale / m : 0.0); }

constexpr int kEmitTokens = 4 * kEmitThreads;        // per block

template <int DT>
__global__ __launch_bounds__(kEmitThreads) void shallow_emit(ShallowParams p, int nblk) {
  typedef typename Elem<DT>::type T;
  constexpr int kPer = 16 / (int)sizeof(T), kLanes = kHeadDim / kPer;   // elements per lane, lanes per row
  __shared__ int wsum[kEmitThreads / kWave];
  __shared__ unsigned sh_at;
  const int item = xcd_item();
  if (item >= p.UT * nblk) return;
  const int ut = item / nblk, blk = item % nblk, n = p.n;
  const size_t base = (size_t)ut * n;
  const int t = ut / p.U, u = ut % p.U;
  const int stored = p.n_codes[t][u];
  if (stored < 0) return;                        // the merge did not finish
  const int *rank = p.rank + base, *slot = p.slot + base, *rank_vert = p.rank_vert + base;
  const int lane = lane_id(), tid = threadIdx.x, wave = tid >> 6;
  const int v0 = blk * kEmitTokens + tid;
  if (blk * kEmitTokens < n) {
    int r[4], ncut = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = v0 + k * kEmitThreads < n ? (int)p.iperm[base + v0 + k * kEmitThreads] : 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = slot[r[k]];
#pragma unroll
    for (int k = 0; k < 4; ++k) r[k] = rank[r[k]];
    unsigned long long mk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = v0 + k * kEmitThreads;
      if (v < n) p.ref[t][(size_t)u * n + v] = r[k];
      mk[k] = __ballot(v < n && r[k] >= p.cap);
      ncut += __popcll(mk[k]);
    }
    if (lane == 0) wsum[wave] = ncut;
    __syncthreads();
    int at = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kEmitThreads / kWave; ++w) {
      at += w < wave ? wsum[w] : 0;
      total += wsum[w];
    }
    if (total) {                                 // one counter update per block
      if (tid == 0) sh_at = atomicAdd(p.ovf_cnt + ut, (unsigned)total);
      __syncthreads();
      at += (int)sh_at;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (mk[k] >> lane & 1ull) p.ovf[base + at + __popcll(mk[k] & ((1ull << lane) - 1ull))] = (uint32_t)(v0 + k * kEmitThreads);
        at += __popcll(mk[k]);
      }
    }
  }
  const int piece = tid % kLanes;
  const bool cut = p.counters[(size_t)ut * kCounters + C_PICKS] > p.cap;
  for (int e = (blk * kEmitThreads + tid) / kLanes; e < stored; e += nblk * (kEmitThreads / kLanes)) {
    const int vert = rank_vert[e];
    const double m = p.m64[base + vert];
    const u4 in = reinterpret_cast<const u4 *>(x_row(p, ut, vert))[piece];
    const T *x = reinterpret_cast<const T *>(&in);
    u4 out;
    T *y = reinterpret_cast<T *>(&out);
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      y[k] = Elem<DT>::from_float(m > 0.0 ? (float)((double)Elem<DT>::to_float(x[k]) / m) : 0.f);
    if (cut) {                                   // for shallow_assign: x 2^10, in fp16
      const float scale = unit_factor(m);
      _Float16 z[kPer];
#pragma unroll
      for (int k = 0; k < kPer; ++k) z[k] = (_Float16)(Elem<DT>::to_float(x[k]) * scale);
      _Float16 *to = p.Xe + (base + e) * kHeadDim + piece * kPer;
      if constexpr (kPer == 8) *reinterpret_cast<u4 *>(to) = *reinterpret_cast<const u4 *>(z);
      else *reinterpret_cast<uint2 *>(to) = *reinterpret_cast<const uint2 *>(z);
    }
    reinterpret_cast<u4 *>(reinterpret_cast<T *>(p.C[t]) + ((size_t)u * p.cap + e) * kHeadDim)[piece] = out;
  }
}

// ---------------------------------------------------------------- codebook cap
// A token whose entry was cut goes to the stored entry of highest cosine (Eq. 4), lowest
// entry index on ties, decided as the double-precision evaluation decides it.
//
// A block takes 256 cut tokens against all stored entries: fp16 matrix-core cosines of the unit vectors (the
// entries' as shallow_emit left them, streamed through LDS two stages ahead; the tokens' made on the spot), off
// from the exact value by less than kGuard.  With F the largest approximate cosine of a
// token, the exact maximum has an approximate value >= F - 2 kGuard, and so has every entry
// that ties with it.  Each lane keeps, for its token and its half of the entries, the
// running maximum and the entries seen within 2 kGuard of it (the list restarts whenever the
// maximum jumps by more than that, so it stays short).  Then a thread per token looks at the entries that are
// left: one as a rule, which is the answer.  Several become pairs of token and entry that all threads of the block
// evaluate in double precision side by side (one thread after the other: 6 us more for 512 fp32 tokens, 13 for 32 x 1024
// fp16 rows).  Where a list ran full or no cosine is a number, all entries are evaluated that way, for eight tokens at a
// time per wave.  Rows of zeros (the padding of a prompt: every one is an entry of its own, so most are cut)
// and rows that hold a NaN or an infinity need no search: their cosines are 0 or no numbers.  1024 tokens, half of them
// zero, 128 entries: the call 426 us with a search for every such token, one token at a time per block, 79 now.
// Where few tokens were cut in all, a block takes 64 of them and its waves a quarter of the products each: four
// times the blocks for four times the reads of the entries.
// What a tile of products costs besides the matrix instructions: its maximum (eight v_max3), the test whether any lane
// is within reach of its token's maximum, and in the tiles where one is, the sixteen tests.  64 problems with half of 32768
// tokens cut, 4096 entries: 1110 us with the tests in every tile and a maximum per lane, 968 now, 1.14 PFLOP/s, where the
// matrix cores alone sustain 1.6 on such operands.
// Lists in memory; in LDS 64 KiB per block, two blocks per CU: 1.81 ms where this took 1.58.
// The exact comparison of every listed entry and the search of what was left as launches of their own, and the
// entries gathered by token: 64 problems with half of 32768 tokens cut, 4096 entries, 1165 + 228 + 4 us, now 1235; 2 with 4000
// cut, 2048 entries, 74 + 20 + 4, now 48.
constexpr int kAssignThreads = 256;
constexpr int kAssignStages = 3;
constexpr int kAssignFew = 512;                        // blocks of 256 below which they take 64 tokens

template <int DT>
__global__ __launch_bounds__(kAssignThreads, 2) void shallow_assign(ShallowParams p) {
  typedef Mma<SPINDLE_F16> M;
  typedef typename Elem<DT>::type T;
  __shared__ __attribute__((aligned(1024))) char stage[kAssignStages * kStageBytes];
  __shared__ int left[kAssignThreads], nleft, npairs, first_odd, infinite;
  __shared__ unsigned long long best[kAssignThreads];   // of a token with several candidates, and its entry
  __shared__ int entry[kAssignThreads];
  const int ut = blockIdx.y, n = p.n;
  const int nov = (int)p.ovf_cnt[ut];
  const bool few = 4 * nov <= n && (long)nov * gridDim.y < (long)kAssignFew * kAssignThreads;   // (4 nov <= n: the blocks and the lists are there)
  const int per = few ? kAssignThreads / 4 : kAssignThreads, slot0 = blockIdx.x * per;
  if (slot0 >= nov) return;
  const int kept = p.n_codes[ut / p.U][ut % p.U];     // = cap whenever tokens were cut
  if (kept <= 0) return;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5, c = lane & 31;
  const char *Xe = reinterpret_cast<const char *>(p.Xe) + (size_t)ut * n * 256;
  const uint32_t *ovf = p.ovf + (size_t)ut * n;
  const float band2 = 2.f * kGuard * kUnitScale * kUnitScale;
  if (threadIdx.x == 0) {
    nleft = npairs = infinite = 0;
    first_odd = kept;
  }

  // the wave's cut tokens: 64 of them, or 32 and one of the two tiles of a stage; MFMA B operand (matrix columns = lanes)
  const int own_tile = few ? wave >> 1 : -1, lists = few ? 4 : 2;
  int slot[2];
  bool valid[2], seeks[2];                             // (a zero row, a NaN or an infinity seeks nothing, see below)
  M::frag af[2][M::kSteps];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    slot[cb] = slot0 + (few ? 32 * (wave & 1) : 64 * wave + 32 * cb) + c;
    valid[cb] = slot[cb] < nov && !(few && cb > 0);
    seeks[cb] = false;
#pragma unroll
    for (int ks = 0; ks < M::kSteps; ++ks) af[cb][ks] = M::zero();
    if (valid[cb]) {
      const int tok = (int)ovf[slot[cb]];
      const double mg = p.m64[(size_t)ut * n + tok];
      seeks[cb] = mg > 0.0 && mg < (double)INFINITY;
      if constexpr (DT == SPINDLE_F32) {
        const char *row = reinterpret_cast<const char *>(p.Xh) + ((size_t)ut * n + tok) * 256;
#pragma unroll
        for (int ks = 0; ks < M::kSteps; ++ks) af[cb][ks] = M::load(row, ks, g);
      } else {
        const char *row = x_row(p, ut, tok);
        const float scale = unit_factor(mg);
#pragma unroll
        for (int ks = 0; ks < M::kSteps; ++ks) {
          const u4 in = *reinterpret_cast<const u4 *>(row + ks * 32 + g * 16);
          const T *x = reinterpret_cast<const T *>(&in);
#pragma unroll
          for (int k = 0; k < 8; ++k) af[cb][ks][k] = (_Float16)(Elem<DT>::to_float(x[k]) * scale);
        }
      }
    }
  }
  // staged entry 16*g + v of a tile is fed to matrix row 8*(v/4) + 4*g + v%4 (as in shallow_rows)
  const int prow = 16 * ((c >> 2) & 1) + 4 * (c >> 3) + (c & 3);
  int soff[M::kSteps];
#pragma unroll
  for (int ks = 0; ks < M::kSteps; ++ks)
    soff[ks] = prow * 256 + (((2 * ks + g) ^ ((prow & 7) | ((prow & 16) >> 1))) << 4);
  const uint32_t stage_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)stage;
  const int nstages = (kept + kStageCols - 1) / kStageCols;
  auto dma = [&](int s) __attribute__((always_inline)) {   // load q of wave w: rows (4 w + q) * 4 + lane / 16; rows past the last entry are masked below
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = (wave * 4 + q) * 4 + (lane >> 4);
      lds_dma16_at(Xe, (uint32_t)min(s * kStageCols + r, kept - 1) * 256u + (((lane & 15) ^ ((r & 7) | ((r & 16) >> 1))) << 4),
                   stage_lds + (s % kAssignStages) * kStageBytes + (wave * 4 + q) * 1024);
    }
  };
  float runmax[2] = {-INFINITY, -INFINITY};
  int cnt[2] = {0, 0};
  uint2 *cand = p.ccand + (size_t)ut * n * 2 * kCandCap;
  auto list_of = [&](int cb) { return (size_t)slot[cb] * lists + (few ? 2 * own_tile : 0) + g; };
  auto collect = [&](f16v a, int cb, int j0) __attribute__((always_inline)) {
    if (j0 + 32 > kept) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + 16 * g + v >= kept) a[v] = -INFINITY;
    }
    float t = a[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) t = fmaxf(t, a[v]);
    // (the two lanes of a token know of each other's maximum)
    const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    const float nm = fmaxf(fmaxf(runmax[cb], __uint_as_float(both[0])), __uint_as_float(both[1]));
    if (nm > runmax[cb] + band2) cnt[cb] = 0;         // everything collected so far is out of reach
    runmax[cb] = nm;
    const float thr = fmaxf(nm - band2, -0x1p126f);   // (nothing but -INFINITY seen: nothing to collect)
    if (!__any(t >= thr)) return;                      // most tiles once the maxima are known
    // bit v of `hits`: a[v] >= thr, from the sign of a[v] - thr (sixteen tests and branches, one per
    // value, cost several times the matrix instructions of the tile; hits are rare)
    uint32_t miss = 0;
#pragma unroll
    for (int v = 15; v >= 0; --v) miss = __builtin_amdgcn_alignbit(miss, __float_as_uint(a[v] - thr), 31);
    uint32_t hits = t >= thr && seeks[cb] ? ~miss & 0xFFFFu : 0u;
    if (hits) {
      uint2 *list = cand + list_of(cb) * kCandCap;     // (with the tile's maximum, which is the value of all but a few)
      do {
        const int v = __builtin_ctz(hits);
        hits &= hits - 1;
        if (cnt[cb] < kCandCap) list[cnt[cb]] = make_uint2((uint32_t)(j0 + 16 * g + v), __float_as_uint(t));
        ++cnt[cb];
      } while (hits);
    }
  };

  dma(0);
  if (nstages > 1) dma(1);
  for (int s = 0; s < nstages; ++s) {
    // the wave's loads of stage s have landed (and everything else before them; those of stage s + 1 may be on their
    // way, and a list entry behind them only makes the wait longer), behind the barrier every wave's; the buffer
    // of stage s - 1 is free
    if (s + 1 < nstages) __builtin_amdgcn_s_waitcnt(0x0F74);
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    if (s + 2 < nstages) dma(s + 2);
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const int j0 = s * kStageCols + 32 * ct;
      if (j0 >= kept) break;
      if (few && ct != own_tile) continue;            // wave-uniform, as below
      const char *st = stage + (s % kAssignStages) * kStageBytes + ct * 32 * 256;
      f16v acc0, acc1;
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc0[v] = 0.f; acc1[v] = 0.f; }
      if (few) {
#pragma unroll
        for (int ks = 0; ks < M::kSteps; ++ks) acc0 = M::mma(*reinterpret_cast<const M::frag *>(st + soff[ks]), af[0][ks], acc0);
        collect(acc0, 0, j0);
      } else {
#pragma unroll
        for (int ks = 0; ks < M::kSteps; ++ks) {
          const M::frag f = *reinterpret_cast<const M::frag *>(st + soff[ks]);
          acc0 = M::mma(f, af[0][ks], acc0);
          acc1 = M::mma(f, af[1][ks], acc1);
        }
        collect(acc0, 0, j0);
        collect(acc1, 1, j0);
      }
    }
  }

  // what the lanes found, by token of the block and list
  __syncthreads();                                    // the stages have been read
  float2 *stat = reinterpret_cast<float2 *>(stage);
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
    if (valid[cb]) stat[list_of(cb) - (size_t)slot0 * lists] = make_float2(runmax[cb], __int_as_float(cnt[cb]));
  __syncthreads();                                    // (and the lists in memory are every wave's to read)
  int32_t *ref = p.ref[ut / p.U] + (size_t)(ut % p.U) * n;
  const int *rank_vert = p.rank_vert + (size_t)ut * n;
  const int tid = threadIdx.x;
  constexpr int kPairs = kAssignThreads * 2 * kCandCap;   // (64 tokens with four lists: half of them)
  unsigned long long *pair_key = reinterpret_cast<unsigned long long *>(stage);      // [kPairs], where `stat` was
  uint32_t *pair = reinterpret_cast<uint32_t *>(pair_key + kPairs);   // [kPairs] token of the block << 16 | entry
  static_assert(sizeof(stage) >= kPairs * 12 && kPairs * 8 >= kAssignThreads * 2 * (int)sizeof(float2), "pairs behind what was found");
  int inf_tok = -1, several = -1;                     // the thread's token if it has that
  best[tid] = 0;
  if (tid < per && slot0 + tid < nov) {
    const int a = (int)ovf[slot0 + tid];
    const float2 *own = stat + tid * lists;
    float top = -INFINITY;
    bool full = false;
    for (int h = 0; h < lists; ++h) {
      top = fmaxf(top, own[h].x);
      full |= __float_as_int(own[h].y) > kCandCap;
    }
    const float thr = top - band2;
    const uint2 *mine = cand + (size_t)(slot0 + tid) * lists * kCandCap;
    int found = 0, bj = 0x7FFFFFFF;
    for (int h = 0; h < lists && !full; ++h)
      for (int i = 0; i < __float_as_int(own[h].y); ++i) {
        const uint2 e = mine[h * kCandCap + i];
        if (__uint_as_float(e.y) >= thr) {
          ++found;
          bj = (int)e.x;
        }
      }
    if (full || found == 0) {
      const double mg = p.m64[(size_t)ut * n + a];
      if (!(mg > 0.0)) ref[a] = 0;                    // a zero row or a NaN: its cosine is 0 with every entry
      else if (mg < (double)INFINITY) left[atomicAdd(&nleft, 1)] = a;
      else inf_tok = a, infinite = 1;
    } else if (found == 1) {
      ref[a] = bj;
    } else {
      several = a;
      int at = atomicAdd(&npairs, found);
      for (int h = 0; h < lists; ++h)
        for (int i = 0; i < __float_as_int(own[h].y); ++i) {
          const uint2 e = mine[h * kCandCap + i];
          if (__uint_as_float(e.y) >= thr) pair[at++] = (uint32_t)tid << 16 | e.x;
        }
    }
  }
  __syncthreads();
  if (npairs) {
    for (int i = tid; i < npairs; i += kAssignThreads) {
      const int t = (int)(pair[i] >> 16), j = (int)(pair[i] & 0xFFFFu);
      const double cv = cos64<DT, 4>(p, ut, (int)ovf[slot0 + t], rank_vert[j]);
      pair_key[i] = cv == cv ? order_key(cv) : 0;
      atomicMax(&best[t], pair_key[i]);
    }
    entry[tid] = 0x7FFFFFFF;
    __syncthreads();
    for (int i = tid; i < npairs; i += kAssignThreads)
      if (pair_key[i] != 0 && pair_key[i] == best[pair[i] >> 16]) atomicMin(&entry[pair[i] >> 16], (int)(pair[i] & 0xFFFFu));
    __syncthreads();
    if (several >= 0) ref[several] = entry[tid] == 0x7FFFFFFF ? 0 : entry[tid];
    __syncthreads();
  }
  if (infinite) {                                     // an infinity: 0 with entries that are zero or hold a NaN, no number else
    for (int j = tid; j < kept; j += kAssignThreads)
      if (!(p.m64[(size_t)ut * n + rank_vert[j]] > 0.0)) atomicMin(&first_odd, j);
    __syncthreads();
    if (inf_tok >= 0) ref[inf_tok] = first_odd < kept ? first_odd : 0;
  }

  // The tokens left over, 32 at a time in four groups: a wave has a group of eight and a share of the entries, a
  // lane an entry and its products with the eight tokens, whose numbers come from LDS (all lanes the same).
  constexpr int kGroup = 8, kWaves = kAssignThreads / kWave;
  typedef float Row[kHeadDim][kGroup];
  Row *rows = reinterpret_cast<Row *>(stage);         // [kWaves]
  double *mag = reinterpret_cast<double *>(stage + kWaves * sizeof(Row));        // [kWaves][kGroup]
  double *best_v = mag + kWaves * kGroup;             // [kWaves][kGroup]
  int *best_j = reinterpret_cast<int *>(best_v + kWaves * kGroup);
  static_assert(sizeof(stage) >= kWaves * (sizeof(Row) + kGroup * 20), "rows of four groups and what their waves found");
  for (int i0 = 0; i0 < nleft; i0 += kWaves * kGroup) {
    const int left_here = nleft - i0, ngroups = left_here > 2 * kGroup ? 4 : left_here > kGroup ? 2 : 1;
    for (int i = tid; i < ngroups * kGroup * kHeadDim; i += kAssignThreads) {
      const int k = i / kHeadDim, dim = i % kHeadDim, tok = left[min(i0 + k, nleft - 1)];
      rows[k / kGroup][dim][k % kGroup] = Elem<DT>::to_float(reinterpret_cast<const T *>(x_row(p, ut, tok))[dim]);
      if (dim == 0) mag[k] = p.m64[(size_t)ut * n + tok];
    }
    __syncthreads();
    const int grp = wave % ngroups, step = kWaves / ngroups;
    double bv[kGroup];
    int bj[kGroup];
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
      bv[k] = -INFINITY;
      bj[k] = 0x7FFFFFFF;
    }
    int j = (wave / ngroups) * kWave + lane, vert = j < kept ? rank_vert[j] : 0;
    for (; j < kept; j += step * kWave) {              // ascending: the first of equal values stays
      const u4 *row = reinterpret_cast<const u4 *>(x_row(p, ut, vert));
      const double mj = p.m64[(size_t)ut * n + vert];
      if (j + step * kWave < kept) vert = rank_vert[j + step * kWave];
      constexpr int kPer = 16 / sizeof(T), kAhead = 8;
      double acc[kGroup] = {};
#pragma unroll 1
      for (int q0 = 0; q0 < kHeadDim / kPer; q0 += kAhead) {
        u4 in[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) in[q] = row[q0 + q];
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
#pragma unroll
          for (int e = 0; e < kPer; ++e) {
            const double y = (double)Elem<DT>::to_float(reinterpret_cast<const T *>(&in[q])[e]);
#pragma unroll
            for (int k = 0; k < kGroup; ++k) acc[k] += (double)rows[grp][(q0 + q) * kPer + e][k] * y;
          }
      }
#pragma unroll
      for (int k = 0; k < kGroup; ++k) {               // as cos64
        const double den = mag[grp * kGroup + k] * mj, cv = den > 0.0 ? acc[k] / den : 0.0;
        if (cv > bv[k]) { bv[k] = cv; bj[k] = j; }
      }
    }
#pragma unroll
    for (int k = 0; k < kGroup; ++k) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(bv[k], o);
        const int oj = __shfl_xor(bj[k], o);
        if (ov > bv[k] || (ov == bv[k] && oj < bj[k])) { bv[k] = ov; bj[k] = oj; }
      }
      if (lane == 0) {
        best_v[wave * kGroup + k] = bv[k];
        best_j[wave * kGroup + k] = bj[k];
      }
    }
    __syncthreads();
    if (tid < min(left_here, ngroups * kGroup)) {
      const int own = tid / kGroup, k = tid % kGroup;
      double v = best_v[own * kGroup + k];
      int jj = best_j[own * kGroup + k];
      for (int w = own + ngroups; w < kWaves; w += ngroups) {
        const double ov = best_v[w * kGroup + k];
        const int oj = best_j[w * kGroup + k];
        if (ov > v || (ov == v && oj < jj)) { v = ov; jj = oj; }
      }
      ref[left[i0 + tid]] = jj == 0x7FFFFFFF ? 0 : jj;   // (no cosine is a number)
    }
    __syncthreads();
  }
}

}  // namespace

spindle_status launch_codebook(const ShallowParams &p, hipStream_t st) {
  const int n = p.n;
  { ProfScope ps("shallow_emit", st);
  // as many blocks as the references or the entries ask for, whichever is more
  const int kept = p.cap < n ? p.cap : n;
  const int nref = (n + kEmitTokens - 1) / kEmitTokens, ncode = (kept + 31) / 32, nblk = nref > ncode ? nref : ncode;
  const dim3 eg(xcd_grid((size_t)p.UT * nblk));
  if (p.dtype == SPINDLE_F16) hipLaunchKernelGGL(shallow_emit<SPINDLE_F16>, eg, dim3(kEmitThreads), 0, st, p, nblk);
  else if (p.dtype == SPINDLE_BF16) hipLaunchKernelGGL(shallow_emit<SPINDLE_BF16>, eg, dim3(kEmitThreads), 0, st, p, nblk);
  else hipLaunchKernelGGL(shallow_emit<SPINDLE_F32>, eg, dim3(kEmitThreads), 0, st, p, nblk); }
  if (p.cap < n) {                                    // (else no entry can be cut)
    ProfScope ps("shallow_assign", st);
    const dim3 ag((n + kAssignThreads - 1) / kAssignThreads, p.UT);
    if (p.dtype == SPINDLE_F16) hipLaunchKernelGGL(shallow_assign<SPINDLE_F16>, ag, dim3(kAssignThreads), 0, st, p);
    else if (p.dtype == SPINDLE_BF16) hipLaunchKernelGGL(shallow_assign<SPINDLE_BF16>, ag, dim3(kAssignThreads), 0, st, p);
    else hipLaunchKernelGGL(shallow_assign<SPINDLE_F32>, ag, dim3(kAssignThreads), 0, st, p);
  }
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}

}  // namespace spindle
