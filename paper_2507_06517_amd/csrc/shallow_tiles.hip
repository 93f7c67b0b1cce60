// Similarity graph of the codebook path as neighbour lists (Eq. 4, 9, 10): the tokens sorted so that
// similar ones stand together, the pairs of 32-token tiles that can hold a pair above theta found
// from short sketches, and the cosines themselves only for those.
#include "mma.h"
#include "shallow.h"

namespace spindle {
namespace {

typedef int i4v __attribute__((ext_vector_type(4)));
typedef int i8v __attribute__((ext_vector_type(8)));
typedef int i16v __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- order
// Every token goes to a pivot (up to 1024 tokens taken at equal distances): the lowest one whose sketch
// product lies in the same step of 16384 (0.18 of a cosine) as the largest.  The lowest instead of
// the nearest, so that the tokens of one cluster stay together when several pivots belong to it, and
// mostly also when none does and the products are all small.  The steps end at 0.51, 0.70, 0.88: near
// 0.53, where the products of unrelated tokens lie, a step would gather every second pivot's tokens at
// the lowest pivots (kStepOffset moves them away from there).
// Keys that share a direction differ in the rest only, so where the mean of a sample of the pivots is more than
// kMeanSome of the mean squared length left without it, it is taken off the pivots' coordinates.  Products of unrelated tokens
// then lie around that of the norms the sketches leave out, with a spread of 0.129 of the length left; the steps
// are about three times that wide, and one ends 2.7 times it above.  Where the mean is most of the length, more than
// kMeanMost, the norms vary more than what is left: their four bytes then carry the token's own product with
// the mean instead.
// The pivots' bytes are rounded to multiples of 16 (0.015 of a cosine), so that products are multiples of 16 and start at
// the number of their result register: the maximum of a tile of pivots, which is all that is taken of it, says which one it
// was; a lower pivot of a tile starts 1/16 of a step ahead of the next, so that tokens near several agree on one (taking
// the nearest parts every fifth cluster of 8192 tokens: 5 % more for shallow_rows).  With the register put into each product
// behind a mask the vector work was twice the matrix instructions.
constexpr int kStepOffset = 3008;
constexpr float kStepEnd = 0.345f, kStep = 0.388f, kMeanSome = 0.15f, kMeanMost = 1.9f;
// Tokens that are near no pivot (a cosine of 0.73, the last step from 0.88 on; without the mean, a product of kMeanNear of the
// length left, between the largest of 1024 unrelated ones and nearly all of a cluster's own) go ahead of the others: what is isolated
// stands together then and doesn't widen the tiles of what is not.  So do small buckets: up to kFewest tokens where more than one token in
// kFarShare is near no pivot, and otherwise what a second pivot took of a cluster: a kRemnant-th of what buckets have as a rule, at most
// kFewest.  More than that is something else, the heavy tokens of clusters in keys with a common mean, and a tile of them is marked for
// ten clusters.  16 problems of 8192 tokens in 128 clusters, a twentieth of them heavy, with a mean of half their length, 4 of 23000 in 200, 2 of
// 18445 in 26, us per call: with the step above instead of kMeanNear and up to eight tokens to a pivot 220, 203, 243, now 166, 178, 235.
// (With isolated tokens, single ones only go first: 2 problems of 32768 kept rows of repeated heads, a fifth isolated, 316 us, not 303, of 48000
// 435 and 424; the 16 problems with a mean, a tenth isolated, 241 and 260.)
// Where sketches aren't asked (kByVector) all tokens keep to their pivots but for the remnants.
constexpr int kMeanOf = 128, kNearStep = 5, kFarShare = 16, kRemnant = 128;
constexpr uint32_t kFewest = 8;
constexpr float kMeanNear = 0.58f;
constexpr int kPivotThreads = 256;

template <int kTiles>                                  // of 32 tokens per wave
__global__ __launch_bounds__(kPivotThreads, 2) void shallow_pivots(ShallowParams p, int npiv, int nblk) {
  __shared__ __attribute__((aligned(16))) char piv[kPivots * kSketchBytes];    // fragment order: tile, half, lane
  __shared__ uint32_t cnt[kBuckets];
  __shared__ __attribute__((aligned(16))) int init[kPivots];                   // what is taken off a pivot's products
  __shared__ __attribute__((aligned(16))) int sum[kSketchBytes], mean4[kSketchBytes / 4];
  __shared__ int sum_sq;
  const int item = xcd_item();
  if (item >= p.UT * nblk) return;
  const int ut = item / nblk, blk = item % nblk, n = p.n;
  const uint8_t *sk = p.sk0 + (size_t)ut * n * kSketchBytes;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, g = lane >> 5, c = lane & 31;
  auto piv_at = [](int j, int piece) { return (j >> 5) * kTileBytes + (piece >> 1) * 1024 + ((piece & 1) * 32 + (j & 31)) * 16; };
  constexpr int kAtOnce = 8;                           // loads of a thread in flight
  for (int i0 = tid; i0 < npiv * 4; i0 += kAtOnce * kPivotThreads) {
    u4 v[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const int i = min(i0 + q * kPivotThreads, npiv * 4 - 1), j = i >> 2, piece = i & 3;   // piece = 2 * half + lane group
      const int tok = (int)((uint32_t)j * (uint32_t)n / (uint32_t)npiv);   // (below 2^26)
      v[q] = *reinterpret_cast<const u4 *>(sk + (size_t)tok * kSketchBytes + piece * 16);
    }
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const int i = i0 + q * kPivotThreads;
      if (i >= npiv * 4) break;
      // every byte + 8 without carries into the next, 127 + 8 back into the range, then the multiple of 16 below
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint32_t sign = v[q][k] & 0x80808080u, up = (v[q][k] & 0x7F7F7F7Fu) + 0x08080808u;
        v[q][k] = ((up ^ sign) - ((up & ~sign & 0x80808080u) >> 3)) & 0xF0F0F0F0u;
      }
      *reinterpret_cast<u4 *>(piv + piv_at(i >> 2, i & 3)) = v[q];
    }
  }
  for (int i = tid; i < kBuckets; i += kPivotThreads) cnt[i] = 0;
  if (tid < kSketchBytes) sum[tid] = 0;
  if (tid == 0) sum_sq = 0;
  // the wave's tokens: matrix columns = lanes
  i4v bf[kTiles][2];
  int tok[kTiles];
#pragma unroll
  for (int r = 0; r < kTiles; ++r) {
    tok[r] = (blk * (kPivotThreads / kWave) + wave) * (kTiles * kTile) + r * kTile + c;
    const uint8_t *s = sk + (size_t)(tok[r] < n ? tok[r] : n - 1) * kSketchBytes + g * 16;
    bf[r][0] = *reinterpret_cast<const i4v *>(s);
    bf[r][1] = *reinterpret_cast<const i4v *>(s + 32);
  }
  const int every = max(1, npiv / kMeanOf), nmean = (npiv + every - 1) / every;
  __syncthreads();
  {
    // a thread sums four bytes of every 16th of the sample
    const int d = tid & 15;
    int a[4] = {0, 0, 0, 0}, sq = 0;
#pragma unroll 8
    for (int j = (tid >> 4) * every; j < npiv; j += 16 * every) {
      const int x = *reinterpret_cast<const int *>(piv + piv_at(j, d >> 2) + (d & 3) * 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] += __builtin_amdgcn_sbfe(x, 8 * k, 8);
      const int y = (d & 3) == 3 ? x & 0x00FFFFFF : x;   // (the last bytes are norms)
      sq = __builtin_amdgcn_sdot4(y, y, sq, false);
    }
#pragma unroll
    for (int o = 32; o >= 16; o >>= 1) {
#pragma unroll
      for (int k = 0; k < 4; ++k) a[k] += __shfl_xor(a[k], o);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o);
    if (lane < 16)
#pragma unroll
      for (int k = 0; k < 4; ++k) atomicAdd(&sum[4 * d + k], a[k]);
    if (lane == 0) atomicAdd(&sum_sq, sq);
  }
  __syncthreads();
  if (tid < kSketchBytes / 4) {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if ((tid & 3) < 3 || k < 3) m |= ((uint32_t)(int)rintf((float)sum[4 * tid + k] / (float)nmean) & 0xFFu) << (8 * k);
    mean4[tid] = (int)m;
  }
  __syncthreads();
  int mm = 0;                                          // squared length of the mean
#pragma unroll
  for (int d = 0; d < kSketchBytes / 4; ++d) mm = __builtin_amdgcn_sdot4(mean4[d], mean4[d], mm, false);
  float norms = 0.f;                                   // mean product of the norms
#pragma unroll
  for (int d = 15; d < kSketchBytes; d += 16) norms += (float)sum[d] * (float)sum[d] / ((float)nmean * (float)nmean);
  // (every block of a problem comes to the same figures)
  const float left = fmaxf((float)sum_sq / (float)nmean - (float)mm, 1.f);
  const bool some = (float)mm > kMeanSome * left, most = (float)mm > kMeanMost * left;
  const int bits = some ? min(14, max(10, (int)rintf(log2f(kStep * left)))) : 14, mask = -(1 << bits), ahead = bits - 4;
  const int off = some ? -(int)((most ? 0.f : norms) + kStepEnd * left) : kStepOffset;
  for (int j = tid; some && j < npiv; j += kPivotThreads) {
    int x = off;
#pragma unroll
    for (int piece = 0; piece < 4; ++piece) {
      const i4v v = *reinterpret_cast<const i4v *>(piv + piv_at(j, piece));
      const i4v m = *reinterpret_cast<const i4v *>(mean4 + 4 * piece);
#pragma unroll
      for (int k = 0; k < 4; ++k) x -= __builtin_amdgcn_sdot4(v[k], m[k], 0, false);
    }
    const int last = 15 - (((j >> 3) & 3) * 4 + (j & 3));   // 15 less the result register of row j of a tile
    init[j] = ((x & ~15) | last) + (last << ahead);
    if (most)
#pragma unroll
      for (int piece = 0; piece < 4; ++piece) piv[piv_at(j, piece) + 15] = 112;
  }
  if (blk == 0 && tid < 2) p.mean[2 * ut + tid] = some ? (uint32_t)mean4[tid] : 0u;
  if (most) {
#pragma unroll
    for (int r = 0; r < kTiles; ++r) {
      int x = 0;                                       // (a lane has pieces g and g + 2 of the four)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const i4v m = *reinterpret_cast<const i4v *>(mean4 + 4 * (2 * h + g));
#pragma unroll
        for (int k = 0; k < 4; ++k) x = __builtin_amdgcn_sdot4(bf[r][h][k], m[k], x, false);
      }
      x += __shfl_xor(x, 32);
      const int q = min(508, max(-508, (int)rintf((float)(mm - x) * (1.f / 112.f))));   // dealt out to the four
      bf[r][0][3] = (bf[r][0][3] & 0x00FFFFFF) | ((q + g) >> 2) << 24;
      bf[r][1][3] = (bf[r][1][3] & 0x00FFFFFF) | ((q + 2 + g) >> 2) << 24;
    }
  }
  __syncthreads();
  // The largest product and, in the four bits below it, its result register; a later tile of pivots only counts if its step is
  // higher.
  int best[kTiles], best_pt[kTiles];
#pragma unroll
  for (int r = 0; r < kTiles; ++r) {
    best[r] = INT32_MIN;
    best_pt[r] = 0;
  }
  auto compare = [&](auto first) __attribute__((always_inline)) {   // first(pt): what the products of a pivot tile start at
    for (int pt = 0; pt < npiv / 32; ++pt) {
      const i4v a0 = *reinterpret_cast<const i4v *>(piv + pt * kTileBytes + lane * 16);
      const i4v a1 = *reinterpret_cast<const i4v *>(piv + pt * kTileBytes + 1024 + lane * 16);
      const i16v off4 = first(pt);
#pragma unroll
      for (int r = 0; r < kTiles; ++r) {
        i16v acc = off4;
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a0, bf[r][0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(a1, bf[r][1], acc, 0, 0, 0);
        int m = acc[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) m = max(m, acc[v]);
        m -= (m & 15) << ahead;
        const bool higher = (m & mask) > best[r];
        best[r] = higher ? m : best[r];                // (no product's step is above the product)
        best_pt[r] = higher ? pt : best_pt[r];
      }
    }
  };
  if (some) {
    compare([&](int pt) {
      i16v x16;
#pragma unroll
      for (int v = 0; v < 16; v += 4) {
        const i4v x = *reinterpret_cast<const i4v *>(init + pt * 32 + mma_row(v, g));
#pragma unroll
        for (int k = 0; k < 4; ++k) x16[v + k] = x[k];
      }
      return x16;
    });
  } else {
    i16v x16;
#pragma unroll
    for (int v = 0; v < 16; ++v) x16[v] = off + 15 - v + ((15 - v) << ahead);
    compare([&](int) { return x16; });
  }
  const int near = p.by[ut / p.U] != kBySketch ? INT32_MIN : some ? (int)((kMeanNear - kStepEnd) * left) : kNearStep << 14;
#pragma unroll
  for (int r = 0; r < kTiles; ++r) {
    const int own = (best[r] & mask) | (1023 - (best_pt[r] * 32 + mma_row(15 - (best[r] & 15), g)));
    const int o = __shfl_xor(own, 32), top = o > own ? o : own, pivot = 1023 - (top & 1023);
    const int b = max(best[r], __shfl_xor(best[r], 32)) >= near ? kPivots + pivot : pivot;
    if (g == 0 && tok[r] < n) {
      p.bucket[(size_t)ut * n + tok[r]] = (uint16_t)b;
      atomicAdd(&cnt[b], 1u);
    }
  }
  __syncthreads();
  // (all additions on their way before the first result is waited for)
  constexpr int kOwn = kBuckets / kPivotThreads;
  uint32_t *total = p.total + (size_t)ut * kBuckets;
  uint16_t *before = p.before + ((size_t)ut * nblk + blk) * kBuckets;
  uint32_t x[kOwn], was[kOwn];
#pragma unroll
  for (int k = 0; k < kOwn; ++k) x[k] = cnt[k * kPivotThreads + tid];
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    was[k] = 0;
    if (x[k]) was[k] = atomicAdd(total + k * kPivotThreads + tid, x[k]);
  }
#pragma unroll
  for (int k = 0; k < kOwn; ++k)
    if (x[k]) before[k * kPivotThreads + tid] = (uint16_t)was[k];
}

// Tokens in the order of their buckets: a counting sort.  shallow_pivots left how many tokens a bucket has and which
// place within it a block's tokens start at.  (With counts per block that every block added up, half as many buckets took 15 us
// on 16 problems of 32768 tokens and 54 on 64; now 6 and 18.)
constexpr int kOrderThreads = 1024;

__global__ __launch_bounds__(kOrderThreads) void shallow_order(ShallowParams p, int nblk, int per) {
  __shared__ int cursor[kBuckets];
  __shared__ uint32_t wsum[kOrderThreads / kWave];
  __shared__ uint2 sums[kOrderThreads / kWave];
  static_assert(kBuckets == 2 * kOrderThreads, "two buckets per thread");
  const int item = xcd_item();
  if (item >= p.UT * nblk) return;
  const int ut = item / nblk, blk = item % nblk, n = p.n;
  const size_t base = (size_t)ut * n;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int tok = blk * per + tid;                     // (per: tokens of a block, no more than threads)
  const bool on = tid < per && tok < n;
  const int b = on ? (int)p.bucket[base + tok] : 0;
  const uint2 total = reinterpret_cast<const uint2 *>(p.total + (size_t)ut * kBuckets)[tid];
  const ushort2 before = reinterpret_cast<const ushort2 *>(p.before + ((size_t)ut * nblk + blk) * kBuckets)[tid];
  // tokens near no pivot, near one, and how many of the latter share a bucket with one of them on average
  uint32_t count = 2 * tid < kPivots ? total.x + total.y : (total.x + total.y) << 16;   // (at most 65535 in all)
  uint32_t square = 2 * tid < kPivots ? 0u : (total.x * total.x >> 7) + (total.y * total.y >> 7);
  count = (uint32_t)lanes_up_to((int)count);
  square = (uint32_t)lanes_up_to((int)square);
  if (lane == kWave - 1) sums[wave] = make_uint2(count, square);
  __syncthreads();
  count = square = 0;
#pragma unroll
  for (int w = 0; w < kOrderThreads / kWave; ++w) {
    count += sums[w].x;
    square += sums[w].y;
  }
  const uint32_t nfar = count & 0xFFFFu, shared = square / max(1u, count >> 16);   // (shared: 128 of them and more)
  static_assert(kRemnant == 128, "what the squares are shifted by");
  const uint32_t few = nfar * (uint32_t)kFarShare >= (uint32_t)n ? kFewest : min(shared, kFewest);
  // both kinds of buckets at once: those that go first in the low half
  auto half = [&](int bucket, uint32_t x) { return bucket < kPivots || x <= few ? 0 : 16; };
  const int h0 = half(2 * tid, total.x), h1 = half(2 * tid + 1, total.y);
  const uint32_t own = (total.x << h0) + (total.y << h1);
  uint32_t incl = (uint32_t)lanes_up_to((int)own), all = 0;
  if (lane == kWave - 1) wsum[wave] = incl;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kOrderThreads / kWave; ++w) {
    const uint32_t x = wsum[w];
    incl += w < wave ? x : 0u;
    all += x;
  }
  const uint32_t at0 = incl - own, at1 = at0 + (total.x << h0), nfirst = all & 0xFFFFu;
  cursor[2 * tid] = (int)((h0 ? nfirst : 0u) + (at0 >> h0 & 0xFFFFu)) + before.x;
  cursor[2 * tid + 1] = (int)((h1 ? nfirst : 0u) + (at1 >> h1 & 0xFFFFu)) + before.y;
  __syncthreads();
  if (on) p.perm[base + atomicAdd(&cursor[b], 1)] = (uint16_t)tok;
}

// A window of 1024 places in that order: the tokens of each pivot sorted by eight signs of their
// sketches less the mean, which keeps together what has no
// pivot of its own.  Then everything later kernels read by position.  Sketches go to fragment order:
// tile, half of the 64 bytes, lane.
// Tokens of a pivot with fewer than kFew in the window count the ones that go before them; more are counted by signs
// (256 bins per pivot, of which no more than kMany fit the window).  Where all of them were compared, isolated tokens, which
// stand with the lowest pivots, cost 2048 comparisons each: 51 us for the kernel on two
// problems of 32768 rows, 182 on 64, now 21 and 99; a bitonic sort took longer than comparing clusters.
typedef uint32_t u6 __attribute__((ext_vector_type(6)));
typedef float f32v __attribute__((ext_vector_type(32)));

// 32 numbers / kSixScale to six-bit floats (a[0], b[0], a[1], b[1], ...) and back, the 192 bits as a lane's half of a row
// in a 32x32x64 matrix instruction.  As assembly, since the result must not share registers with the operands
// (which are read while it is written); the compiler's own form lets it.  The result may not be read by the
// instruction right behind.
__device__ __forceinline__ u6 to_six(const f16v &a, const f16v &b) {
  u6 r;
  asm("v_cvt_scalef32_2xpk16_fp6_f32 %0, %1, %2, %3\n\ts_nop 7" : "=&v"(r) : "v"(a), "v"(b), "v"(kSixScale));
  return r;
}
__device__ __forceinline__ f32v from_six(const u6 &x) {
  f32v r;
  asm("v_cvt_scalef32_pk32_f32_fp6 %0, %1, %2\n\ts_nop 7" : "=&v"(r) : "v"(x), "v"(kSixScale));
  return r;
}

// Over the two lane groups of 32; over the lanes of a group.
__device__ __forceinline__ float groups_sum(float x) {
  const auto y = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(y[0]) + __uint_as_float(y[1]);
}
__device__ __forceinline__ uint32_t max32(uint32_t x) {
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true));    // quad_perm [1,0,3,2]
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true));    // quad_perm [2,3,0,1]
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true));   // row_half_mirror
  x = max(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true));   // row_mirror
  const auto y = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return max(y[0], y[1]);
}

constexpr int kWindowThreads = 512;
constexpr int kFew = 64, kMany = kWindow / kFew;

__global__ __launch_bounds__(kWindowThreads) void shallow_window(ShallowParams p, int nwin) {
  __shared__ uint16_t order_by[kWindow];               // pivots, then the tokens' signs by place
  __shared__ uint16_t at_place[kWindow];
  __shared__ int first[kBuckets], last[kBuckets];      // places of a bucket's tokens
  __shared__ __attribute__((aligned(16))) int count[kMany][256];
  __shared__ uint8_t slot[kBuckets];
  __shared__ int nslots;
  __shared__ uint32_t starts[kWindow / kTile];         // per tile the places where a bucket starts
  __shared__ __attribute__((aligned(16))) float centre[kWindowThreads / kWave][kSketchBytes];
  const int item = xcd_item();
  if (item >= p.UT * nwin) return;
  const int ut = item / nwin, n = p.n, w0 = (item % nwin) * kWindow, w1 = min(n, w0 + kWindow);
  const size_t base = (size_t)ut * n;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const uint2 mean = reinterpret_cast<const uint2 *>(p.mean)[ut];
  const bool asks = p.asks[ut / p.U];
  static_assert(kWindow == 2 * kWindowThreads, "two places per thread");
  int tok[2], b[2], signs[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + k * kWindowThreads;
    tok[k] = w0 + i < w1 ? (int)p.perm[base + w0 + i] : -1;
  }
  for (int i = tid; i < kMany * 256 / 4; i += kWindowThreads) reinterpret_cast<int4 *>(&count[0][0])[i] = make_int4(0, 0, 0, 0);
  if (tid == 0) nslots = 0;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    b[k] = signs[k] = 0;
    if (tok[k] < 0) continue;
    b[k] = (int)p.bucket[base + tok[k]];
    const uint2 s = *reinterpret_cast<const uint2 *>(p.sk0 + (base + tok[k]) * kSketchBytes);
#pragma unroll
    for (int d = 0; d < 8; ++d)
      signs[k] |= (int)((int8_t)((d < 4 ? s.x : s.y) >> 8 * (d & 3)) < (int8_t)((d < 4 ? mean.x : mean.y) >> 8 * (d & 3))) << d;
    order_by[tid + k * kWindowThreads] = (uint16_t)b[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {                        // the tokens of a pivot stand together
    const int i = tid + k * kWindowThreads;
    if (tok[k] < 0) continue;
    if (i == 0 || order_by[i - 1] != b[k]) first[b[k]] = i;
    if (w0 + i == w1 - 1 || i == kWindow - 1 || order_by[i + 1] != b[k]) last[b[k]] = i;
  }
  __syncthreads();
  int lo[2], hi[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + k * kWindowThreads;
    lo[k] = hi[k] = 0;
    if (tok[k] < 0) continue;
    lo[k] = first[b[k]];
    hi[k] = last[b[k]] + 1;
    order_by[i] = (uint16_t)signs[k];
    if (i == lo[k] && hi[k] - lo[k] >= kFew) slot[b[k]] = (uint8_t)atomicAdd(&nslots, 1);
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const unsigned long long at = __ballot(tok[k] >= 0 && lo[k] == tid + k * kWindowThreads);
    if (lane < 2) starts[(k * kWindowThreads + wave * kWave) / kTile + lane] = (uint32_t)(at >> (32 * lane));
  }
  __syncthreads();
  int before[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + k * kWindowThreads;
    before[k] = 0;
    if (hi[k] - lo[k] >= kFew) {
      before[k] = atomicAdd(&count[slot[b[k]]][signs[k]], 1);   // of those with the same signs
    } else {
      for (int j = lo[k]; j < hi[k]; ++j) before[k] += order_by[j] < signs[k] || (order_by[j] == signs[k] && j < i);
    }
  }
  __syncthreads();
  for (int q = wave; q < nslots; q += kWindowThreads / kWave) {   // counts to those of lower signs
    int4 c = *reinterpret_cast<int4 *>(&count[q][4 * lane]);
    const int sum = c.x + c.y + c.z + c.w;
    int incl = sum;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int x = __shfl_up(incl, o);
      if (lane >= o) incl += x;
    }
    incl -= sum;
    *reinterpret_cast<int4 *>(&count[q][4 * lane]) = make_int4(incl, incl + c.x, incl + c.x + c.y, incl + c.x + c.y + c.z);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (tok[k] < 0) continue;
    const int under = hi[k] - lo[k] >= kFew ? count[slot[b[k]]][signs[k]] : 0;
    at_place[lo[k] + under + before[k]] = (uint16_t)tok[k];
  }
  __syncthreads();
  // A wave takes 32 places at a time: their sketches are read four lanes to a row, turned to fragment order in LDS
  // (which the counts no longer need) and rounded to six-bit floats.  Then the ball around them: the rounded mean, and how far
  // the farthest is from it.  Where a bucket starts inside the tile, the one that starts next to its middle parts it
  // in two, each with a ball of its own, as far as a window has room for seconds (a tile of many buckets is of isolated
  // tokens, and stays whole).
  uint8_t *sk = p.sk + (size_t)ut * p.Tp * kSixBytes;
  char *turn = reinterpret_cast<char *>(&count[0][0]) + wave * kTileBytes;
  static_assert(sizeof(count) >= kWindowThreads / kWave * kTileBytes, "a tile per wave");
  // (a window has half of the tiles whose balls stand together, and half of the seconds)
  static_assert(kBallTiles * kTile == 2 * kWindow && kWindow / kTile == kTile, "two windows, a lane per tile of one");
  const int half_at = (item % nwin & 1) * kTile;       // its first tile among them
  const size_t group = (size_t)ut * (nwin / 2) + item % nwin / 2;
  uint8_t *centres = p.skc + group * (3 * kSixBytes);
  float2 *balls = p.ball + group * kBalls;
  const uint32_t inside = starts[lane & 31] >> 1;
  const uint32_t parted = (uint32_t)__ballot(inside != 0 && __popc(inside) <= 2);
  constexpr int kSeconds = kTile / 2;
  const int second0 = half_at / 2;
  if (asks && wave == 0 && lane >= __popc(parted) && lane < kSeconds) balls[2 * kTile + second0 + lane] = make_float2(-0x1p30f, 0.f);
  constexpr float kUnit = 1.f / (kSixScale * kSixScale);   // products of six-bit floats are in units of kSixScale squared
  const int end = w1 < n ? w1 : p.Tp * kTile;         // the last window also fills the places past the last token
  for (int p0 = w0 + wave * kTile; p0 < end; p0 += kWindowThreads / kWave * kTile) {
    u4 v[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int pos = p0 + 16 * j + (lane >> 2);
      v[j] = u4{0, 0, 0, 0};
      if (pos < n) v[j] = reinterpret_cast<const u4 *>(p.sk0 + (base + at_place[pos - w0]) * kSketchBytes)[lane & 3];
    }
    float off = 0.f;                                   // of the bytes from what they stand for
    const int pos = p0 + (lane & 31);
    if (pos < n) {
      const int t = (int)at_place[pos - w0];
      const float2 f = p.inv_err[base + t];
      off = f.y;
      if (lane < kTile) {
        p.perm[base + pos] = (uint16_t)t;
        p.iperm[base + t] = (uint16_t)pos;
        p.invp[base + pos] = f.x;
      }
    }
    // piece k of row r at place k ^ (r / 4) % 4: sixteen consecutive lanes of either access hit all banks
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the tile before has been read
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int r = 16 * j + (lane >> 2);
      *reinterpret_cast<u4 *>(turn + r * kSketchBytes + (((lane & 3) ^ ((r >> 2) & 3)) << 4)) = v[j];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS keeps the order of one wave's accesses
    u6 six;
    float d2 = 0.f, norm2 = 0.f;                       // squared distance of the six-bit floats from the bytes, their length
    {
      f16v x[2];                                       // a row's pieces g and g + 2
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int r = lane & 31, piece = 2 * k + (lane >> 5);
        const u4 y = *reinterpret_cast<const u4 *>(turn + r * kSketchBytes + ((piece ^ ((r >> 2) & 3)) << 4));
#pragma unroll
        for (int i = 0; i < 16; ++i) x[k][i] = (float)(int)__builtin_amdgcn_sbfe((int)y[i >> 2], 8 * (i & 3), 8);
      }
      six = to_six(x[0], x[1]);
      const f32v back = from_six(six);
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const float e = back[i] - x[i & 1][i >> 1];
        d2 = fmaf(e, e, d2);
        norm2 = fmaf(back[i], back[i], norm2);
      }
      uint8_t *d = sk + (size_t)(p0 >> 5) * kSixBytes;
      reinterpret_cast<u4 *>(d)[lane] = u4{six[0], six[1], six[2], six[3]};
      reinterpret_cast<uint2 *>(d + 1024)[lane] = make_uint2(six[4], six[5]);
    }
    d2 = groups_sum(d2);
    norm2 = groups_sum(norm2) * kUnit;                 // (exact, as all sums of products of six-bit floats)
    // |a.b - a'.b'| <= e_a + e_b + e_a e_b for sketches a', b' at distances e_a, e_b; the last term is at
    // most half of the two squares.  In sketch units squared, rounded up.
    const float dist = off + sqrtf(d2) * (1.0001f / kSketchScale);
    uint32_t e = off >= 0.f && dist < 4.f ? (uint32_t)((dist + 0.5f * dist * dist) * (kSketchScale * kSketchScale * (1.f + 1e-5f))) + 2u : kSketchUnknown;
    if (pos >= n) e = 0;
    e = max32(e);
    if (!asks) {                                       // uniform
      if (lane == 0) p.etile[(size_t)ut * p.Tp + (p0 >> 5)] = e;
      continue;
    }
    const int tw = (p0 - w0) >> 5;                     // tile of the window
    const uint32_t inner = __builtin_amdgcn_readfirstlane(starts[tw]) & ~1u;
    const int nth = __popc(parted & ((1u << tw) - 1u));
    const bool two = (parted >> tw & 1) && nth < kSeconds;   // wave-uniform
    int split = kTile;
    if (two) {
      const int up = inner >> 16 ? 16 + __builtin_ctz(inner >> 16) : 64, down = inner & 0xFFFFu ? 31 - __builtin_clz(inner & 0xFFFFu) : -64;
      split = up - 16 <= 16 - down ? up : down;
    }
    // sums of the bytes over the rows of either part: a lane takes four coordinates of every fourth row
    int part[4] = {0, 0, 0, 0}, rest[4] = {0, 0, 0, 0};
    const int q = lane & 15, h = lane >> 4;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int r = 4 * j + h;
      const int x = *reinterpret_cast<const int *>(turn + r * kSketchBytes + (((q >> 2) ^ (j & 3)) << 4) + (q & 3) * 4);
      const int x0 = two && r >= split ? 0 : x;
#pragma unroll
      for (int k = 0; k < 4; ++k) part[k] = __builtin_amdgcn_sdot4(x0, 1 << (8 * k), part[k], false);
      if (two) {
#pragma unroll
        for (int k = 0; k < 4; ++k) rest[k] = __builtin_amdgcn_sdot4(x ^ x0, 1 << (8 * k), rest[k], false);
      }
    }
    const int rows = min(kTile, max(n - p0, 0)), rows0 = min(split, rows), row = lane & 31;
    for (int half = 0; half < (two ? 2 : 1); ++half) {
      const int count_of = half ? rows - rows0 : rows0;
      const float each = count_of > 0 ? 1.f / (float)count_of : 0.f;
      float4 m;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        int x = half ? rest[k] : part[k];
        const auto y = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)x, false, false);
        x = (int)(y[0] + y[1]);
        const auto z = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)x, false, false);
        reinterpret_cast<float *>(&m)[k] = (float)(int)(z[0] + z[1]) * each;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the centre before has been read
      if (lane < 16) *reinterpret_cast<float4 *>(&centre[wave][4 * q]) = m;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      f16v x[2];
#pragma unroll
      for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
          const float4 y = *reinterpret_cast<const float4 *>(&centre[wave][(2 * k + (lane >> 5)) * 16 + i]);
          x[k][i] = y.x; x[k][i + 1] = y.y; x[k][i + 2] = y.z; x[k][i + 3] = y.w;
        }
      const u6 c = to_six(x[0], x[1]);
      // squared distances from the products with the centre, which is all rows of one operand
      const i8v ca = {(int)c[0], (int)c[1], (int)c[2], (int)c[3], (int)c[4], (int)c[5], 0, 0};
      const i8v sa = {(int)six[0], (int)six[1], (int)six[2], (int)six[3], (int)six[4], (int)six[5], 0, 0};
      const f16v zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const float with = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ca, sa, zero, 2, 2, 0, 0, 0, 0)[0];
      const float own = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(ca, ca, zero, 2, 2, 0, 0, 0, 0)[0];
      const float r2 = row < rows && (row < split) == (half == 0) ? fmaxf(norm2 - 2.f * with + own, 0.f) : 0.f;
      const float far2 = __uint_as_float(max32(__float_as_uint(r2)));
      const int at = half ? 2 * kTile + second0 + nth : half_at + tw, cl = (lane & 32) + (at & 31);
      uint8_t *to = centres + (at >> 5) * kSixBytes;
      if (row == 0) {
        *reinterpret_cast<u4 *>(to + cl * 16) = u4{c[0], c[1], c[2], c[3]};
        *reinterpret_cast<uint2 *>(to + 1024 + cl * 8) = make_uint2(c[4], c[5]);
      }
      if (lane == 0) {
        balls[at] = make_float2((float)e * kUnit + 0x1p-9f, sqrtf(far2) * (1.f + 1e-5f));   // (the power: rounding of thresholds)
        if (half) p.second[group * kTile + second0 + nth] = (uint8_t)(half_at + tw);
      }
    }
    const float longest2 = __uint_as_float(max32(__float_as_uint(norm2)));
    if (lane == 0) {
      p.etile[(size_t)ut * p.Tp + (p0 >> 5)] = e;
      p.tnorm[(size_t)ut * p.Tp + (p0 >> 5)] = sqrtf(longest2) * (1.f + 1e-5f);
    }
  }
}

// ---------------------------------------------------------------- scan
// Work of shallow_scan and shallow_refine: a panel of 16 row tiles against a run of column tiles from its own
// first tile onwards.  Blocks are dealt round-robin to the 8 XCDs: an XCD sweeps the panels of one (problem,
// column group) at a time, the groups rotated by problem so that every XCD sees long and short ones.
struct ScanItem {
  int ut, I, s0, s1;                                   // stages of kScanStage column tiles
};

__device__ __forceinline__ ScanItem scan_item(const ShallowParams &p, int item, int xcd) {
  const int nI = p.Tp / kScanPanel, nS = p.Tp / kScanStage, pj = item / nI * 8 + xcd, Jg = pj % p.njg;
  ScanItem w;
  w.I = item % nI;
  w.ut = pj / p.njg;
  w.s0 = (Jg + w.ut) % p.njg * p.stages_per_item;
  w.s1 = pj < p.UT * p.njg ? min(nS, w.s0 + p.stages_per_item) : 0;
  w.s0 = max(w.s0, w.I * (kScanPanel / kScanStage));
  return w;
}

// A wave's marks, one byte per row tile and stage, into both directions of tpairs.
template <int kRowTiles>
__device__ __forceinline__ void put_marks(const ShallowParams &p, int ut, int r0, int s0, int s1, const uint8_t (*marks)[kScanRun]) {
  static_assert(kScanRun == 16, "a lane per row tile and stage");
  uint32_t *tp = p.tpairs + (size_t)ut * p.T * p.TW;
  const int lane = lane_id(), T = p.T;
  {
    const int r = lane / kScanRun, s = s0 + lane % kScanRun;
    if (r < kRowTiles && s < s1 && r0 + r < T) {
      uint32_t b = marks[r][lane % kScanRun];
      const int left = T - s * kScanStage;             // tiles that exist
      if (left < kScanStage) b &= left <= 0 ? 0u : (1u << left) - 1u;
      if (b) atomicOr(tp + (size_t)(r0 + r) * p.TW + (s >> 2), b << (8 * (s & 3)));
    }
  }
  for (int i = lane; i < (s1 - s0) * kScanStage; i += kWave) {
    const int ct = s0 * kScanStage + i;
    uint32_t m = 0;
#pragma unroll
    for (int r = 0; r < kRowTiles; ++r)
      if (r0 + r < T) m |= (uint32_t)(marks[r][i / kScanStage] >> (i % kScanStage) & 1) << r;
    if (m && ct < T) atomicOr(tp + (size_t)ct * p.TW + (r0 >> 5), m << (r0 & 31));
  }
}

// A block first asks the balls (shallow_window): a pair of a tile A and a ball with centre c and radius R can hold a sketch
// product above a threshold only if the largest product of A's sketches with c, plus R times the length of the longest
// of them, is above it.  One matrix instruction answers that for a tile and 32 balls (the ballot of the lanes is the answer as bits),
// where the sketches of 32 tiles take 32.  The panel's tiles are asked against the columns' balls, and what is
// left of the columns against the panel's balls: a tight tile excludes what it doesn't reach whatever stands on the other side.
// Then the sketches of what is left: per 32 x 32 pairs one 32x32x64 matrix instruction on six-bit floats; all the results are
// needed for is their maximum, eight v_max3 per lane (which take as long as the matrix instruction), and one comparison.
// As a rule a wave takes every fourth column tile that is left, in registers, and the panel's tiles that it is left for from LDS.
// Where most is left (isolated tokens) the row tiles' sketches stay in registers, four tiles per wave, and the column tiles
// are staged through LDS, eight at a time (fragment order: loads and reads are both linear, no bank conflicts).
// Tiles that pass are marked in both directions.
// 16 problems of 32768 tokens in drifting clusters: 280 us with all sketch products, 125 now; 64 of which half of the tokens are
// isolated 1035 and 567; 128 of 8192 in clusters 210 and 58 (and 12 to 27 more in shallow_window for the balls).  Of those 567 us the
// questions to the balls are a quarter (17400 cycles per block, by counts and clocks), the dense blocks, where a pair of tiles takes
// 43 cycles of a SIMD, four tenths, and the pairs by themselves, 165 cycles each, mostly latency, a sixth.
// A block that finds more than kRefineShare of its column tiles marked (keys with a common component, low
// thresholds) leaves all of its pairs to shallow_refine.  The panel's own columns don't count, and a
// run of similar tokens behind them is allowed for: those are true neighbours.
constexpr int kScanThreads = 256;
constexpr int kScanCols = kScanRun * kScanStage;
constexpr int kScanWords = (kScanCols + 2 * kWave - 2) / kWave * 2;   // of 32 tiles, whole windows around a run
constexpr float kBallLoose = 8.f;                      // radius that excludes nothing (0.43 of a sketch)

template <bool kWithBalls>
__global__ __launch_bounds__(kScanThreads, 4) void shallow_scan(ShallowParams p) {
  __shared__ __attribute__((aligned(1024))) char stage[2 * kScanStage * kSixBytes];   // the panel's tiles, or two stages
  static_assert(2 * kScanStage == kScanPanel, "the panel's tiles fit");
  __shared__ __attribute__((aligned(16))) uint8_t marks[kScanPanel][kScanRun];
  __shared__ int found[kScanRun];                      // marks of a stage, once for four row tiles
  __shared__ uint32_t need[kScanPanel][kScanWords];    // bit per column tile that a row tile is left with
  __shared__ float col_thr[kScanCols], col_norm[kScanCols];   // theta less a column tile's error; longest sketch
  __shared__ float row_thr[kScanPanel];                // theta less a row tile's error
  __shared__ uint32_t list[kScanThreads / kWave][kScanCols];
  const int xcd = blockIdx.x & 7;
  const ScanItem w = scan_item(p, blockIdx.x >> 3, xcd);
  if (w.s0 >= w.s1 || p.by[w.ut / p.U] != kBySketch) {
    if (threadIdx.x == 0) p.todo[blockIdx.x] = w.s0 < w.s1 && p.by[w.ut / p.U] == kByVector;
    return;
  }
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), c = lane & 31, g = lane >> 5;
  const char *sk = reinterpret_cast<const char *>(p.sk) + (size_t)w.ut * p.Tp * kSixBytes;
  const uint32_t *et = p.etile + (size_t)w.ut * p.Tp;
  const float *norm = p.tnorm + (size_t)w.ut * p.Tp;
  const int r0 = w.I * kScanPanel + wave * 4, c0 = w.s0 * kScanStage, c1 = w.s1 * kScanStage;
  const int win0 = c0 / kBallTiles, win1 = (c1 - 1) / kBallTiles;   // groups of balls of the columns
  static_assert(kBallTiles == kWave, "places of tiles in a group");
  const size_t windows = (size_t)w.ut * ((p.Tp + kBallTiles - 1) / kBallTiles);
  const int thr0 = p.scan_thr[w.ut / p.U];
  constexpr float kUnit = 1.f / (kSixScale * kSixScale);   // products are in units of kSixScale squared
  const uint32_t stage_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)stage;
  constexpr int kLoads = kScanStage * kSixBytes / 1024 / (kScanThreads / kWave);   // of 1 KiB per wave and stage
  static_assert(kLoads * 1024 * (kScanThreads / kWave) == kScanStage * kSixBytes, "whole loads");
  auto dma = [&](int s, int buffer) __attribute__((always_inline)) {
    const char *src = sk + (size_t)s * (kScanStage * kSixBytes) + wave * (kLoads * 1024);
#pragma unroll
    for (int q = 0; q < kLoads; ++q)
      lds_dma16_at(src, (uint32_t)(q * 1024 + lane * 16),
                   stage_lds + buffer * (kScanStage * kSixBytes) + wave * (kLoads * 1024) + q * 1024);
  };
  const bool asks = kWithBalls && p.asks[w.ut / p.U];
  if (asks) {
    dma(w.I * 2, 0);
    dma(w.I * 2 + 1, 1);
  }
  reinterpret_cast<uint8_t *>(marks)[threadIdx.x] = 0;
  if (threadIdx.x < kScanRun) found[threadIdx.x] = 0;
  if (lane < 4 * kScanWords) need[wave * 4 + lane / kScanWords][lane % kScanWords] = 0;
  static_assert(4 * kScanWords <= kWave, "a lane per word");
  auto tile_at = [&](const char *t) __attribute__((always_inline)) {
    const u4 a = *reinterpret_cast<const u4 *>(t + lane * 16);
    const uint2 b = *reinterpret_cast<const uint2 *>(t + 1024 + lane * 8);
    return i8v{(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)b.x, (int)b.y, 0, 0};
  };
  auto products = [&](const i8v &a, const i8v &b) __attribute__((always_inline)) {
    f16v acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    // (formats 2: six bits, two of them exponent; no block scales)
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 2, 2, 0, 0, 0, 0);
  };
  // largest of a lane's products (as integers: floats order alike as far as it matters)
  auto most = [&](const f16v &acc) __attribute__((always_inline)) {
    int x = __float_as_int(acc[0]);
#pragma unroll
    for (int v = 1; v < 16; ++v) x = max(x, __float_as_int(acc[v]));
    return x;
  };
  // What the integers of results above a threshold exceed: all of them where it isn't positive (no result is -0).
  auto above = [](float thr) __attribute__((always_inline)) { return thr > 0.f ? __float_as_int(thr) : INT32_MIN; };
  auto both_groups = [](unsigned long long m) __attribute__((always_inline)) { return (uint32_t)m | (uint32_t)(m >> 32); };
  i8v bf[4];
  float ethr[4], rnorm[4];                             // theta less the row tile's error; longest sketch
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    bf[r] = tile_at(sk + (size_t)(r0 + r) * kSixBytes);
    ethr[r] = (float)(thr0 - (int)et[r0 + r]) * kUnit;
    rnorm[r] = asks ? norm[r0 + r] : 0.f;
  }
  constexpr int kPerStage = kScanPanel / 4 * kScanStage;   // column tiles, once per wave
  const int own = (w.I + 1) * (kScanPanel / kScanStage);   // first stage behind the panel's own columns
  bool dense = true, refine = false;
  if constexpr (kWithBalls) if (asks) {
  for (int i = threadIdx.x; i < c1 - c0; i += kScanThreads) {
    col_thr[i] = (float)(thr0 - (int)et[c0 + i]) * kUnit;
    col_norm[i] = norm[c0 + i];
  }
  if (threadIdx.x < kScanPanel) row_thr[threadIdx.x] = (float)(thr0 - (int)et[w.I * kScanPanel + threadIdx.x]) * kUnit;

  // ---- the panel's balls: the first of row tile i in column i, seconds from column 16 on
  const int pwin = w.I * kScanPanel / kWave, prow = w.I * kScanPanel % kWave;   // window of the panel, its first tile there
  const float2 *pinfo = p.ball + (windows + pwin) * kBalls;
  int prow_of;                                         // a lane's row tile of the panel, -1: no ball
  float2 pball;
  i8v pc;
  {
    const float e2 = pinfo[2 * kTile + c].x;
    const int row2 = ((int)p.second[(windows + pwin) * kTile + c] & (kWave - 1)) - prow;
    const uint32_t mine = (uint32_t)__ballot(e2 > -0x1p29f && row2 >= 0 && row2 < kScanPanel);   // slots, ascending tiles: a run
    const int slot = mine ? __builtin_ctz(mine) + (c & 15) : 0;
    const bool second = c >= kScanPanel;
    const int at = second ? 2 * kTile + min(slot, kTile - 1) : prow + c;
    pball = pinfo[at];
    const char *t = reinterpret_cast<const char *>(p.skc) + (windows + pwin) * (3 * kSixBytes) + (at >> 5) * kSixBytes;
    const u4 x = *reinterpret_cast<const u4 *>(t + (g * 32 + (at & 31)) * 16);
    const uint2 y = *reinterpret_cast<const uint2 *>(t + 1024 + (g * 32 + (at & 31)) * 8);
    pc = i8v{(int)x[0], (int)x[1], (int)x[2], (int)x[3], (int)y.x, (int)y.y, 0, 0};
    const int of2 = __shfl(row2, min(slot, kTile - 1));
    prow_of = !second ? c : slot < kTile && (mine >> slot & 1) ? of2 : -1;
  }
  const uint32_t loose = (uint32_t)__ballot(lane < kScanPanel && !(pball.y < kBallLoose));   // row tiles (the same in all waves)

  // ---- the panel's tiles against the columns' balls
  for (int win = win0; win <= win1; ++win) {
    const char *ct = reinterpret_cast<const char *>(p.skc) + (windows + win) * (3 * kSixBytes);
    const float2 *info = p.ball + (windows + win) * kBalls;
    const int tw = (int)p.second[(windows + win) * kTile + c] & (kWave - 1);
    i8v b[3];
    float2 f[3];
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      b[part] = tile_at(ct + part * kSixBytes);
      f[part] = info[part * kTile + c];
    }
    if (!__any(f[0].y < kBallLoose || f[1].y < kBallLoose || (f[2].y < kBallLoose && f[2].x > -0x1p29f))) {   // isolated tokens
      if (lane < 8) need[wave * 4 + (lane >> 1)][(win - win0) * 2 + (lane & 1)] = 0xFFFFFFFFu;
      continue;
    }
#pragma unroll
    for (int part = 0; part < 3; ++part) {
      const int first = win * kWave + part * kTile, word = (win - win0) * 2 + part;
      if (part < 2 && (first >= c1 || first + kTile <= c0)) continue;   // block-uniform
      uint32_t hits[4];
#pragma unroll
      for (int r = 0; r < 4; r += 2) {
        const f16v x = products(bf[r], b[part]), y = products(bf[r + 1], b[part]);
        hits[r] = both_groups(__ballot(most(x) > above(ethr[r] - f[part].x - rnorm[r] * f[part].y)));
        hits[r + 1] = both_groups(__ballot(most(y) > above(ethr[r + 1] - f[part].x - rnorm[r + 1] * f[part].y)));
      }
      if (part < 2) {
        if (lane < 4) need[wave * 4 + lane][part < 2 ? word : 0] = lane == 0 ? hits[0] : lane == 1 ? hits[1] : lane == 2 ? hits[2] : hits[3];
      } else if (lane < kTile) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (hits[r] >> c & 1) atomicOr(&need[wave * 4 + r][(win - win0) * 2 + (tw >> 5)], 1u << (tw & 31));
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0): this wave's part of the panel has landed
  __syncthreads();
  // Column tiles that any row tile is left with, in order: tile of the run | a bit per row tile << 16 (every wave the same).
  int nlist = 0, npairs = 0, nloose = 0;               // pairs of tiles; of loose row tiles
#pragma unroll
  for (int half = 0; half < kScanCols; half += kWave) {
    const int t = half + lane, at = c0 + t - win0 * kWave;
    uint32_t rows = 0;
#pragma unroll
    for (int r = 0; r < kScanPanel; ++r) rows |= (need[r][at >> 5] >> (at & 31) & 1u) << r;
    if (t >= c1 - c0) rows = 0;
    const unsigned long long m = __ballot(rows != 0);
    if (rows) list[wave][nlist + __popcll(m & ((1ull << lane) - 1ull))] = (uint32_t)t | rows << 16;
    nlist += __popcll(m);
    npairs += __popc(rows) + (__popc(rows & loose) << 16);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) npairs += __shfl_xor(npairs, o);
  nloose = npairs >> 16;
  npairs &= 0xFFFF;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // What tight row tiles are left with their balls will mostly exclude, unless nothing is excluded at all; so a block is
  // dense by what its loose row tiles are left with.  A pair of its own takes four times what it does among all, yet half
  // of all such pairs is the better line than a quarter of them, since balls of the panel take some of the rest: 64 problems of
  // 32768 tokens, half isolated, 542 us (a third 557, a quarter 558); 16 in drifting clusters with noise 0.3 204 (206, 216).
  dense = __builtin_amdgcn_readfirstlane(2 * nloose > (c1 - c0) * kScanPanel || 5 * npairs > 4 * (c1 - c0) * kScanPanel);

  if (!dense) {
    // Every fourth column tile that is left is the wave's, one per lane: what a step needs of it comes from the lane that
    // has it, and what it finds goes there (as scalars: lists and flags in LDS were a dozen waits per step).
    constexpr int kStep = kScanThreads / kWave;
    const int ncols = nlist > wave ? (nlist - wave + kStep - 1) / kStep : 0;   // at most 32
    const uint32_t e = lane < ncols ? list[wave][wave + kStep * lane] : 0u;
    const float ethr_l = col_thr[e & 127], norm_l = col_norm[e & 127], row_thr_l = row_thr[lane & 15];
    uint32_t hit_l = 0;                                // row tiles that pass with the lane's tile
    i8v a{}, a1{};
    auto fetch = [&](int i) __attribute__((always_inline)) { return tile_at(sk + (size_t)(c0 + (__builtin_amdgcn_readlane(e, min(i, ncols - 1)) & 127)) * kSixBytes); };
    if (ncols > 0) {
      a = fetch(0);
      a1 = fetch(1);
    }
    for (int i = 0; i < ncols; ++i) {
      const i8v a2 = fetch(i + 2);
      const float tthr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ethr_l), i)), tn = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(norm_l), i));
      const float off = tthr - (float)thr0 * kUnit;    // less the column tile's error
      const uint32_t balls = both_groups(__ballot(prow_of >= 0 && most(products(a, pc)) > above(tthr - pball.x - tn * pball.y)));
      uint32_t rows = balls & 0xFFFFu, hit = 0;
      for (uint32_t m = balls >> 16; m; m &= m - 1) rows |= 1u << __builtin_amdgcn_readlane(prow_of, 16 + __builtin_ctz(m));
      rows &= (uint32_t)__builtin_amdgcn_readlane(e, i) >> 16;
      while (rows) {                                   // two row tiles at a time
        const int ra = __builtin_ctz(rows);
        rows &= rows - 1;
        const int rb = rows ? __builtin_ctz(rows) : ra;
        rows &= rows - 1;
        const i8v xa = tile_at(stage + ra * kSixBytes), xb = tile_at(stage + rb * kSixBytes);
        const f16v pa = products(xa, a), pb = products(xb, a);
        const float ta = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(row_thr_l), ra)), tb = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(row_thr_l), rb));
        hit |= (uint32_t)(__ballot(most(pa) > above(ta + off)) != 0) << ra | (uint32_t)(__ballot(most(pb) > above(tb + off)) != 0) << rb;
      }
      hit_l = lane == i ? hit : hit_l;
      a = a1;
      a1 = a2;
    }
    for (; hit_l; hit_l &= hit_l - 1) {
      const int t = (int)(e & 127);
      atomicOr(reinterpret_cast<uint32_t *>(&marks[__builtin_ctz(hit_l)][0]) + (t >> 5), 1u << (t & 31));
    }
    __syncthreads();
    // column tiles marked behind the panel's own, once for four row tiles: lane 16 q + s
    int all = 0;
    {
      const int q = lane >> 4, s = lane & 15;
      if (w.s0 + s >= own && w.s0 + s < w.s1)
        all = __popc((uint32_t)marks[4 * q][s] | marks[4 * q + 1][s] | marks[4 * q + 2][s] | marks[4 * q + 3][s]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) all += __shfl_xor(all, o);
    }
    refine = w.s1 > own && all > (w.s1 - max(own, w.s0)) * (int)(kRefineShare * kPerStage) + kPerStage / 3;
  }
  }
  if (dense) {
    const float emin = fminf(fminf(ethr[0], ethr[1]), fminf(ethr[2], ethr[3]));
    int all = 0;                                       // marks of the stages behind the panel's own
    dma(w.s0, 0);                                      // (no wave reads the panel's tiles)
    for (int s = w.s0;; ++s) {
      const float ecol = s < w.s1 ? (float)et[s * kScanStage + (lane & 7)] * kUnit : 0.f;
      __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): this wave's part of stage s has landed
      __syncthreads();                                 // ... and every wave's; the other buffer is free
      if (s > w.s0 && s > own) {
        all += found[s - 1 - w.s0];
        refine = all > (s - max(own, w.s0)) * (int)(kRefineShare * kPerStage) + kPerStage / 3;
        if (refine) break;
      }
      if (s == w.s1) break;
      if (s + 1 < w.s1) dma(s + 1, (s + 1 - w.s0) & 1);
      const char *st = stage + ((s - w.s0) & 1) * (kScanStage * kSixBytes);
      const int least = above(emin - ecol);            // lane t: of column tile t
      uint32_t hit[4] = {0, 0, 0, 0};
#pragma unroll
      for (int t = 0; t < kScanStage; ++t) {
        const i8v a = tile_at(st + t * kSixBytes);
        int m[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = most(products(a, bf[r]));
        if (__any(max(max(m[0], m[1]), max(m[2], m[3])) > __builtin_amdgcn_readlane(least, t))) {
          const float ec = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(ecol), t));
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (__any(m[r] > above(ethr[r] - ec))) hit[r] |= 1u << t;
        }
      }
      if (hit[0] | hit[1] | hit[2] | hit[3]) {
        if (lane == 0) {
#pragma unroll
          for (int r = 0; r < 4; ++r) marks[wave * 4 + r][s - w.s0] = (uint8_t)hit[r];
          atomicAdd(&found[s - w.s0], __popc(hit[0] | hit[1] | hit[2] | hit[3]));
        }
      }
    }
  }
  if (threadIdx.x == 0) p.todo[blockIdx.x] = refine;
  if (!refine) put_marks<4>(p, w.ut, r0, w.s0, w.s1, marks + wave * 4);
}

// What shallow_scan left over, from the rows themselves (fp32 inputs: from their fp16 unit vectors): a tile pair is marked
// if one of its cosines can be above theta, refine_guard allowed for.  Half of a scan block's panel at a time: two row
// tiles per wave in registers as unit vectors (x 2^10, rounded to the type of the rows), the columns as they are, gathered
// into LDS in their order, 64 at a time, two steps ahead of their use.  A lane has a column and sixteen rows of a tile's
// products: their maximum, times the factor of the column, is tested once, while the matrix cores work on the next tile.
// The blocks stay and deal the work out among them in the scan's order, so that an XCD's blocks share their columns in its L2.
// 16 problems of 32768 fp16 tokens, all pairs: 1.95 ms; with raw rows on both sides, where every product has a factor
// of its own, 2.1; 1.8 from unit vectors on both sides, but these cost shallow_prep 20 us per 16 problems of every
// call, and hardly a call comes here.
constexpr int kRefineThreads = 256;
constexpr int kRefineBlocks = 512;                     // two per compute unit
constexpr int kRefineStages = 3;
constexpr int kRefineList = 2048;                      // items looked at in one go

// Rounding one of the two unit vectors changes a cosine by at most the type's unit roundoff (2^-11, 2^-9); the sums and the
// factors add less than 2e-5.
template <int DT>
__host__ __device__ constexpr float refine_guard() { return DT == SPINDLE_F32 ? kGuard : (DT == SPINDLE_F16 ? 0x1p-11f : 0x1p-9f) + kRowsGuard; }

template <int DT>
__global__ __launch_bounds__(kRefineThreads, 2) void shallow_refine(ShallowParams p, int nitems) {
  typedef Mma<DT == SPINDLE_BF16 ? SPINDLE_BF16 : SPINDLE_F16> M;
  typedef typename Elem<DT>::type T;
  constexpr bool kRaw = DT != SPINDLE_F32;
  __shared__ __attribute__((aligned(1024))) char stage[kRefineStages][kStageBytes];
  __shared__ uint16_t cols[kScanRun * kScanStage * kTile];
  __shared__ float factor[kRaw ? kScanRun * kScanStage * kTile : 1];
  __shared__ unsigned long long odd_s[2];              // column tiles with rows whose products say nothing
  __shared__ uint8_t marks[kScanPanel / 2][kScanRun];
  __shared__ uint16_t list[kRefineList];
  __shared__ int wave_n[kRefineList / kWave];
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5, c = lane & 31;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, nslots = gridDim.x >> 3, n = p.n;
  int soff[M::kSteps];                                 // byte offset of this lane's fragment ks in tile 0 of a stage
#pragma unroll
  for (int ks = 0; ks < M::kSteps; ++ks) soff[ks] = c * 256 + (((2 * ks + g) ^ ((c & 7) | ((c & 16) >> 1))) << 4);
  const uint32_t stage_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)stage;
  for (int i0 = 0; i0 < nitems; i0 += kRefineList) {
    // the items left over, every block the same list: so many per run of 64, then their places
    constexpr int kRuns = kRefineList / kWave / (kRefineThreads / kWave);
    unsigned long long on[kRuns], any = 0;
    if (i0 > 0) __syncthreads();
#pragma unroll
    for (int k = 0; k < kRuns; ++k) {
      const int i = i0 + (k * (kRefineThreads / kWave) + wave) * kWave + lane;
      on[k] = __ballot(i < nitems && p.todo[(size_t)min(i, nitems - 1) * 8 + xcd] != 0);
      if (lane == 0) wave_n[k * (kRefineThreads / kWave) + wave] = __popcll(on[k]);
      any |= on[k];
    }
    if (!__syncthreads_or(any != 0)) continue;         // the ordinary case
    int total = 0;
    for (int q = 0; q < kRefineList / kWave; ++q) {
      const int x = wave_n[q];
      if (q % (kRefineThreads / kWave) == wave) {
        const int k = q / (kRefineThreads / kWave);
        unsigned long long m = 0;
#pragma unroll
        for (int j = 0; j < kRuns; ++j) m = j == k ? on[j] : m;
        if (m >> lane & 1) list[total + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(q * kWave + lane);
      }
      total += x;
    }
    __syncthreads();
    // few items are cut along their columns too, as long as there are blocks without any (one item by two blocks: 30 us)
    int cuts = 1;
    while (cuts < kScanRun / 2 && 4 * cuts * total <= nslots) cuts *= 2;
    for (int at = slot; at < 2 * cuts * total; at += nslots) {
      ScanItem w = scan_item(p, i0 + list[at / (2 * cuts)], xcd);
      const int some = (w.s1 - w.s0 + cuts - 1) / cuts;   // stages
      w.s0 += (at >> 1) % cuts * some;
      w.s1 = min(w.s1, w.s0 + some);
      if (w.s0 >= w.s1) continue;                      // (the same for the block)
      const size_t base = (size_t)w.ut * n;
      const char *X = kRaw ? x_row(p, w.ut, 0) : reinterpret_cast<const char *>(p.Xh) + base * 256;
      const size_t pitch = kRaw ? (size_t)p.lay.st : 256;
      const bool narrow = pitch < 1u << 24 && pitch * n <= 0xFFFFFFFFull;   // (a product of 64 bits is sixteen times the cycles)
      const float *inv = p.invp + base;
      const uint16_t *perm = p.perm + base;
      const uint32_t *et = p.etile + (size_t)w.ut * p.Tp;
      const int r0 = w.I * kScanPanel + (at & 1) * (kScanPanel / 2) + 2 * wave;
      const int tile0 = w.s0 * kScanStage, ntiles = (w.s1 - w.s0) * kScanStage, nsteps = ntiles * kTile / kStageCols;
      const float least = (p.theta[w.ut / p.U] - refine_guard<DT>()) * (kRaw ? kUnitScale : kUnitScale * kUnitScale);
      __syncthreads();                                 // the item before is done with these
      if (threadIdx.x < 2) odd_s[threadIdx.x] = 0;
      __syncthreads();
      for (int i = threadIdx.x; i < ntiles * kTile; i += kRefineThreads) {   // (a wave has two tiles)
        const int pos = min(tile0 * kTile + i, n - 1);
        cols[i] = perm[pos];
        if (kRaw) {
          const float f = inv[pos];
          factor[i] = f == f ? f : 0.f;
          const unsigned long long nan = __ballot(f != f);
          const int t = i >> 5;
          if (c == 0 && (uint32_t)(nan >> (32 * g))) atomicOr(&odd_s[t >> 6], 1ull << (t & 63));
        }
      }
      if (threadIdx.x < sizeof(marks)) reinterpret_cast<uint8_t *>(marks)[threadIdx.x] = 0;
      typename M::frag af[2][M::kSteps];
      bool odd[2];                                     // row tiles with rows whose products say nothing,
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) {
        const int pos = min((r0 + cb) * kTile + c, n - 1);
        const char *row = X + (size_t)perm[pos] * pitch;
#pragma unroll
        for (int ks = 0; ks < M::kSteps; ++ks) af[cb][ks] = M::load(row, ks, g);
        odd[cb] = et[r0 + cb] >= kSketchUnknown;
        if constexpr (kRaw) {
          const float f = inv[pos], scale = f * kUnitScale;
          odd[cb] |= __any(f != f) != 0;
#pragma unroll
          for (int ks = 0; ks < M::kSteps; ++ks) {
            u4 x = __builtin_bit_cast(u4, af[cb][ks]);
            T *e = reinterpret_cast<T *>(&x);
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = Elem<DT>::from_float(Elem<DT>::to_float(e[j]) * scale);
            af[cb][ks] = __builtin_bit_cast(typename M::frag, x);
          }
        }
      }
      unsigned long long odd_cols[2];                  // ... and columns, a bit per tile
#pragma unroll
      for (int k = 0; k < 2; ++k)
        odd_cols[k] = __ballot(k * kWave + lane < ntiles && et[tile0 + min(k * kWave + lane, ntiles - 1)] >= kSketchUnknown);
      __syncthreads();
#pragma unroll
      for (int k = 0; k < 2; ++k) odd_cols[k] |= odd_s[k];
      auto dma = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int r = (wave * 4 + q) * 4 + (lane >> 4);
          const uint32_t tok = cols[s * kStageCols + r], piece = (((lane & 15) ^ ((r & 7) | ((r & 16) >> 1))) << 4);
          const uint32_t to = stage_lds + (s % kRefineStages) * kStageBytes + (wave * 4 + q) * 1024;
          if (narrow) lds_dma16_at(X, __umul24(tok, (uint32_t)pitch) + piece, to);
          else lds_dma16(X + tok * pitch + piece, to);
        }
      };
      // results of column tile t; `least` is positive: floats order as integers as far as it matters
      auto look = [&](int t, const f16v &x0, const f16v &x1) __attribute__((always_inline)) {
        const float f = kRaw ? factor[t * kTile + c] : 1.f;
        int m0 = __float_as_int(x0[0]), m1 = __float_as_int(x1[0]);
#pragma unroll
        for (int v = 1; v < 16; ++v) { m0 = max(m0, __float_as_int(x0[v])); m1 = max(m1, __float_as_int(x1[v])); }
        const bool oddc = odd_cols[t >> 6] >> (t & 63) & 1;
        const bool hit0 = oddc | odd[0] | (__any(__int_as_float(m0) * f > least) != 0);
        const bool hit1 = oddc | odd[1] | (__any(__int_as_float(m1) * f > least) != 0);
        if ((hit0 | hit1) && lane < 2 && (lane ? hit1 : hit0)) marks[2 * wave + lane][t >> 3] |= (uint8_t)(1u << (t & 7));
      };
      f16v y0, y1;
#pragma unroll
      for (int v = 0; v < 16; ++v) { y0[v] = 0.f; y1[v] = 0.f; }   // (below `least`)
      dma(0);
      dma(1);                                          // (a stage of the scan is four steps)
      for (int s = 0; s < nsteps; ++s) {
        // the wave's loads of step s have landed (those of step s + 1 may be on their way), and behind the barrier
        // every wave's; the buffer of step s - 1 is free
        if (s + 1 < nsteps) __builtin_amdgcn_s_waitcnt(0x0F74);
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        __syncthreads();
        if (s + 2 < nsteps) dma(s + 2);
        const char *st = stage[s % kRefineStages];
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
          f16v x0, x1;
#pragma unroll
          for (int v = 0; v < 16; ++v) { x0[v] = 0.f; x1[v] = 0.f; }
          typename M::frag f[M::kSteps];
#pragma unroll
          for (int ks = 0; ks < M::kSteps; ++ks) f[ks] = *reinterpret_cast<const typename M::frag *>(st + ct * kTile * 256 + soff[ks]);
          __builtin_amdgcn_sched_barrier(0);           // all reads on their way before the first instruction waits
#pragma unroll
          for (int ks = 0; ks < M::kSteps; ++ks) {
            x0 = M::mma(af[0][ks], f[ks], x0);
            x1 = M::mma(af[1][ks], f[ks], x1);
          }
          if (ct > 0 || s > 0) look(2 * s + ct - 1, y0, y1);
          y0 = x0;
          y1 = x1;
        }
      }
      look(2 * nsteps - 1, y0, y1);
      put_marks<2>(p, w.ut, r0, w.s0, w.s1, marks + 2 * wave);
    }
  }
}

// ---------------------------------------------------------------- rows
// Cosines of the marked tile pairs, neighbour words and degrees.
// fp16 and bf16: the products are taken on the raw rows (exact products, fp32 sums), whose error is
// that of the sums alone; fp32: on the fp16 unit vectors and their remainders, x_h y_h + 2^-11 (x_h y_l +
// x_l y_h), which leaves out 2^-22 of the cosine.  With f_a the factor of a row (1 / m_a, or 1 / 1024 for
// the unit vectors) the decision S_ab > theta is the sign of dot * f_b - theta / f_a.  The sums are good
// to 2e-5 (128 terms, even with truncation); a result within kRowsGuard / f_a of zero is decided in
// double precision as the definition says (the pairs wait in LDS for a wave's worth of them).
//
// A block takes 4 / kCols neighbouring row tiles and walks over the column tiles that any of them is
// marked for, kCols at a time: their rows are gathered straight into LDS, ahead of their
// use, and every wave multiplies one of them with one row tile (held in registers).  kCols = 1: what
// similar rows have in common is read once for four row tiles; kCols = 4: short problems, where there
// are too few row tiles to fill the chip.  Bound by latency (half of a block's 18 us is its lists and first rows, the rest
// gathered rows, mostly from L2, products and tests), so what counts is blocks per compute unit: LDS and registers
// allow four with two stages and 28 steps' bits, where three stages and 32 steps allowed three.  16 problems of 32768 tokens
// 173 -> 146 us, 128 of 8192 in clusters of 128 200 -> 168, 64 of 32768 with half isolated 379 -> 315.
constexpr int kRowsThreads = 256;
constexpr int kRowsPitch = kWave + 2;              // result bits of a step, and a word so that one lane's bits of 32 steps are 32 banks

// kShort: problems whose list of tiles is short enough (kShortTiles) that four blocks fit with 32 steps and fewer waiting pairs,
// too.  Where tokens are not sorted every block takes all tiles; where they are, the few blocks that take the most end last.  The
// kernel on 32 problems of 1000 tokens 49 us with 28 steps, 38 so, on 128 74 and 66, on 16 of 2060 in seven clusters 45 and 31.
constexpr int kShortTiles = 120;
constexpr size_t kLdsBytes = 160 * 1024;           // of a compute unit

template <int DT, int kCols, bool kShort>
struct RowsLds {
  static constexpr int kQueue = kShort ? 160 : 192;                      // waiting pairs per wave
  static constexpr int kPart = kTile * 256;                              // 32 rows of 128 two-byte elements
  static constexpr int kStage = kCols * kPart * (DT == SPINDLE_F32 ? 2 : 1);
  static constexpr int kStages = kCols == 1 && DT == SPINDLE_F32 ? 3 : 2;
  static constexpr int kBatch = kCols > 1 ? 16 : DT == SPINDLE_F32 || kShort ? 32 : 28;   // steps whose result bits a wave keeps
  char stage[kStages][kStage];
  float inv[kBatch * kCols][kTile];
  uint16_t tok[kBatch * kCols][kTile];
  uint16_t bits[4][kBatch * kRowsPitch];
  __attribute__((aligned(4))) uint16_t queue[4][kQueue];                                         // at the end: degree << 16 | words of every lane
  int ntiles;
  __device__ uint16_t *tiles() { return reinterpret_cast<uint16_t *>(this + 1); }  // [T] column tile | 1 << (11 + row tile of the block)
  static constexpr size_t bytes(int T) { return sizeof(RowsLds) + ((size_t)T * sizeof(uint16_t) + 15) / 16 * 16; }
};

// A wave's rows r0 .. r0 + nr - 1 of row tile R from the bits in memory (word t of a row's room: column tile t, written for the
// tiles of the list): counted, and turned into words in place.  A row is in registers before any of
// it is overwritten, kRows rows at a time for the latency of the reads: a block that has one tile more than a batch holds is the last
// to end, 20 us with four at a time, 12 with sixteen (the call on 4 problems of 23000 tokens 203 us and 196).  16 problems of
// 32768 similar tokens: 9.9 ms for the kernel, 19.6 where cosines were taken again to write words whose number was known by then.
template <int kRows, int kWords>
__device__ __forceinline__ void rows_from_memory(const ShallowParams &p, int ut, int R, int r0, int nr, int rows_here,
                                                 const uint16_t *tiles, int ntiles) {
  const int lane = lane_id(), n = p.n, T = p.T, pitch = p.list_row;
  const size_t base = (size_t)ut * n;
  uint32_t *lists = p.lists + base * pitch + (size_t)R * kTile * pitch;
  const unsigned long long below = (1ull << lane) - 1ull;
  int deg = 0;                                         // lane i: those of row r0 + i
  uint32_t words = 0;
  const int r1 = min(r0 + nr, rows_here);
  for (int r = r0; r < r1; r += kRows) {
    uint32_t w[kRows][kWords];
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      const int i = k * kWave + lane;
      if (k * kWave < ntiles) {                        // wave-uniform, as below
        const int t = (int)(tiles[min(i, ntiles - 1)] & 2047u);
#pragma unroll
        for (int j = 0; j < kRows; ++j) w[j][k] = i < ntiles && r + j < r1 ? lists[(size_t)(r + j) * pitch + t] : 0u;
      } else {
#pragma unroll
        for (int j = 0; j < kRows; ++j) w[j][k] = 0u;
      }
    }
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
      if (r + j >= r1) continue;
      int d = 0, total = 0;
#pragma unroll
      for (int k = 0; k < kWords; ++k)
        if (k * kWave < ntiles) {
          d += __popc(w[j][k]);
          total += __popcll(__ballot((w[j][k] & 0xFFFFu) != 0)) + __popcll(__ballot(w[j][k] >> 16 != 0));
        }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o);
      const bool dense = total > pitch;
      if (lane == r + j - r0) {
        deg = d;
        words = dense ? kDenseRow | (uint32_t)(2 * T) : (uint32_t)total;
      }
      uint32_t *out = lists + (size_t)(r + j) * pitch;
      if (dense) {
        if (ntiles == T) continue;                     // every tile has its word already
        for (int t = lane; t < T; t += kWave) out[t] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // before the bits of the marked ones are written
#pragma unroll
        for (int k = 0; k < kWords; ++k)
          if (k * kWave + lane < ntiles) out[tiles[k * kWave + lane] & 2047u] = w[j][k];
        continue;
      }
      int at = 0;
#pragma unroll
      for (int k = 0; k < kWords; ++k)
        if (k * kWave < ntiles) {
          const uint32_t lo = w[j][k] & 0xFFFFu, hi = w[j][k] >> 16;
          const unsigned long long mlo = __ballot(lo != 0), mhi = __ballot(hi != 0);
          if (w[j][k]) {
            const uint32_t half = 2u * (tiles[k * kWave + lane] & 2047u);
            uint32_t *o = out + at + __popcll(mlo & below) + __popcll(mhi & below);
            if (lo) *o++ = half << 16 | lo;
            if (hi) *o = (half + 1) << 16 | hi;
          }
          at += __popcll(mlo) + __popcll(mhi);
        }
    }
  }
  if (lane < r1 - r0) {
    const int row = R * kTile + r0 + lane, tok = (int)p.perm[base + row];
    p.key[(size_t)ut * p.n32 + row] = ((uint32_t)deg << 16) | (uint32_t)(0xFFFF - tok);
    p.rows[base + row] = make_uint2((uint32_t)row * pitch, words);
    if (p.deg_out[ut / p.U]) p.deg_out[ut / p.U][(size_t)(ut % p.U) * n + tok] = deg;
  }
}

template <int DT, int kCols, bool kShort>
__global__ __launch_bounds__(kRowsThreads, kCols == 1 && DT != SPINDLE_F32 ? 4 : 2) void shallow_rows(ShallowParams p, int nblk) {
  typedef Mma<DT == SPINDLE_BF16 ? SPINDLE_BF16 : SPINDLE_F16> M;
  typedef RowsLds<DT, kCols, kShort> L;
  constexpr bool kSplit = DT == SPINDLE_F32;
  constexpr int kRT = 4 / kCols;                       // row tiles of the block
  extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
  L &l = *reinterpret_cast<L *>(lds_raw);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id(), g = lane >> 5, c = lane & 31;
  const int tid = threadIdx.x, member = wave % kCols, rt = wave / kCols;
  const int item = xcd_item();
  if (item >= p.UT * nblk) return;
  const int ut = item / nblk, n = p.n, T = p.T, R0 = (item % nblk) * kRT, R = R0 + rt;
  const bool mine = R < T;                             // (the last block's last row tiles may not exist)
  const size_t base = (size_t)ut * n;
  uint16_t *bits = l.bits[wave], *queue = l.queue[wave], *tiles = l.tiles();
  const uint16_t *perm = p.perm + base;
  const float *inv = p.invp + base;
  const float theta = p.theta[ut / p.U];

  const char *X, *Xlo = nullptr;
  size_t row_bytes;
  if (kSplit) {
    X = reinterpret_cast<const char *>(p.Xh) + base * 256;
    Xlo = reinterpret_cast<const char *>(p.Xl) + base * 256;
    row_bytes = 256;
  } else {
    X = x_row(p, ut, 0);
    row_bytes = (size_t)p.lay.st;
  }
  // column tiles any row tile of the block is marked for, each with the row tiles it is for
  if (wave == 0) {
    if (p.by[ut / p.U] != kByNone) {
      uint32_t word[kRT], any = 0;                     // lane w: word w of the rows of tpairs
#pragma unroll
      for (int k = 0; k < kRT; ++k) {
        word[k] = 0;
        if (R0 + k < T && lane < p.TW) word[k] = p.tpairs[((size_t)ut * T + R0 + k) * p.TW + lane];
        if (R0 + k < T && lane == (R0 + k) >> 5) word[k] |= 1u << ((R0 + k) & 31);   // G_aa = 1 whatever theta is
        any |= word[k];
      }
      int at = __popc(any);
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const int x = __shfl_up(at, o);
        if (lane >= o) at += x;
      }
      if (lane == kWave - 1) l.ntiles = at;
      at -= __popc(any);
      for (; any; any &= any - 1) {
        const int t = __builtin_ctz(any);
        uint32_t e = (uint32_t)(lane * 32 + t);
#pragma unroll
        for (int k = 0; k < kRT; ++k) e |= (word[k] >> t & 1u) << (11 + k);
        tiles[at++] = (uint16_t)e;
      }
    } else {
      for (int t = lane; t < T; t += kWave) tiles[t] = (uint16_t)(t | ((1 << kRT) - 1) << 11);
      if (lane == 0) l.ntiles = T;
    }
  }
  // the wave's rows: matrix columns = lanes
  const int row = R * kTile + c;
  const bool row_on = row < n;
  const int row_tok = (int)perm[row_on ? row : n - 1];
  typename M::frag bf[M::kSteps], bl[kSplit ? M::kSteps : 1];
  {
    const size_t at = (size_t)row_tok * row_bytes;
#pragma unroll
    for (int ks = 0; ks < M::kSteps; ++ks) {
      bf[ks] = M::load(X + at, ks, g);
      if (kSplit) bl[kSplit ? ks : 0] = M::load(Xlo + at, ks, g);
    }
  }
  const float frow = inv[row_on ? row : n - 1];
  const bool odd_row = frow != frow;                   // every pair of it is decided in double precision
  // zero vectors: cosine 0, as if theta / f_a were huge (and of the sign of theta)
  const float mrow = odd_row ? 1.f : frow > 0.f ? 1.f / frow : 0x1p100f;
  const float lim = frow == 0.f && theta == 0.f ? 1.f : theta * mrow;
  const float band = frow > 0.f ? kRowsGuard * mrow : 0.f;
  const bool any_odd_row = __any(odd_row);

  // Rows of a staged tile keep their 16-byte piece k at place k ^ swz(row), so that sixteen consecutive
  // lanes of a 128-bit read hit sixteen different bank groups.  The token at place 16 g + v feeds matrix
  // row 8 (v / 4) + 4 g + v % 4, so that result v of lane group g is column 16 g + v.
  const int prow = 16 * ((c >> 2) & 1) + 4 * (c >> 3) + (c & 3);
  auto swz = [](int r) { return (r & 7) | ((r & 16) >> 1); };
  int soff[M::kSteps];
#pragma unroll
  for (int ks = 0; ks < M::kSteps; ++ks) soff[ks] = prow * 256 + (((2 * ks + g) ^ swz(prow)) << 4);
  const uint32_t stage_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)lds_raw;
  __syncthreads();
  const int ntiles = __builtin_amdgcn_readfirstlane(l.ntiles);
  const int nall = (ntiles + kCols - 1) / kCols;       // steps

  // Bits of more steps than a batch holds go to the rows' room in the lists, word t for column tile t, and
  // from there into words at the end.
  const int nbatch = (nall + L::kBatch - 1) / L::kBatch;
  const int rows_here = mine ? min(kTile, n - R * kTile) : 0;
  uint32_t *lists = p.lists + base * p.list_row;
  int nq = 0, ndecided = 0;
  for (int batch = 0; batch < nbatch; ++batch) {
    const int s0 = batch * L::kBatch, ns = min(L::kBatch, nall - s0);
    const int t0 = s0 * kCols, nt = min(L::kBatch * kCols, ntiles - t0);
    if (batch > 0) __syncthreads();                    // the batch before is done with these
    for (int i = tid; i < nt * kTile; i += kRowsThreads) {
      const int col = (int)(tiles[t0 + (i >> 5)] & 2047u) * kTile + (i & 31);
      l.tok[i >> 5][i & 31] = perm[col < n ? col : n - 1];
      l.inv[i >> 5][i & 31] = col < n ? inv[col] : 0.f;
    }
    __syncthreads();
    // loads of step s: the wave brings in 8 rows of every tile, four rows of 256 bytes per load
    auto fetch = [&](int s) __attribute__((always_inline)) {
#pragma unroll
      for (int k = 0; k < kCols; ++k) {
        const int i = min(s * kCols + k, nt - 1);      // (a last step may have fewer tiles)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int r = wave * 8 + q * 4 + (lane >> 4);
          const size_t at = (size_t)l.tok[i][r] * row_bytes + (size_t)(((lane & 15) ^ swz(r)) << 4);
          const uint32_t to = stage_lds + (uint32_t)((s % L::kStages) * L::kStage + k * L::kPart + (wave * 8 + q * 4) * 256);
          lds_dma16(X + at, to);
          if (kSplit) lds_dma16(Xlo + at, to + kCols * L::kPart);
        }
      }
    };
    fetch(0);
    if (L::kStages > 2 && ns > 1) fetch(1);
    for (int s = 0; s < ns; ++s) {
      // the wave's loads of step s have landed (those of step s + 1 may still be on their way), and behind
      // the barrier every wave's; the buffer of step s - 1 is free
      if (L::kStages > 2 && s + 1 < ns) __builtin_amdgcn_s_waitcnt(kSplit ? 0x0F74 : 0x0F72);
      else __builtin_amdgcn_s_waitcnt(0x0F70);
      __syncthreads();
      if (s + L::kStages - 1 < ns) fetch(s + L::kStages - 1);
      const int i = s * kCols + member;                // this wave's tile of the batch
      const uint32_t entry = i < nt ? (uint32_t)__builtin_amdgcn_readfirstlane((int)tiles[t0 + i]) : 0u;
      if (!(entry >> (11 + rt) & 1u)) {                // wave-uniform
        bits[s * kRowsPitch + lane] = 0;
        continue;
      }
      const int t = (int)(entry & 2047u);
      const char *st = l.stage[s % L::kStages] + member * L::kPart;
      f16v acc, lo;
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc[v] = 0.f; lo[v] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < M::kSteps; ++ks) {
        const typename M::frag f = *reinterpret_cast<const typename M::frag *>(st + soff[ks]);
        acc = M::mma(f, bf[ks], acc);
        if (kSplit) {
          const typename M::frag fl = *reinterpret_cast<const typename M::frag *>(st + kCols * L::kPart + soff[ks]);
          lo = M::mma(f, bl[kSplit ? ks : 0], lo);
          lo = M::mma(fl, bf[ks], lo);
        }
      }
      const float *fc = l.inv[i];
      const bool odd = any_odd_row || __any(fc[c] != fc[c]);
      uint32_t neg = 0;
      float mn = INFINITY;
      float x[16];
#pragma unroll
      for (int v = 15; v >= 0; --v) {
        const float d = kSplit ? fmaf(lo[v], 0x1p-11f, acc[v]) : acc[v];
        x[v] = fmaf(d, fc[16 * g + v], -lim);
        neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(x[v]), 31);
        mn = fminf(mn, fabsf(x[v]));
      }
      uint32_t yes = ~neg & 0xFFFFu;
      uint32_t valid = row_on ? 0xFFFFu : 0u;
      const int nv = n - t * kTile - 16 * g;           // columns past the end
      if (nv < 16) valid = nv <= 0 ? 0u : valid & ((1u << nv) - 1u);
      yes &= valid;
      const bool self = t == R && (c >> 4) == g;
      uint32_t close = 0;
      if (odd || __any(mn < band)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float fv = fc[16 * g + v];
          if (odd_row || fv != fv || fabsf(x[v]) < band) close |= 1u << v;
        }
        close &= valid;
        if (self) close &= ~(1u << (c & 15));
        yes &= ~close;
      }
      if (self && row_on) yes |= 1u << (c & 15);       // G_aa = 1
      bits[s * kRowsPitch + lane] = (uint16_t)yes;
      for (;;) {                                       // one close pair per lane at a time into the queue
        const unsigned long long m = __ballot(close != 0);
        if (nq > L::kQueue - kWave || (m == 0 && nq > 0 && s + 1 == ns)) {
          // (the bits are written as halves elsewhere and as words here: keep the compiler from reordering them)
          asm volatile("" ::: "memory");
          for (int j = lane; j < nq; j += kWave) {
            const uint32_t e = queue[j];
            const int slot = (int)(e >> 10), ln = (int)((e >> 4) & 63), v = (int)(e & 15);
            const int a = (int)perm[R * kTile + (ln & 31)], b = (int)l.tok[slot * kCols + member][16 * (ln >> 5) + v];
            ++ndecided;
            if (cos64<DT, 4>(p, ut, a, b) > (double)theta) {
              const int at = slot * kRowsPitch + ln;
              atomicOr(reinterpret_cast<uint32_t *>(bits) + (at >> 1), 1u << (v + 16 * (at & 1)));
            }
          }
          nq = 0;
          asm volatile("" ::: "memory");
        }
        if (m == 0) break;
        if (close) {
          const int v = __builtin_ctz(close);
          close &= close - 1;
          queue[nq + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)(s << 10 | lane << 4 | v);
        }
        nq += __popcll(m);
      }
    }
    // (the last step may not have been this wave's: pairs still waiting)
    if (nq > 0) {
      asm volatile("" ::: "memory");
      for (int j = lane; j < nq; j += kWave) {
        const uint32_t e = queue[j];
        const int slot = (int)(e >> 10), ln = (int)((e >> 4) & 63), v = (int)(e & 15);
        const int a = (int)perm[R * kTile + (ln & 31)], b = (int)l.tok[slot * kCols + member][16 * (ln >> 5) + v];
        ++ndecided;
        if (cos64<DT, 8>(p, ut, a, b) > (double)theta) {
          const int at = slot * kRowsPitch + ln;
          atomicOr(reinterpret_cast<uint32_t *>(bits) + (at >> 1), 1u << (v + 16 * (at & 1)));
        }
      }
      nq = 0;
      asm volatile("" ::: "memory");
    }
    if (nbatch == 1) break;
    constexpr int kRowsAtOnce = kWave / L::kBatch;     // lanes along the steps: runs of neighbouring tiles are runs of memory
    const int ls = lane % L::kBatch, li = ls * kCols + member;
    if (ls < ns && li < nt && lane < kRowsAtOnce * L::kBatch) {
      const int t = (int)(tiles[t0 + li] & 2047u);
      for (int r = lane / L::kBatch; r < rows_here; r += kRowsAtOnce)
        lists[(size_t)(R * kTile + r) * p.list_row + t] =
            (uint32_t)bits[ls * kRowsPitch + r] | (uint32_t)bits[ls * kRowsPitch + 32 + r] << 16;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ndecided += __shfl_xor(ndecided, o);
  // (A place for every wave: sums of a problem's waves in one word each put 16384 additions into one cache line that all
  // dies ask for, and the kernel waited: 268 us for 16 problems of 32768 fp16 tokens, 221 now.)
  if (lane == 0 && mine) p.pairs_exact[((size_t)ut * T + R) * kCols + member] = (unsigned)ndecided;
  if (lane == 0 && member == 0 && mine) {
    const uint32_t ones = rows_here == kTile ? 0xFFFFFFFFu : (1u << rows_here) - 1u;
    p.live[0][(size_t)ut * T + R] = ones;
    p.live[1][(size_t)ut * T + R] = ones;
    p.live[2][(size_t)ut * T + R] = ones;
  }
  if (nbatch > 1) {
    __syncthreads();                                   // (and the words in memory are every wave's to read)
    if (kCols == 1 && ntiles <= kWave) rows_from_memory<16, 1>(p, ut, R, member * (kTile / kCols), kTile / kCols, rows_here, tiles, ntiles);
    else if (ntiles <= 8 * kWave) rows_from_memory<4, 8>(p, ut, R, member * (kTile / kCols), kTile / kCols, rows_here, tiles, ntiles);
    else rows_from_memory<1, 32>(p, ut, R, member * (kTile / kCols), kTile / kCols, rows_here, tiles, ntiles);
    return;
  }
  int deg = 0, words = 0;
  for (int s = 0; s < nall; ++s) {
    const uint32_t m = bits[s * kRowsPitch + lane];
    deg += __popc(m);
    words += m != 0;
  }
  static_assert(L::kQueue * sizeof(uint16_t) >= kWave * sizeof(uint32_t), "the counts take the queue's place");
  auto counts = [&](int w) { return reinterpret_cast<uint32_t *>(l.queue[w]); };
  asm volatile("" ::: "memory");                       // (read as halves before)
  counts(wave)[lane] = (uint32_t)deg << 16 | (uint32_t)words;
  __syncthreads();
  // a row's words: those of lane group 0 of every wave of its row tile, then those of group 1
  int total = 0, d = 0, at = 0;
#pragma unroll
  for (int q = 0; q < kCols; ++q) {
    const int w = rt * kCols + q;
    const uint32_t n0 = counts(w)[c], n1 = counts(w)[32 + c];
    const int x0 = (int)(n0 & 0xFFFFu), x1 = (int)(n1 & 0xFFFFu);
    d += (int)(n0 >> 16) + (int)(n1 >> 16);
    total += x0 + x1;
    at += g == 0 ? (q < member ? x0 : 0) : x0 + (q < member ? x1 : 0);
  }
  int incl = total;                                    // over the 32 rows (the same in both lane groups)
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    const int y = __shfl_up(incl, o, 32);
    if (c >= o) incl += y;
  }
  const bool dense = __builtin_amdgcn_readlane(incl, 31) > rows_here * p.list_row;
  const uint32_t first = dense ? (uint32_t)row * p.list_row : (uint32_t)(R * kTile * p.list_row + incl - total);
  if (g == 0 && row_on && member == 0) {
    p.key[(size_t)ut * p.n32 + row] = ((uint32_t)d << 16) | (uint32_t)(0xFFFF - row_tok);
    p.rows[base + row] = make_uint2(first, dense ? kDenseRow | (uint32_t)(2 * T) : (uint32_t)total);
    if (p.deg_out[ut / p.U]) p.deg_out[ut / p.U][(size_t)(ut % p.U) * n + row_tok] = d;
  }
  uint32_t *out = lists + first + (dense ? 0 : at);
  if (dense && p.scan && member == 0) {                // tiles that were not marked: no bits
    for (int i = lane; i < rows_here * p.list_row; i += kWave) lists[(size_t)R * kTile * p.list_row + i] = 0;
    __builtin_amdgcn_s_waitcnt(0x0F70);                // before the bits of the marked ones are written
  }
  __syncthreads();
  for (int s = 0; s < nall; ++s) {
    const int i = s * kCols + member;
    if (i >= ntiles) break;
    const uint32_t m = bits[s * kRowsPitch + lane], half = 2u * (tiles[i] & 2047u) + g;
    if (dense) {
      if (row_on) reinterpret_cast<uint16_t *>(out)[half] = (uint16_t)m;
    } else if (m) {
      *out++ = half << 16 | m;
    }
  }
}

// ---------------------------------------------------------------- adjacency export
// One wave per row: its words, from positions to tokens, collected as bits in LDS.
__global__ __launch_bounds__(256) void shallow_adjacency(ShallowParams p, uint32_t *out, int t) {
  __shared__ uint32_t acc[4][65536 / 32];
  const int wave = threadIdx.x >> 6, lane = lane_id(), n = p.n, W = (n + 31) / 32;
  const size_t nrows = (size_t)p.U * n;
  for (size_t i0 = (size_t)blockIdx.x * 4; i0 < nrows; i0 += (size_t)gridDim.x * 4) {
    const size_t i = i0 + wave;
    if (i < nrows)
      for (int k = lane; k < W; k += kWave) acc[wave][k] = 0;
    __syncthreads();
    const size_t base = (size_t)(t * p.U) * n + i / n * n;
    int row = 0;
    if (i < nrows) {
      const int v = (int)(i % n);
      const uint2 info = p.rows[base + v];
      const uint32_t *w = p.lists + base * p.list_row + info.x;
      const bool dense = (info.y & kDenseRow) != 0;
      const int nw = (int)(info.y & ~kDenseRow);
      row = (int)p.perm[base + v];
      for (int k = lane; k < nw; k += kWave) {
        const uint32_t x = dense ? (uint32_t)k << 16 | reinterpret_cast<const uint16_t *>(w)[k] : w[k];
        for (uint32_t m = x & 0xFFFFu; m; m &= m - 1) {
          const int b = (int)p.perm[base + (x >> 16) * 16 + __builtin_ctz(m)];
          atomicOr(&acc[wave][b >> 5], 1u << (b & 31));
        }
      }
    }
    __syncthreads();
    if (i < nrows)
      for (int k = lane; k < W; k += kWave) out[(i / n * n + row) * W + k] = acc[wave][k];
    __syncthreads();
  }
}

}  // namespace

namespace {
// How the tile pairs that count are found; of K and V the one that is looked at first.
int most_by(const ShallowParams &p) { return p.UT > p.U && p.by[1] > p.by[0] ? p.by[1] : p.by[0]; }

template <int DT, int kCols, bool kShort>
spindle_status launch_rows(const ShallowParams &p, hipStream_t st) {
  typedef RowsLds<DT, kCols, kShort> L;
  constexpr int kRT = 4 / kCols;
  static LdsLimit lim;
  if (spindle_status e = allow_lds(lim, reinterpret_cast<const void *>(&shallow_rows<DT, kCols, kShort>), L::bytes(2048))) return e;
  const int nblk = (p.T + kRT - 1) / kRT;
  const size_t lds = L::bytes(p.T);
  ProfScope ps("shallow_rows", st, most_by(p) == kByNone);
  hipLaunchKernelGGL((shallow_rows<DT, kCols, kShort>), dim3(xcd_grid((size_t)p.UT * nblk)), dim3(kRowsThreads), lds,
                     st, p, nblk);
  return SPINDLE_OK;
}
template <int DT>
spindle_status launch_rows(const ShallowParams &p, hipStream_t st) {
  if (rows_waves(p.UT, p.T) == 4) return launch_rows<DT, 4, false>(p, st);
  if constexpr (DT != SPINDLE_F32) {
    static_assert(RowsLds<DT, 1, true>::bytes(kShortTiles) <= kLdsBytes / 4, "four blocks");
    if (p.T > RowsLds<DT, 1, false>::kBatch && p.T <= kShortTiles) return launch_rows<DT, 1, true>(p, st);
  }
  return launch_rows<DT, 1, false>(p, st);
}
}  // namespace

spindle_status launch_tiles(const ShallowParams &p, hipStream_t st) {
  const int n = p.n;
  if (p.scan) {
    // 1024 tokens per block where that leaves a block for every place on the chip (two per compute unit): what a block does
    // before and after its products takes 14 of 30 us with 512 tokens.
    const int per = (long)p.UT * ((n + 2 * kOrderTokens - 1) / (2 * kOrderTokens)) >= 512 ? 2 * kOrderTokens : kOrderTokens;
    const int nblk = (n + per - 1) / per, nwin = 2 * ((n + 2 * kWindow - 1) / (2 * kWindow));
    int npiv = (n / 16) & ~31;
    if (npiv > kPivots) npiv = kPivots;
    { ProfScope ps("shallow_pivots", st);
    const dim3 pg(xcd_grid((size_t)p.UT * nblk));
    if (per == kOrderTokens) hipLaunchKernelGGL(shallow_pivots<4>, pg, dim3(kPivotThreads), 0, st, p, npiv, nblk);
    else hipLaunchKernelGGL(shallow_pivots<8>, pg, dim3(kPivotThreads), 0, st, p, npiv, nblk); }
    { ProfScope ps("shallow_order", st);
    hipLaunchKernelGGL(shallow_order, dim3(xcd_grid((size_t)p.UT * nblk)), dim3(kOrderThreads), 0, st, p, nblk, per); }
    { ProfScope ps("shallow_window", st);
    hipLaunchKernelGGL(shallow_window, dim3(xcd_grid((size_t)p.UT * nwin)), dim3(kWindowThreads), 0, st, p, nwin); }
    const int nitems = scan_blocks(p) / 8;
    { ProfScope ps("shallow_scan", st, most_by(p) == kBySketch);
    if (p.balls) hipLaunchKernelGGL(shallow_scan<true>, dim3((unsigned)(8 * nitems)), dim3(kScanThreads), 0, st, p);
    else hipLaunchKernelGGL(shallow_scan<false>, dim3((unsigned)(8 * nitems)), dim3(kScanThreads), 0, st, p); }
    { ProfScope ps("shallow_refine", st, most_by(p) == kByVector);
    if (p.dtype == SPINDLE_F16) hipLaunchKernelGGL(shallow_refine<SPINDLE_F16>, dim3(kRefineBlocks), dim3(kRefineThreads), 0, st, p, nitems);
    else if (p.dtype == SPINDLE_BF16) hipLaunchKernelGGL(shallow_refine<SPINDLE_BF16>, dim3(kRefineBlocks), dim3(kRefineThreads), 0, st, p, nitems);
    else hipLaunchKernelGGL(shallow_refine<SPINDLE_F32>, dim3(kRefineBlocks), dim3(kRefineThreads), 0, st, p, nitems); }
  }
  if (p.dtype == SPINDLE_F16) return launch_rows<SPINDLE_F16>(p, st);
  if (p.dtype == SPINDLE_BF16) return launch_rows<SPINDLE_BF16>(p, st);
  return launch_rows<SPINDLE_F32>(p, st);
}

spindle_status launch_adjacency(const ShallowParams &p, uint32_t *const out[2], hipStream_t st) {
  for (int t = 0; t < p.UT / p.U; ++t)
    if (out[t]) hipLaunchKernelGGL(shallow_adjacency, dim3(2048), dim3(256), 0, st, p, out[t], t);
  return SPINDLE_OK;
}

}  // namespace spindle
