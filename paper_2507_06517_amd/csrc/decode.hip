// Decode-time merge (Sec. "Similarity Based Token Replacement", the paragraph after Eq. 14):
// tokens generated after the prefill first look for a stored codebook entry within theta;
// those that find none get entries of their own by the construction of Alg. 1, appended to
// the codebook.
//
// Kernels, enqueued on the caller's stream; u indexes one (batch, kv-head) problem of m new tokens:
//   decode_match   per new token and slice of 512 stored entries, the entry of highest cosine
//                  (Eq. 4) if it exceeds theta, lowest index on ties: matrix-core cosines leave
//                  the few entries that can be it, those are decided in double precision with
//                  the dimension-order sums the adjacency decision is defined by
//   decode_build   one workgroup per problem: magnitudes (Eq. 8), the unmatched tokens' adjacency
//                  matrix (Eq. 9) in LDS, the greedy highest-degree loop (Eq. 10-13) as stated,
//                  new entries and references
//   decode_small   all of it in one launch when a call brings at most four tokens per problem
#include <math.h>

#include <mutex>

#include "mma.h"

// Scratch memory of spindle_decode_merge_static: lives in the code object, one copy per GPU
// the library is loaded on, for the life of the process.  In host code this name is only a
// handle for hipGetSymbolAddress; the address kernels get is looked up per device below.
constexpr size_t kStaticScratchBytes = (size_t)6 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace spindle {
namespace {

constexpr int kDecodeMax = 1024;     // new tokens per problem and call
constexpr int kMatchTokens = 32;     // new tokens per workgroup of decode_match: the columns of a matrix tile
constexpr int kMatchThreads = 256;
constexpr int kMatchWaves = kMatchThreads / kWave;
constexpr int kWaveTiles = 4;        // tiles of 32 stored entries per wave
constexpr int kSliceEntries = kMatchWaves * kWaveTiles * 32;
constexpr int kBuildThreads = 1024;

struct DecodeParams {
  const char *X;        // [U][m][128] new tokens in `dtype`
  char *C;              // [U][cap][128] codebook in `dtype`, rows < n_codes[u] valid, appended to
  int32_t *n_codes;     // [U] in: stored entries, out: stored entries afterwards
  int32_t *n_found;     // [U] entries needed (stored + new picks), may exceed cap
  int32_t *n_matched;   // [U] optional: tokens merged with an existing entry
  int32_t *ref;         // [U][m]
  float *mag;           // [U][m]
  double *part_v;       // workspace [U][slices][m16] best cosine of a token within a slice of entries
  int *part_i;          //           and its entry, -1 if none exceeds theta
  int dtype, U, m, cap;
  int m16, slices;      // m rounded up to 16; ceil(cap / 512)
  double theta;
};

template <int DT>
__device__ __forceinline__ const char *token_row(const DecodeParams &p, int u, int a) {
  return p.X + ((size_t)u * p.m + a) * (kHeadDim * sizeof(typename Elem<DT>::type));
}

// (value, index) maximum with the lower index winning ties
__device__ __forceinline__ void take_better(double &bv, int &bi, double ov, int oi) {
  if (oi >= 0 && (bi < 0 || ov > bv || (ov == bv && oi < bi))) {
    bv = ov;
    bi = oi;
  }
}

// The fragments of a lane's row for the matrix instructions.  Which dimensions a lane group holds for a step
// is free as long as both operands agree: fp32 rows are read 16 bytes at a time.
template <int DT>
__device__ __forceinline__ void load_row(typename Mma<DT>::frag (&f)[Mma<DT>::kSteps], const char *row, int g) {
  if constexpr (DT == SPINDLE_F32) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const u4 x = *reinterpret_cast<const u4 *>(row + (8 * j + 4 * g) * 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) f[4 * j + i] = __uint_as_float(x[i]);
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < Mma<DT>::kSteps; ++ks) f[ks] = Mma<DT>::load(row, ks, g);
  }
}

template <int DT>
__device__ __forceinline__ f16v row_products(const typename Mma<DT>::frag (&a)[Mma<DT>::kSteps],
                                             const typename Mma<DT>::frag (&b)[Mma<DT>::kSteps]) {
  f16v acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
  for (int ks = 0; ks < Mma<DT>::kSteps; ++ks) acc = Mma<DT>::mma(a[ks], b[ks], acc);
  return acc;
}

// A tile of 32 rows one behind the other, read as it lies in memory and turned into fragments in LDS (piece j of row r
// at place j ^ r): lanes next to each other with different rows, 16 bytes each, take four times as long to read.
template <int DT>
struct TileRows {
  static constexpr int row_bytes = Mma<DT>::kRowBytes, kPieces = row_bytes / 16, kLoads = 32 * kPieces / kWave;
  u4 v[kLoads];
  __device__ __forceinline__ void read(const char *rows, int n) {   // n: rows that exist; the last one again past them
    const int lane = lane_id();
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int i = q * kWave + lane;
      v[q] = *reinterpret_cast<const u4 *>(rows + (size_t)min(i / kPieces, n - 1) * row_bytes + i % kPieces * 16);
    }
  }
  __device__ __forceinline__ void turn(char *lds, typename Mma<DT>::frag (&f)[Mma<DT>::kSteps]) {
    const int lane = lane_id(), g = lane >> 5, c = lane & 31;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the tile before has been read
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      const int i = q * kWave + lane, r = i / kPieces;
      *reinterpret_cast<u4 *>(lds + r * row_bytes + ((i % kPieces ^ r % kPieces) << 4)) = v[q];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS keeps the order of one wave's accesses
#pragma unroll
    for (int j = 0; j < kPieces / 2; ++j) {
      const u4 x = *reinterpret_cast<const u4 *>(lds + c * row_bytes + (((2 * j + g) ^ c % kPieces) << 4));
      if constexpr (DT == SPINDLE_F32) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[4 * j + i] = __uint_as_float(x[i]);
      } else {
        f[j] = __builtin_bit_cast(typename Mma<DT>::frag, x);
      }
    }
  }
};

// 1 / norm of a row from its squared norm in fp32: 0 for a zero row, NaN where that or the products may leave
// the range of fp32 or are no numbers (such rows are decided in double precision).
__device__ __forceinline__ float inverse_of(float ss, bool zero) {
  if (zero) return 0.f;
  return ss > 0x1p-80f && ss < 0x1p100f ? __builtin_amdgcn_rsqf(ss) : NAN;
}

// Whether a row is zero, where every wave-mate from `group` lanes on has a part of it.  Squares of fp16 numbers don't
// vanish; for the other types the bits say whether a squared norm of 0 stands for zeros: the padding of a prompt is
// no reason to decide all of a row's pairs in double precision.  bits(): all words of the lane's part or'ed.
template <int DT, class F>
__device__ __forceinline__ bool zero_row(float ss, bool asks, int group, F bits) {
  if (DT == SPINDLE_F16 || !__any(asks && ss == 0.f)) return ss == 0.f;
  uint32_t x = bits();
  for (int o = group; o < kWave; o <<= 1) x |= (uint32_t)__shfl_xor((int)x, o);
  return ss == 0.f && (x & (DT == SPINDLE_F32 ? 0x7FFFFFFFu : 0x7FFF7FFFu)) == 0u;
}

// The same where a lane pair (lane, lane + 32) holds the row's fragments.
template <int DT>
__device__ __forceinline__ float inverse_norm(const typename Mma<DT>::frag (&f)[Mma<DT>::kSteps]) {
  float ss = 0.f;
#pragma unroll
  for (int ks = 0; ks < Mma<DT>::kSteps; ++ks) {
    if constexpr (DT == SPINDLE_F32) {
      ss = fmaf(f[ks], f[ks], ss);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = (float)f[ks][j];
        ss = fmaf(x, x, ss);
      }
    }
  }
  ss += __shfl_xor(ss, 32);
  return inverse_of(ss, zero_row<DT>(ss, true, 32, [&]() {
    uint32_t x = 0;
#pragma unroll
    for (int ks = 0; ks < Mma<DT>::kSteps; ++ks) {
      if constexpr (DT == SPINDLE_F32) {
        x |= __float_as_uint(f[ks]);
      } else {
        const u4 w = __builtin_bit_cast(u4, f[ks]);
        x |= w[0] | w[1] | w[2] | w[3];
      }
    }
    return x;
  }));
}

// cos(x, c) as the decision is defined: double precision, every sum over the dimensions in order, 0 for a zero row.
template <int DT>
__device__ __forceinline__ double exact_cosine(const char *x, const char *c) {
  typedef typename Elem<DT>::type T;
  constexpr int per = 16 / sizeof(T), pieces = kHeadDim / per, kBatch = 4;
  const u4 *rx = reinterpret_cast<const u4 *>(x), *rc = reinterpret_cast<const u4 *>(c);
  double acc = 0.0, xx = 0.0, cc = 0.0;
  for (int q0 = 0; q0 < pieces; q0 += kBatch) {
    u4 vx[kBatch], vc[kBatch];
#pragma unroll
    for (int q = 0; q < kBatch; ++q) { vx[q] = rx[q0 + q]; vc[q] = rc[q0 + q]; }
#pragma unroll
    for (int q = 0; q < kBatch; ++q)
#pragma unroll
      for (int k = 0; k < per; ++k) {
        const double a = (double)Elem<DT>::to_float(reinterpret_cast<const T *>(&vx[q])[k]);
        const double b = (double)Elem<DT>::to_float(reinterpret_cast<const T *>(&vc[q])[k]);
        acc += a * b;
        xx += a * a;
        cc += b * b;
      }
  }
  const double den = sqrt(xx) * sqrt(cc);
  return den > 0.0 ? acc / den : 0.0;
}

// Products of 128 terms in fp32 (truncated sums included) and the norms: approximate cosines are off by less than 2.5e-5.
constexpr float kDecodeGuard = 7e-5f;

// One workgroup = 32 new tokens x 512 stored entries.  A wave multiplies the tokens (matrix columns) with
// four tiles of 32 entries; the largest approximate cosine F of a token over the block and the threshold leave
// the entries with a value of at least F - 2 kDecodeGuard and theta - kDecodeGuard, one or none as a rule.  Their
// (token, entry) pairs go to a list in LDS that has room for all of them, and a thread each evaluates them in
// double precision, every sum over the dimensions in order, as the decision is defined.  Rows that leave
// the range of the approximation are on the list with everything.  The best entry of each token within the
// slice goes to the workspace; decode_build combines the slices.
// Bound by the latency of rows, norms, list and pairs.  8 heads, 256 fp16 tokens against 1650 entries: 44 us with every
// pair in double precision and a launch before it for the tokens as doubles (6 us), 16 now; with decode_build, 103 us and
// 39; 32 heads, 1024 tokens against 4096 1170 and 329 (fp32 1820 and 719).
template <int DT>
__global__ __launch_bounds__(kMatchThreads, 2) void decode_match(DecodeParams p) {
  typedef typename Elem<DT>::type T;
  typedef Mma<DT> M;
  constexpr int row_bytes = kHeadDim * sizeof(T);
  extern __shared__ __attribute__((aligned(16))) char turn[];      // a tile of 32 rows per wave
  __shared__ __attribute__((aligned(16))) float inv_s[kMatchWaves][kWaveTiles][32];
  __shared__ float max_s[kMatchWaves][32];
  __shared__ uint16_t list[kMatchTokens * kSliceEntries];          // token << 9 | entry of the slice
  __shared__ unsigned long long best_s[kMatchTokens], prev_s[kMatchTokens];
  __shared__ int idx_s[kMatchTokens], nlist;
  static_assert(kSliceEntries == 512 && kMatchTokens <= 128, "list words");
  const int ntiles = (p.m + kMatchTokens - 1) / kMatchTokens;
  const int u = blockIdx.y, a0 = (int)(blockIdx.x % ntiles) * kMatchTokens, slice = blockIdx.x / ntiles, tid = threadIdx.x;
  const int lane = lane_id(), wave = tid >> 6, g = lane >> 5, c = lane & 31;
  int nc = p.n_codes[u];
  nc = nc < 0 ? 0 : (nc > p.cap ? p.cap : nc);
  if (slice * kSliceEntries >= nc) return;          // decode_build only reads the slices below nc
  const char *Cu = p.C + (size_t)u * p.cap * row_bytes;
  if (tid < kMatchTokens) {
    best_s[tid] = prev_s[tid] = 0;
    idx_s[tid] = INT32_MAX;
  }
  if (tid == 0) nlist = 0;

  constexpr bool kTurn = DT != SPINDLE_F32;          // (fp32 tiles would take the registers of a second wave per SIMD)
  char *own = turn + wave * (32 * row_bytes);
  TileRows<DT> ahead;
  typename M::frag xf[M::kSteps];
  if constexpr (kTurn) {
    ahead.read(token_row<DT>(p, u, a0), p.m - a0);
    ahead.turn(own, xf);
  } else {
    load_row<DT>(xf, token_row<DT>(p, u, min(a0 + c, p.m - 1)), g);
  }
  const bool on = a0 + c < p.m;
  const float im = inverse_norm<DT>(xf);
  const int e_wave = slice * kSliceEntries + wave * (kWaveTiles * 32);
  if (kTurn && e_wave < nc) ahead.read(Cu + (size_t)e_wave * row_bytes, nc - e_wave);
  f16v x[kWaveTiles];
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < kWaveTiles; ++t) {
    if (e_wave + 32 * t >= nc) break;                // wave-uniform
    typename M::frag cf[M::kSteps];
    const int next = e_wave + 32 * t + 32;
    if constexpr (kTurn) {
      ahead.turn(own, cf);
      if (t + 1 < kWaveTiles && next < nc) ahead.read(Cu + (size_t)next * row_bytes, nc - next);
    } else {
      load_row<DT>(cf, Cu + (size_t)min(next - 32 + c, nc - 1) * row_bytes, g);
    }
    x[t] = row_products<DT>(cf, xf);
    const float ie = inverse_norm<DT>(cf);
    if (g == 0) inv_s[wave][t][c] = ie;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS keeps the order of one wave's accesses
#pragma unroll
    for (int v = 0; v < 16; v += 4) {
      const float4 f = *reinterpret_cast<const float4 *>(&inv_s[wave][t][mma_row(v, g)]);
      const float fv[4] = {f.x, f.y, f.z, f.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float cs = x[t][v + k] * fv[k] * im;   // NaN: a row out of range
        const bool there = e_wave + 32 * t + mma_row(v + k, g) < nc;
        x[t][v + k] = there ? cs : -INFINITY;
        mx = fmaxf(mx, there && fabsf(cs) <= 2.f ? cs : -INFINITY);
      }
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  if (g == 0) max_s[wave][c] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kMatchWaves; ++w) mx = fmaxf(mx, max_s[w][c]);
  const float thr = fmaxf((float)p.theta - kDecodeGuard, mx - 2.f * kDecodeGuard);
#pragma unroll
  for (int t = 0; t < kWaveTiles; ++t) {
    if (e_wave + 32 * t >= nc) break;
    uint32_t take = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) take |= (uint32_t)!(x[t][v] < thr) << v;   // (NaN: take)
    if (!on) take = 0;
    if (take) {
      int at = atomicAdd(&nlist, __popc(take));
      for (; take; take &= take - 1) {
        const int v = __builtin_ctz(take);
        list[at++] = (uint16_t)(c << 9 | (wave * (kWaveTiles * 32) + 32 * t + mma_row(v, g)));
      }
    }
  }
  __syncthreads();

  for (int i0 = 0; i0 < nlist; i0 += kMatchThreads) {
    unsigned long long key = 0;
    int tok = 0, e = 0;
    if (i0 + tid < nlist) {
      tok = list[i0 + tid] >> 9;
      e = slice * kSliceEntries + (list[i0 + tid] & 511);
      const double cs = exact_cosine<DT>(token_row<DT>(p, u, a0 + tok), Cu + (size_t)e * row_bytes);
      if (cs > p.theta) {
        key = order_key(cs);
        atomicMax(&best_s[tok], key);
      }
    }
    __syncthreads();
    const bool top = key != 0 && best_s[tok] == key;
    if (top && prev_s[tok] != key) idx_s[tok] = INT32_MAX;
    __syncthreads();
    if (top) {
      atomicMin(&idx_s[tok], e);
      prev_s[tok] = key;
    }
    __syncthreads();
  }
  if (tid < kMatchTokens && a0 + tid < p.m) {
    const unsigned long long b = best_s[tid];
    const size_t at = ((size_t)u * p.slices + slice) * p.m16 + a0 + tid;
    p.part_v[at] = b == 0 ? 0.0 : __longlong_as_double((long long)(b >> 63 ? b & ~(1ull << 63) : ~b));
    p.part_i[at] = b == 0 ? -1 : idx_s[tid];
  }
}

template <int DT>
constexpr size_t match_lds() { return DT == SPINDLE_F32 ? 0 : kMatchWaves * 32 * Mma<DT>::kRowBytes; }

// LDS of decode_build, in 32-bit words, for m new tokens: their magnitudes as doubles and 1 / them as floats, the
// adjacency rows with an odd pitch (thread i walks row i: consecutive rows must start in
// different banks), two bitmaps, then four 16-bit arrays (position in the input, degree, pick
// number per token; the pick list).  156,000 bytes at m = 1024.
__host__ __device__ inline int build_pitch(int m) { return ((m + 31) / 32) | 1; }
__host__ __device__ inline size_t build_lds_words(int m) {
  return 3 * (size_t)((m + 1) & ~1) + (size_t)m * build_pitch(m) + 2 * (size_t)((m + 31) / 32) +
         2 * (size_t)((m + 1) & ~1);
}

// The loop of Alg. 1 on at most 64 K tokens by one wave: a lane has tokens lane, lane + 64, ... with their rows in
// registers, the remaining tokens are 2 K words that all lanes keep.  No barriers: a pick is a reduction over the
// wave, where the workgroup needs four barriers for it.
template <int K>
__device__ __forceinline__ int build_by_wave(const uint32_t *adj, int pitch, int r, uint16_t *rref, uint16_t *picks) {
  const int lane = lane_id();
  uint32_t rows[K][2 * K], alive[2 * K];
#pragma unroll
  for (int w = 0; w < 2 * K; ++w) {
    alive[w] = r >= 32 * w + 32 ? 0xFFFFFFFFu : (r > 32 * w ? (1u << (r - 32 * w)) - 1u : 0u);
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int t = lane + 64 * k;
      rows[k][w] = t < r && 32 * w < r ? adj[(size_t)t * pitch + w] : 0u;
    }
  }
  int npicks = 0;
  for (;;) {
    uint32_t top = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      uint32_t own = 0;                              // the word of `alive` that holds token lane + 64 k
      int d = 0;
#pragma unroll
      for (int w = 0; w < 2 * K; ++w) {
        d += __popc(rows[k][w] & alive[w]);
        if (w == 2 * k + (lane >> 5)) own = alive[w];
      }
      const uint32_t key = own >> (lane & 31) & 1u ? (uint32_t)d << 16 | (uint32_t)(0xFFFF - (lane + 64 * k)) : 0u;
      top = key > top ? key : top;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const uint32_t x = __shfl_xor(top, o);
      top = x > top ? x : top;
    }
    top = (uint32_t)__builtin_amdgcn_readfirstlane((int)top);
    if (top == 0u) break;                            // nobody left
    if (top >> 16 == 1u) {
      // only isolated tokens are left: each is its own entry, in index order
      int before = npicks;
#pragma unroll
      for (int w = 0; w < 2 * K; ++w) {
        const int k = w / 2;
        if ((lane >> 5) == (w & 1) && (alive[w] >> (lane & 31) & 1u)) {
          const int at = before + __popc(alive[w] & ((1u << (lane & 31)) - 1u));
          rref[lane + 64 * k] = (uint16_t)at;
          picks[at] = (uint16_t)(lane + 64 * k);
        }
        before += __popc(alive[w]);
      }
      npicks = before;
      break;
    }
    const int v = 0xFFFF - (int)(top & 0xFFFFu);
    if (lane == 0) picks[npicks] = (uint16_t)v;
#pragma unroll
    for (int w = 0; w < 2 * K; ++w) {
      const uint32_t dying = 32 * w < r ? adj[(size_t)v * pitch + w] & alive[w] : 0u;
      if ((lane >> 5) == (w & 1) && (dying >> (lane & 31) & 1u)) rref[lane + 64 * (w / 2)] = (uint16_t)npicks;   // Eq. 12
      alive[w] &= ~dying;                            // Eq. 13: degrees are counted among the remaining ones
    }
    ++npicks;
  }
  return npicks;
}

// Bound by latency, one workgroup per problem.  8 heads, 256 fp16 tokens of which some 70 match nothing: 61 us with
// every pair of them in double precision and four barriers per pick, 23 us now.
template <int DT>
__global__ __launch_bounds__(kBuildThreads) void decode_build(DecodeParams p) {
  typedef typename Elem<DT>::type T;
  typedef Mma<DT> M;
  constexpr int per = 16 / sizeof(T);
  constexpr int pieces = kHeadDim / per;
  constexpr int kWaves = kBuildThreads / kWave;
  extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
  __shared__ int wave_sum[kWaves];
  __shared__ uint32_t wave_key[kWaves];
  __shared__ int sh_r, sh_npicks;
  const int u = blockIdx.x, m = p.m, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int m2 = (m + 1) & ~1, pitch = build_pitch(m);
  double *mag64 = reinterpret_cast<double *>(lds);   // [m2] of a token
  float *inv = reinterpret_cast<float *>(mag64 + m2);   // [m2] 1 / magnitude, 0 or NaN as inverse_norm, of an unmatched token
  uint32_t *adj = lds + 3 * m2;                      // [m][pitch]
  uint32_t *alive = adj + (size_t)m * pitch;         // [(m + 31) / 32]
  uint32_t *dying = alive + (m + 31) / 32;           // [(m + 31) / 32]
  uint16_t *rest = reinterpret_cast<uint16_t *>(dying + (m + 31) / 32);   // unmatched tokens, input order
  uint16_t *deg = rest + m2;
  uint16_t *rref = deg + m2;                         // pick number of each unmatched token
  uint16_t *picks = rref + m2;                       // unmatched-token index of each pick
  int nc = p.n_codes[u];
  nc = nc < 0 ? 0 : (nc > p.cap ? p.cap : nc);
  int32_t *ref = p.ref + (size_t)u * m;

  // magnitudes; best stored entry of each token over the slices (ascending, so ties stay with the
  // lower index), then the unmatched tokens in input order
  {
    int mine = -1;
    if (tid < m) {
      const u4 *row = reinterpret_cast<const u4 *>(token_row<DT>(p, u, tid));
      const int used = (nc + kSliceEntries - 1) / kSliceEntries;
      const size_t at = (size_t)u * p.slices * p.m16 + tid;
      u4 v[pieces];
#pragma unroll
      for (int q = 0; q < pieces; ++q) v[q] = row[q];
      double bv = 0.0;
      for (int sl = 0; sl < used; ++sl) take_better(bv, mine, p.part_v[at + (size_t)sl * p.m16], p.part_i[at + (size_t)sl * p.m16]);
      ref[tid] = mine;
      double ss = 0.0;
#pragma unroll
      for (int q = 0; q < pieces; ++q)
#pragma unroll
        for (int k = 0; k < per; ++k) {
          const double x = (double)Elem<DT>::to_float(reinterpret_cast<const T *>(&v[q])[k]);
          ss += x * x;
        }
      const double mg = sqrt(ss);
      mag64[tid] = mg;
      p.mag[(size_t)u * m + tid] = (float)mg;
    }
    const bool un = tid < m && mine < 0;
    const unsigned long long mk = __ballot(un);
    if (lane == 0) wave_sum[wave] = __popcll(mk);
    __syncthreads();
    int before = 0, total = 0;
    for (int w = 0; w < kWaves; ++w) {
      before += w < wave ? wave_sum[w] : 0;
      total += wave_sum[w];
    }
    if (un) {
      const int i = before + __popcll(mk & ((1ull << lane) - 1ull));
      const double mg = mag64[tid];
      rest[i] = (uint16_t)tid;
      inv[i] = mg == 0.0 ? 0.f : mg > 0x1p-40 && mg < 0x1p50 ? (float)(1.0 / mg) : NAN;
    }
    if (tid == 0) sh_r = total;
  }
  __syncthreads();
  const int r = sh_r, Wr = (r + 31) / 32;
  if (tid == 0 && p.n_matched) p.n_matched[u] = m - r;

  // Eq. 9 among the unmatched tokens, 32 x 32 pairs at a time, each tile of them once: matrix-core cosines, those
  // within the guard of theta in double precision.  Word J of rows 32 I .. and word I of rows 32 J .. come from one decision.
  {
    const int g = lane >> 5, c = lane & 31;
    const float lo = (float)p.theta - kDecodeGuard, hi = (float)p.theta + kDecodeGuard;
    for (int pair = wave, I = 0, J = 0, at = 0; pair < Wr * (Wr + 1) / 2; pair += kWaves) {
      for (; at + (Wr - I) <= pair; ++I) at += Wr - I;
      J = I + pair - at;
      typename M::frag xj[M::kSteps], xi[M::kSteps];
      const int i = 32 * I + c, j = 32 * J + c;
      load_row<DT>(xj, token_row<DT>(p, u, rest[min(j, r - 1)]), g);
      load_row<DT>(xi, token_row<DT>(p, u, rest[min(i, r - 1)]), g);
      const f16v x = row_products<DT>(xi, xj);
      const float fj = inv[min(j, r - 1)];
      uint32_t yes = 0, close = 0;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int a = 32 * I + mma_row(v, g);
        const float cs = x[v] * inv[min(a, r - 1)] * fj;
        const bool there = a < r && j < r;
        if (there && cs > hi) yes |= 1u << v;
        else if (there && !(cs < lo)) close |= 1u << v;
      }
      for (; close; close &= close - 1) {
        const int v = __builtin_ctz(close), a = 32 * I + mma_row(v, g);
        const int ta = rest[a], tb = rest[j];
        const double den = mag64[ta] * mag64[tb];
        const double cs = den > 0.0 ? dot64<DT, 4>(token_row<DT>(p, u, ta), token_row<DT>(p, u, tb)) / den : 0.0;
        if (cs > p.theta) yes |= 1u << v;
      }
      uint32_t bits = 0;                             // of the lane's token j: rows of the tile it is adjacent to
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const bool b = yes >> v & 1u || (I == J && mma_row(v, g) == c && j < r);   // G_aa = 1
        bits |= (uint32_t)b << mma_row(v, g);
        const unsigned long long mk = __ballot(b);
        if (I != J && lane == 0) {
          if (32 * I + mma_row(v, 0) < r) adj[(size_t)(32 * I + mma_row(v, 0)) * pitch + J] = (uint32_t)mk;
          if (32 * I + mma_row(v, 1) < r) adj[(size_t)(32 * I + mma_row(v, 1)) * pitch + J] = (uint32_t)(mk >> 32);
        }
      }
      bits |= (uint32_t)__shfl_xor((int)bits, 32);
      if (g == 0 && j < r) adj[(size_t)j * pitch + I] = bits;
    }
  }
  __syncthreads();

  // Alg. 1: take the remaining token of highest degree (lowest index on ties), give its
  // remaining neighbourhood its entry, remove it, lower the degrees of the others (Eq. 11-13)
  int npicks = 0;
  if (r <= 256) {
    if (wave == 0) {
      if (r <= 64) npicks = build_by_wave<1>(adj, pitch, r, rref, picks);
      else if (r <= 128) npicks = build_by_wave<2>(adj, pitch, r, rref, picks);
      else npicks = build_by_wave<4>(adj, pitch, r, rref, picks);
      if (lane == 0) sh_npicks = npicks;
    }
    __syncthreads();
    npicks = sh_npicks;
  } else {
    for (int w = tid; w < Wr; w += kBuildThreads) {
      const int lo = w * 32;
      alive[w] = r >= lo + 32 ? 0xFFFFFFFFu : (1u << (r - lo)) - 1u;
    }
    if (tid < r) {                                   // Eq. 10
      int d = 0;
      for (int w = 0; w < Wr; ++w) d += __popc(adj[(size_t)tid * pitch + w]);
      deg[tid] = (uint16_t)d;
    }
    __syncthreads();
    for (;;) {
      const bool live = tid < r && ((alive[tid >> 5] >> (tid & 31)) & 1u);
      uint32_t key = live ? ((uint32_t)deg[tid] << 16) | (uint32_t)(0xFFFF - tid) : 0u;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const uint32_t ok = __shfl_xor(key, o);
        key = ok > key ? ok : key;
      }
      if (lane == 0) wave_key[wave] = key;
      __syncthreads();
      uint32_t top = 0;
      for (int w = 0; w < kWaves; ++w) top = wave_key[w] > top ? wave_key[w] : top;
      if (top == 0u) break;                          // nobody left
      if ((top >> 16) == 1u) {
        // only isolated tokens are left: each is its own entry, in index order
        if (live) {
          int before = 0;
          for (int w = 0; w < (tid >> 5); ++w) before += __popc(alive[w]);
          before += __popc(alive[tid >> 5] & ((1u << (tid & 31)) - 1u));
          rref[tid] = (uint16_t)(npicks + before);
          picks[npicks + before] = (uint16_t)tid;
        }
        int total = 0;
        for (int w = 0; w < Wr; ++w) total += __popc(alive[w]);
        npicks += total;
        break;
      }
      const int v = 0xFFFF - (int)(top & 0xFFFFu);
      if (tid < Wr) dying[tid] = adj[(size_t)v * pitch + tid] & alive[tid];
      if (tid == 0) picks[npicks] = (uint16_t)v;
      __syncthreads();
      if (live) {
        if ((dying[tid >> 5] >> (tid & 31)) & 1u) {
          rref[tid] = (uint16_t)npicks;              // Eq. 12
        } else {
          int gone = 0;
          for (int w = 0; w < Wr; ++w) {
            const uint32_t dw = dying[w];
            if (dw) gone += __popc(adj[(size_t)tid * pitch + w] & dw);
          }
          deg[tid] = (uint16_t)(deg[tid] - gone);    // Eq. 13, as a degree update
        }
      }
      __syncthreads();
      if (tid < Wr) alive[tid] &= ~dying[tid];
      ++npicks;
      __syncthreads();
    }
    __syncthreads();
  }

  // outputs: references of the unmatched tokens, the new rows, the counts
  const int room = p.cap - nc > 0 ? p.cap - nc : 0;
  const int stored = npicks < room ? npicks : room;
  if (tid < r) ref[rest[tid]] = (int)rref[tid] < room ? nc + (int)rref[tid] : -1;
  T *Cu = reinterpret_cast<T *>(p.C) + (size_t)u * p.cap * kHeadDim;
  for (int j = wave; j < stored; j += kWaves) {
    const int tok = rest[picks[j]];
    const T *src = reinterpret_cast<const T *>(token_row<DT>(p, u, tok));
    const double mg = mag64[tok];
    for (int d = lane; d < kHeadDim; d += kWave) {
      const double x = (double)Elem<DT>::to_float(src[d]);
      Cu[(size_t)(nc + j) * kHeadDim + d] = Elem<DT>::from_float(mg > 0.0 ? (float)(x / mg) : 0.f);
    }
  }
  if (tid == 0) {
    p.n_found[u] = nc + npicks;
    p.n_codes[u] = nc + stored;
  }
}

// The usual decode step brings one token per head (a few with speculative decoding): then
// two launches cost more than the work.  One workgroup per problem does it all: the search of the
// stored entries, then Alg. 1 on the at most MT unmatched tokens by the first wave (adjacency in one word
// per token, the loop as stated).
constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;

template <int MT>
struct SmallLds {
  __attribute__((aligned(16))) double xs[kHeadDim][MT];
  double mag[MT];
  int ref[MT];                                       // entry a token matched, -1 if none; slots past m count as matched
  uint32_t adjm[MT];
};

// The tokens as doubles and, by the threads of the last wave, their magnitudes.  Ends without a barrier.
template <int DT, int MT>
__device__ __forceinline__ void small_tokens(const DecodeParams &p, int u, SmallLds<MT> &l) {
  typedef typename Elem<DT>::type T;
  const int tid = threadIdx.x;
  for (int i = tid; i < MT * kHeadDim; i += kSmallThreads) {
    const int tok = i / kHeadDim, dim = i % kHeadDim;
    l.xs[dim][tok] = tok < p.m ? (double)Elem<DT>::to_float(reinterpret_cast<const T *>(token_row<DT>(p, u, tok))[dim]) : 0.0;
  }
  __syncthreads();
  const int t = tid - (kSmallThreads - kWave);
  if (t >= 0 && t < MT) {
    double ss = 0.0;
#pragma unroll 16
    for (int dim = 0; dim < kHeadDim; ++dim) ss += l.xs[dim][t] * l.xs[dim][t];
    const double mg = sqrt(ss);
    l.mag[t] = mg;
    l.adjm[t] = 0u;
    if (t < p.m) p.mag[(size_t)u * p.m + t] = (float)mg;
  }
}

// The rest, by the first wave.
template <int DT, int MT>
__device__ __forceinline__ void small_finish(const DecodeParams &p, int u, int nc, SmallLds<MT> &l) {
  typedef typename Elem<DT>::type T;
  const int lane = lane_id(), m = p.m;
  // the unmatched tokens, in input order, among themselves (Eq. 9-13)
  const bool un = lane < m && l.ref[lane < MT ? lane : 0] < 0;
  const unsigned long long mask = __ballot(un);
  const int r = __popcll(mask);
  int rest[MT];                                      // token of each unmatched position (wave-uniform)
  {
    unsigned long long left = mask;
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      rest[i] = left ? __builtin_ctzll(left) : 0;
      left &= left - 1;
    }
  }
  for (int pair = lane; pair < MT * MT; pair += kWave) {
    const int i = pair / MT, j = pair % MT;
    if (i < j && j < r) {
      const int a = rest[i], b = rest[j];
      double acc = 0.0;
      for (int dim = 0; dim < kHeadDim; ++dim) acc += l.xs[dim][a] * l.xs[dim][b];
      const double den = l.mag[a] * l.mag[b];
      const double cs = den > 0.0 ? acc / den : 0.0;
      if (cs > p.theta) {
        atomicOr(&l.adjm[i], 1u << j);
        atomicOr(&l.adjm[j], 1u << i);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0);
  __builtin_amdgcn_wave_barrier();
  int rref[MT], picks[MT];
  int npicks = 0;
  {
    uint32_t alive = r >= 32 ? 0xFFFFFFFFu : (1u << r) - 1u;
    uint32_t rows[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      rows[i] = l.adjm[i] | (1u << i);                 // G_aa = 1
      rref[i] = 0;
      picks[i] = 0;
    }
    while (alive) {                                  // every lane runs the same tiny loop
      int pick = 0, top = 0;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const int d = (alive >> i) & 1u ? __popc(rows[i] & alive) : 0;
        if (d > top) { top = d; pick = i; }          // strict: lowest index on ties
      }
      uint32_t leaving = 0;
#pragma unroll
      for (int i = 0; i < MT; ++i)
        if (i == pick) leaving = rows[i] & alive;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        if ((leaving >> i) & 1u) rref[i] = npicks;
        if (i == npicks) picks[i] = pick;
      }
      alive &= ~leaving;
      ++npicks;
    }
  }
  const int room = p.cap - nc > 0 ? p.cap - nc : 0;
  const int stored = npicks < room ? npicks : room;
  if (lane < m) {
    int out = l.ref[lane < MT ? lane : 0];
    if (out < 0) {
      const int pos = __popcll(mask & ((1ull << lane) - 1ull));
      int rr = 0;
#pragma unroll
      for (int i = 0; i < MT; ++i)
        if (i == pos) rr = rref[i];
      out = rr < room ? nc + rr : -1;
    }
    p.ref[(size_t)u * m + lane] = out;
  }
  T *Cu = reinterpret_cast<T *>(p.C) + (size_t)u * p.cap * kHeadDim;
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    if (j < stored) {
      int tok = 0;
#pragma unroll
      for (int i = 0; i < MT; ++i)
        if (i == picks[j]) tok = rest[i];
      const double mg = l.mag[tok];
      for (int d = lane; d < kHeadDim; d += kWave)
        Cu[(size_t)(nc + j) * kHeadDim + d] = Elem<DT>::from_float(mg > 0.0 ? (float)(l.xs[d][tok] / mg) : 0.f);
    }
  }
  if (lane == 0) {
    p.n_found[u] = nc + npicks;
    p.n_codes[u] = nc + stored;
    if (p.n_matched) p.n_matched[u] = m - r;
  }
}

// The value of lane i of the four neighbouring ones.
template <int i>
__device__ __forceinline__ float quad_lane(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), i * 0x55, 0xF, 0xF, true));
}

// fp16 and bf16.  A wave multiplies 16 stored entries at a time with themselves, whose diagonal is their squared norms,
// and with the tokens, four of them over and over in the 16 columns, so that four neighbouring lanes have four entries'
// norms and their products with the four tokens.  The
// entries are read as they lie in memory, two tiles in flight (three and four: 0.4 and 1.5 us slower, more
// registers and all waves' loads at once), and turned round in LDS: read in fragment order,
// where lanes next to each other have different rows, the 422 KB of 1650 entries take a compute unit 12 us, in
// whole rows 3.  Few entries come
// near theta; of those only the ones within 2 kDecodeGuard of a token's largest approximate cosine can be its maximum.
// One such entry that is above theta by more than the guard is the answer; otherwise they are decided in double
// precision as in decode_match, and should the list not hold them (equal entries by the hundred), every pair is.
// Bound by latency: the first rows are asked for before the number of entries is known (the table has them
// all), one barrier before and one after the search.
// One fp16 token each against 1650 entries in 8 heads 14.6 us with all sums in double precision, 10.9 now; four tokens 24.6
// and 13.5; one against 4000 in 32 heads 28.3 and 17.8; 1000 in 256 heads 15.9 and 13.3.
constexpr int kSmallList = 1024;

template <int DT>
__global__ __launch_bounds__(kSmallThreads) void decode_small(DecodeParams p) {
  typedef typename Elem<DT>::type T;
  typedef typename Mma<DT>::frag frag;
  typedef float f4v __attribute__((ext_vector_type(4)));
  constexpr int MT = 4, kTiles = 2, row_bytes = kHeadDim * sizeof(T);
  __shared__ __attribute__((aligned(16))) char turn[kSmallWaves][16 * row_bytes];
  __shared__ SmallLds<MT> l;
  __shared__ float max_s[kSmallWaves][MT];
  __shared__ int list_e[kSmallList];
  __shared__ float list_x[kSmallList];
  __shared__ uint8_t list_t[kSmallList];
  __shared__ unsigned long long best_s[MT], prev_s[MT];
  __shared__ int nlist, nleft[MT], unsure;
  const int u = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, m = p.m;
  const int r16 = lane & 15, quarter = lane >> 4;
  int nc = p.n_codes[u];
  const char *Cu = p.C + (size_t)u * p.cap * row_bytes;
  auto product = [](frag a, frag b, f4v c) __attribute__((always_inline)) {
    if constexpr (DT == SPINDLE_F16) return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  };
  u4 ring[kTiles][4];
  auto load = [&](int k, int t) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      ring[k][s] = *reinterpret_cast<const u4 *>(Cu + (size_t)min(t * 16 + 4 * s + quarter, p.cap - 1) * row_bytes + r16 * 16);
  };
#pragma unroll
  for (int k = 0; k < kTiles; ++k) load(k, wave + k * kSmallWaves);
  frag xf[4];                                        // (which dimensions a quarter of the wave holds is free)
  const int tok = lane & 3;                          // the lane's column
  {
    const char *row = token_row<DT>(p, u, min(tok, m - 1)) + quarter * 16;
#pragma unroll
    for (int s = 0; s < 4; ++s) xf[s] = *reinterpret_cast<const frag *>(row + s * 64);
  }
  if (tid < MT) {
    best_s[tid] = prev_s[tid] = 0;
    l.ref[tid] = tid < m ? -1 : 0;
    nleft[tid] = 0;
  }
  if (tid == 0) nlist = unsure = 0;
  small_tokens<DT, MT>(p, u, l);
  float im, mx = -INFINITY;
  {
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < 8; ++j) ss = fmaf((float)xf[s][j], (float)xf[s][j], ss);
    ss += __shfl_xor(ss, 16);
    ss += __shfl_xor(ss, 32);
    im = inverse_of(ss, zero_row<DT>(ss, true, 16, [&]() {
      uint32_t x = 0;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const u4 w = __builtin_bit_cast(u4, xf[s]);
        x |= w[0] | w[1] | w[2] | w[3];
      }
      return x;
    }));
  }
  nc = nc < 0 ? 0 : (nc > p.cap ? p.cap : nc);
  const int ntiles = (nc + 15) / 16;
  const float near = (float)p.theta - kDecodeGuard;
  // Result v of a lane: entry 4 quarter + v, column r16.  Lanes 4 quarter .. of a row of 16 have a norm each.
  const bool mine = quarter == r16 >> 2 && tok < m;
  for (int t0 = wave; t0 < ntiles; t0 += kTiles * kSmallWaves) {
#pragma unroll
    for (int k = 0; k < kTiles; ++k) {
      const int tile = t0 + k * kSmallWaves;
      if (tile >= ntiles) break;                     // wave-uniform
      f4v dot = {0.f, 0.f, 0.f, 0.f}, own = {0.f, 0.f, 0.f, 0.f};
      // piece j of row r at place j ^ r: sixteen consecutive lanes of either access hit all banks
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the tile before has been read
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = 4 * s + quarter;
        *reinterpret_cast<u4 *>(turn[wave] + r * row_bytes + ((r16 ^ r) << 4)) = ring[k][s];
      }
      if (tile + kTiles * kSmallWaves < ntiles) load(k, tile + kTiles * kSmallWaves);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS keeps the order of one wave's accesses
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const frag f = *reinterpret_cast<const frag *>(turn[wave] + r16 * row_bytes + (((4 * s + quarter) ^ r16) << 4));
        own = product(f, f, own);
        dot = product(f, xf[s], dot);
      }
      const float ss = (r16 & 2) ? ((r16 & 1) ? own[3] : own[2]) : ((r16 & 1) ? own[1] : own[0]);
      const float ie = inverse_of(ss, zero_row<DT>(ss, quarter == r16 >> 2 && tile * 16 + r16 < nc, 16, [&]() {
        uint32_t x = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const u4 w = *reinterpret_cast<const u4 *>(turn[wave] + r16 * row_bytes + (((4 * s + quarter) ^ r16) << 4));
          x |= w[0] | w[1] | w[2] | w[3];
        }
        return x;
      }));
      const float thr = fmaxf(near, mx - 2.f * kDecodeGuard);
      float x[4];                                    // NaN: a row out of range
      x[0] = dot[0] * quad_lane<0>(ie) * im;
      x[1] = dot[1] * quad_lane<1>(ie) * im;
      x[2] = dot[2] * quad_lane<2>(ie) * im;
      x[3] = dot[3] * quad_lane<3>(ie) * im;
      const int e0 = tile * 16 + 4 * quarter;
      uint32_t take = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) take |= (uint32_t)(mine && e0 + v < nc && !(x[v] < thr)) << v;
      for (; take; take &= take - 1) {
        const int v = __builtin_ctz(take), at = atomicAdd(&nlist, 1);
        const float cs = v == 0 ? x[0] : v == 1 ? x[1] : v == 2 ? x[2] : x[3];
        if (fabsf(cs) <= 2.f) mx = fmaxf(mx, cs);
        if (at < kSmallList) {
          list_e[at] = e0 + v;
          list_x[at] = cs;
          list_t[at] = (uint8_t)tok;
        }
      }
    }
  }
  if (__any(mx > -INFINITY))                         // (mostly not)
#pragma unroll
    for (int o = 4; o < kWave; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  if (lane < MT) max_s[wave][lane] = mx;
  __syncthreads();
  const bool all = nlist > kSmallList;
  auto in_reach = [&](int i) {                       // of the largest approximate cosine of its token
    float top = -INFINITY;
#pragma unroll
    for (int w = 0; w < kSmallWaves; ++w) top = fmaxf(top, max_s[w][list_t[i]]);
    return !(list_x[i] < top - 2.f * kDecodeGuard);
  };
  if (!all && tid < nlist && in_reach(tid)) {
    atomicAdd(&nleft[list_t[tid]], 1);
    l.ref[list_t[tid]] = list_e[tid];
    if (!(list_x[tid] > (float)p.theta + kDecodeGuard)) unsure = 1;
  }
  __syncthreads();
  bool exact = all || unsure;
#pragma unroll
  for (int t = 0; t < MT; ++t) exact = exact || nleft[t] > 1;
  if (exact) {
    __syncthreads();
    if (tid < m) l.ref[tid] = -1;
    __syncthreads();
    const size_t nitems = all ? (size_t)nc * m : (size_t)nlist;
    for (size_t i0 = 0; i0 < nitems; i0 += kSmallThreads) {
      unsigned long long key = 0;
      int t = 0, e = 0;
      const size_t i = i0 + tid;
      if (i < nitems && (all || in_reach((int)i))) {
        t = all ? (int)(i % m) : list_t[i];
        e = all ? (int)(i / m) : list_e[i];
        const double cs = exact_cosine<DT>(token_row<DT>(p, u, t), Cu + (size_t)e * row_bytes);
        if (cs > p.theta) {
          key = order_key(cs);
          atomicMax(&best_s[t], key);
        }
      }
      __syncthreads();
      const bool top = key != 0 && best_s[t] == key;
      if (top && prev_s[t] != key) l.ref[t] = INT32_MAX;
      __syncthreads();
      if (top) {
        atomicMin(&l.ref[t], e);
        prev_s[t] = key;
      }
      __syncthreads();
    }
  }
  if (wave != 0) return;
  small_finish<DT, MT>(p, u, nc, l);
}

// fp32: every pair in double precision (fp32 matrix instructions would take as long), every thread a few
// stored entries, then a reduction over the workgroup.
// A sum runs over the dimensions in order, so a lane has a stored row to itself; but rows read by
// their lanes 16 bytes at a time are 64 cache lines per load, which a compute unit's cache loses
// again before the next piece of them is read.  So a wave reads its 64 rows one cache line of each at a
// time, eight lanes per line, a line ahead in registers, and turns them round in LDS.
// The sums in double precision bound it (a token slot costs a multiply-add per element, so the tokens
// are counted in the kernel's type).
constexpr int kSmallLine = 128;                      // bytes of a row at a time
constexpr int kSmallLds = kSmallThreads * kSmallLine;

template <int MT>
__global__ __launch_bounds__(kSmallThreads) void decode_small_f32(DecodeParams p) {
  constexpr int DT = SPINDLE_F32, per = 4, kWaves = kSmallWaves;
  constexpr int row_bytes = kHeadDim * 4, kLines = row_bytes / kSmallLine, kPieces = kSmallLine / 16;
  extern __shared__ __attribute__((aligned(16))) char lines[];
  __shared__ SmallLds<MT> l;
  __shared__ double red_v[kWaves][MT];
  __shared__ int red_i[kWaves][MT];
  const int u = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, m = p.m;
  int nc = p.n_codes[u];
  nc = nc < 0 ? 0 : (nc > p.cap ? p.cap : nc);
  // the wave's entries: 64 of every 1024
  const int ngroups = nc > wave * kWave ? (nc - wave * kWave + kSmallThreads - 1) / kSmallThreads : 0;
  const char *Cb = p.C + (size_t)u * p.cap * row_bytes;
  u4 ahead[kPieces];
  auto load = [&](int step) __attribute__((always_inline)) {   // line step % kLines of group step / kLines
    const int c0 = (step / kLines) * kSmallThreads + wave * kWave;
#pragma unroll
    for (int q = 0; q < kPieces; ++q) {
      const int c = min(c0 + q * (kWave / kPieces) + lane / kPieces, nc - 1);
      ahead[q] = *reinterpret_cast<const u4 *>(Cb + (size_t)c * row_bytes + (step % kLines) * kSmallLine +
                                               (lane % kPieces) * 16);
    }
  };
  if (ngroups > 0) load(0);
  small_tokens<DT, MT>(p, u, l);
  __syncthreads();

  double best[MT];
  int bidx[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    best[t] = 0.0;
    bidx[t] = -1;
  }
  // Few pairs come near theta, and a double-precision division costs as much as twenty multiply-adds: the quotient
  // is only formed where the dot product is not already clearly below theta times the norms (for theta >= 0; a
  // quotient that close to theta from below cannot round up past it).
  const double low = p.theta >= 0.0 ? p.theta * (1.0 - 1e-12) : -INFINITY;
  // piece k of row r at place k ^ (r / 2) % 8: sixteen consecutive lanes of either access hit all 64 banks
  char *own = lines + wave * (kWave * kSmallLine);
  for (int grp = 0; grp < ngroups; ++grp) {          // ascending: the first of equal values stays
    const int c = grp * kSmallThreads + tid;
    double acc[MT], css = 0.0;
#pragma unroll
    for (int t = 0; t < MT; ++t) acc[t] = 0.0;
    auto add = [&](const u4 &v, int dim) __attribute__((always_inline)) {   // 16 bytes from dimension `dim` on
#pragma unroll
      for (int j = 0; j < per; ++j) {
        const double y = (double)__uint_as_float(v[j]);
        css += y * y;
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] += l.xs[dim + j][t] * y;
      }
    };
#pragma unroll 1
    for (int line = 0; line < kLines; ++line) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the line before has been read
#pragma unroll
      for (int q = 0; q < kPieces; ++q) {
        const int r = q * (kWave / kPieces) + lane / kPieces;
        *reinterpret_cast<u4 *>(own + r * kSmallLine + (((lane % kPieces) ^ ((r >> 1) & 7)) << 4)) = ahead[q];
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // LDS keeps the order of one wave's accesses
      const int step = grp * kLines + line;
      if (step + 1 < ngroups * kLines) load(step + 1);
#pragma unroll
      for (int pc = 0; pc < kPieces; ++pc) {
        add(*reinterpret_cast<const u4 *>(own + lane * kSmallLine + ((pc ^ ((lane >> 1) & 7)) << 4)),
            (line * kPieces + pc) * per);
        if (pc & 1) __builtin_amdgcn_sched_barrier(0);   // (all tokens' values at once would not fit the registers)
      }
    }
    if (c >= nc) continue;                           // (lanes past the end summed the last row)
    const double cn = sqrt(css);
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const double den = l.mag[t] * cn;
      if (t < m && (!(den > 0.0) || acc[t] > low * den)) {
        const double cs = den > 0.0 ? acc[t] / den : 0.0;
        if (cs > p.theta) take_better(best[t], bidx[t], cs, c);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    double bv = best[t];
    int bi = bidx[t];
    if (__ballot(bi >= 0) != 0) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double ov = __shfl_xor(bv, o);
        const int oi = __shfl_xor(bi, o);
        take_better(bv, bi, ov, oi);
      }
    }
    if (lane == 0) {
      red_v[wave][t] = bv;
      red_i[wave][t] = bi;
    }
  }
  __syncthreads();
  if (tid < MT) {
    double bv = red_v[0][tid];
    int bi = red_i[0][tid];
    for (int w = 1; w < kWaves; ++w) take_better(bv, bi, red_v[w][tid], red_i[w][tid]);
    l.ref[tid] = tid < m ? bi : 0;
  }
  __syncthreads();
  if (wave != 0) return;

  small_finish<DT, MT>(p, u, nc, l);
}

spindle_status check_decode(const spindle_kv_desc *desc) {
  spindle_status s = check_desc(desc);
  if (s != SPINDLE_OK) return s;
  if (desc->stride_b || desc->stride_h || desc->stride_t)
    SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED, "the new tokens of a decode step are contiguous: strides must be 0");
  if (desc->seq_len > kDecodeMax)
    SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED, "at most %d new tokens per call, got %d", kDecodeMax, desc->seq_len);
  return SPINDLE_OK;
}

// Carves the workspace (or only sizes it when `ws` is null).  The kernels use the partial results alone, and none of it for
// up to four tokens per problem; the size also counts the new tokens as doubles and their magnitudes, 16 KiB per 16
// tokens and problem, which callers have been told and what fits the built-in array is measured by.
size_t decode_carve(const spindle_kv_desc *desc, int cap, void *ws, DecodeParams *p) {
  const size_t U = (size_t)desc->batch * desc->n_kv_heads;
  const int tiles = (desc->seq_len + 15) / 16;
  const int slices = (cap + kSliceEntries - 1) / kSliceEntries;
  Carver cv(ws);
  cv.take<double>(U * desc->seq_len);
  cv.take<double>(U * tiles * kHeadDim * 16);
  double *pv = cv.take<double>(U * tiles * slices * 16);
  int *pi = cv.take<int>(U * tiles * slices * 16);
  if (p) {
    p->part_v = pv;
    p->part_i = pi;
    p->m16 = tiles * 16;
    p->slices = slices;
  }
  return cv.total();
}

}  // namespace
}  // namespace spindle

using namespace spindle;

extern "C" spindle_status spindle_decode_workspace_bytes(const spindle_kv_desc *desc, int32_t max_codes, size_t *bytes) {
  if (!bytes) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "bytes is NULL");
  spindle_status s = check_decode(desc);
  if (s != SPINDLE_OK) return s;
  if (max_codes < 1) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "max_codes must be >= 1");
  *bytes = decode_carve(desc, max_codes, nullptr, nullptr);
  return SPINDLE_OK;
}

namespace {

// Validation both entry points share; *need = spindle_decode_workspace_bytes of the call.
spindle_status decode_check_args(const spindle_kv_desc *desc, const void *X_new, float theta, int32_t max_codes,
                                 const void *C, const int32_t *n_codes, const int32_t *n_found, const int32_t *ref,
                                 const float *mag, size_t *need) {
  spindle_status s = check_decode(desc);
  if (s != SPINDLE_OK) return s;
  if (max_codes < 1) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "max_codes must be >= 1");
  if (!(theta > -1.f && theta < 1.f)) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "theta must lie in (-1, 1)");
  if (!X_new || !C || !n_codes || !n_found || !ref || !mag)
    SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "X_new, C, n_codes, n_found, ref and mag are required");
  if ((reinterpret_cast<uintptr_t>(X_new) | reinterpret_cast<uintptr_t>(C)) & 15)
    SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  *need = decode_carve(desc, max_codes, nullptr, nullptr);
  return SPINDLE_OK;
}

template <int DT>
spindle_status launch_small(const DecodeParams &p, hipStream_t st) {
  hipLaunchKernelGGL(decode_small<DT>, dim3(p.U), dim3(kSmallThreads), 0, st, p);
  return SPINDLE_OK;
}
template <int MT>
spindle_status launch_small_f32(const DecodeParams &p, hipStream_t st) {
  static LdsLimit lim;
  if (spindle_status e = allow_lds(lim, reinterpret_cast<const void *>(&decode_small_f32<MT>), kSmallLds)) return e;
  hipLaunchKernelGGL(decode_small_f32<MT>, dim3(p.U), dim3(kSmallThreads), kSmallLds, st, p);
  return SPINDLE_OK;
}
// By the number of tokens: every token slot costs a multiply-add per element of the codebook, used or not.
template <>
spindle_status launch_small<SPINDLE_F32>(const DecodeParams &p, hipStream_t st) {
  if (p.m == 1) return launch_small_f32<1>(p, st);
  if (p.m == 2) return launch_small_f32<2>(p, st);
  return launch_small_f32<4>(p, st);
}

// Enqueues the kernels of one merge; `scratch_mem` has decode_carve's size and needs no
// initial content: every element a kernel reads was written by an earlier kernel of the same call.
spindle_status decode_enqueue(const spindle_kv_desc *desc, const void *X_new, float theta, int32_t max_codes,
                              void *C, int32_t *n_codes, int32_t *n_found, int32_t *n_matched, int32_t *ref,
                              float *mag, void *scratch_mem, hipStream_t st) {
  DecodeParams p;
  p.X = static_cast<const char *>(X_new);
  p.C = static_cast<char *>(C);
  p.n_codes = n_codes;
  p.n_found = n_found;
  p.n_matched = n_matched;
  p.ref = ref;
  p.mag = mag;
  decode_carve(desc, max_codes, scratch_mem, &p);
  p.dtype = desc->dtype;
  p.U = desc->batch * desc->n_kv_heads;
  p.m = desc->seq_len;
  p.cap = max_codes;
  p.theta = (double)theta;
  if (p.m <= 4) {
    ProfScope ps("decode_small", st);
    spindle_status e;
    if (p.dtype == SPINDLE_F16) e = launch_small<SPINDLE_F16>(p, st);
    else if (p.dtype == SPINDLE_BF16) e = launch_small<SPINDLE_BF16>(p, st);
    else e = launch_small<SPINDLE_F32>(p, st);
    if (e != SPINDLE_OK) return e;
    SPINDLE_HIP(hipGetLastError());
    return SPINDLE_OK;
  }
  const dim3 mg((p.m + kMatchTokens - 1) / kMatchTokens * p.slices, p.U);
  const size_t lds = build_lds_words(p.m) * sizeof(uint32_t);
#define SPINDLE_DECODE_LAUNCH(DT)                                                                          \
  do {                                                                                                     \
    static LdsLimit lim, lim_match;                                                                        \
    if (spindle_status e = allow_lds(lim_match, reinterpret_cast<const void *>(&decode_match<DT>),         \
                                     match_lds<DT>()))                                                     \
      return e;                                                                                            \
    if (spindle_status e = allow_lds(lim, reinterpret_cast<const void *>(&decode_build<DT>),               \
                                     build_lds_words(kDecodeMax) * sizeof(uint32_t)))                      \
      return e;                                                                                            \
    {                                                                                                      \
      ProfScope ps("decode_match", st);                                                                    \
      hipLaunchKernelGGL(decode_match<DT>, mg, dim3(kMatchThreads), match_lds<DT>(), st, p);                       \
    }                                                                                                      \
    {                                                                                                      \
      ProfScope ps("decode_build", st);                                                                    \
      hipLaunchKernelGGL(decode_build<DT>, dim3(p.U), dim3(kBuildThreads), lds, st, p);                    \
    }                                                                                                      \
  } while (0)
  if (p.dtype == SPINDLE_F16) SPINDLE_DECODE_LAUNCH(SPINDLE_F16);
  else if (p.dtype == SPINDLE_BF16) SPINDLE_DECODE_LAUNCH(SPINDLE_BF16);
  else SPINDLE_DECODE_LAUNCH(SPINDLE_F32);
#undef SPINDLE_DECODE_LAUNCH
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}

}  // namespace

extern "C" spindle_status spindle_decode_merge(const spindle_kv_desc *desc, const void *X_new, float theta,
                                               int32_t max_codes, void *C, int32_t *n_codes, int32_t *n_found,
                                               int32_t *n_matched, int32_t *ref, float *mag, void *workspace,
                                               size_t workspace_bytes, void *stream) {
  size_t need = 0;
  spindle_status s = decode_check_args(desc, X_new, theta, max_codes, C, n_codes, n_found, ref, mag, &need);
  if (s != SPINDLE_OK) return s;
  if (!workspace) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "workspace is required");
  if (reinterpret_cast<uintptr_t>(workspace) & 15) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "workspace must be 16-byte aligned");
  if (workspace_bytes < need) SPINDLE_FAIL(SPINDLE_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, need);
  return decode_enqueue(desc, X_new, theta, max_codes, C, n_codes, n_found, n_matched, ref, mag, workspace,
                        static_cast<hipStream_t>(stream));
}

namespace {

constexpr int kStaticMaxDevices = 64;
std::mutex g_static_mu;
void *g_static_ptr[kStaticMaxDevices] = {};     // device address of `scratch` on each GPU, once looked up

// Device address of `scratch` on the current device (each GPU holds its own copy of the array
// at its own address).
spindle_status static_scratch(void **out) {
  int dev = 0;
  SPINDLE_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kStaticMaxDevices) SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED, "device %d: at most %d devices", dev, kStaticMaxDevices);
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (!g_static_ptr[dev]) {
    void *ptr = nullptr;
    SPINDLE_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) SPINDLE_FAIL(SPINDLE_ERR_HIP, "hipGetSymbolAddress returned a null address for the scratch array");
    g_static_ptr[dev] = ptr;
  }
  *out = g_static_ptr[dev];
  return SPINDLE_OK;
}

}  // namespace

extern "C" size_t spindle_decode_static_capacity(void) { return kStaticScratchBytes; }

extern "C" spindle_status spindle_decode_merge_static(const spindle_kv_desc *desc, const void *X_new, float theta,
                                                      int32_t max_codes, void *C, int32_t *n_codes, int32_t *n_found,
                                                      int32_t *n_matched, int32_t *ref, float *mag, void *stream) {
  size_t need = 0;
  spindle_status s = decode_check_args(desc, X_new, theta, max_codes, C, n_codes, n_found, ref, mag, &need);
  if (s != SPINDLE_OK) return s;
  if (need > kStaticScratchBytes)
    SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED,
                 "the scratch memory of this call counts %zu bytes (spindle_decode_workspace_bytes), the built-in buffer "
                 "is for calls of up to %zu: fewer new tokens or problems per call, a smaller max_codes, or "
                 "spindle_decode_merge with a workspace",
                 need, kStaticScratchBytes);
  void *mem = nullptr;
  s = static_scratch(&mem);
  if (s != SPINDLE_OK) return s;
  return decode_enqueue(desc, X_new, theta, max_codes, C, n_codes, n_found, n_matched, ref, mag, mem,
                        static_cast<hipStream_t>(stream));
}
