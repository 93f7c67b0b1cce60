// Attention-weight token eviction (Sec. "Attention Weight Based Token Eviction").
//
// Kernels, all enqueued on the caller's stream:
//   deep_stats        window logits by MFMA, per-row softmax statistics of a chunk of keys (Eq. 1)
//   deep_accumulate   merges the per-chunk statistics into max + log2(sum) per query row,
//                     recomputes the logits, forms softmax weights, sums them over the window
//                     queries and the GQA group (Eq. 2, 3)
//   deep_select       max-pool, 4096-bin histogram of the pooled scores over many workgroups
//   deep_finish       the k-th largest score from the histogram and the few scores that share its bin,
//                     the kept positions in order (Eq. 7), K_out = K[kept], V_out = V[kept] (of many or
//                     very long units without the copies)
//   deep_select_unit, deep_gather
//                     the same for shorter contexts: one workgroup per unit, scores and keys in LDS, and
//                     the copies of the rows
//
// Both passes over K stream stages of up to 64 KiB of keys through LDS with direct global->LDS loads
// (two stages, the next one in flight while the current one is multiplied); the 16-byte pieces
// of a row are XOR-swizzled by the row number so that the fragment reads of sixteen
// consecutive rows fall into different banks.
#include <math.h>

#include "common.h"
#include "mma.h"

namespace spindle {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kMaxStagesPerBlock = 16;
constexpr int kBins = 4096;          // histogram over the top 12 bits of the order-preserving score keys

// Staging geometry: KEYS keys per stage, WR waves split the (padded) query rows in groups of 32, the others the 32-key
// tiles of a stage.  Sixteen waves where there are tiles for them: with 32 rows a wave fits 128 registers, and four
// waves per SIMD find each other in different phases, so that the matrix instructions of some run beside the
// exponentials of others (two waves of 64 rows mostly waited in the same one).
template <int DT, int WR, int KEYS>
struct Geo {
  typedef Mma<DT> M;
  static constexpr int kRowBytes = M::kRowBytes;
  static constexpr int kPieces = kRowBytes / 16;                   // 16-byte pieces per key
  static constexpr int kStageKeys = KEYS;
  static constexpr int kStageBytes = kStageKeys * kRowBytes;
  static constexpr int kWaves = WR * (KEYS / 32) < 16 ? WR * (KEYS / 32) : 16;
  static constexpr int kThreads = 64 * kWaves;
  static constexpr int kTiles = kStageKeys / 32;                   // 32-key MFMA tiles per stage
  static constexpr int kRowsPerLoad = 1024 / kRowBytes;            // keys one wave-wide load brings
  static constexpr int kLoadsPerWave = kStageBytes / 1024 / kWaves;

  // Stage of keys key0 .. key0 + kStageKeys - 1 into the LDS buffer at byte address `lds`; keys
  // past the end of the sequence repeat the last one (the callers never use their results).
  static __device__ __forceinline__ void load(const char *Kunit, size_t pitch, int key0, int l, uint32_t lds,
                                              int wave, int lane) {
#pragma unroll
    for (int j = 0; j < kLoadsPerWave; ++j) {
      const int q = wave * kLoadsPerWave + j;
      const int r = q * kRowsPerLoad + lane / kPieces;
      const int piece = (lane % kPieces) ^ (r & (kPieces - 1));
      int key = key0 + r;
      key = key < l ? key : l - 1;
      lds_dma16(Kunit + (size_t)key * pitch + piece * 16, lds + q * 1024);
    }
  }
  // The same for a stage that lies inside the sequence, with this lane's byte offsets within a
  // stage worked out once (`offsets`): a load is then its address registers and nothing else.
  static __device__ __forceinline__ void offsets(size_t pitch, int wave, int lane, uint32_t (&off)[kLoadsPerWave]) {
#pragma unroll
    for (int j = 0; j < kLoadsPerWave; ++j) {
      const int q = wave * kLoadsPerWave + j;
      const int r = q * kRowsPerLoad + lane / kPieces;
      const int piece = (lane % kPieces) ^ (r & (kPieces - 1));
      off[j] = (uint32_t)((size_t)r * pitch + (size_t)piece * 16);
    }
  }
  static __device__ __forceinline__ void load_inside(const char *Kunit, size_t pitch, int key0, uint32_t lds, int wave,
                                                     const uint32_t (&off)[kLoadsPerWave]) {
    const char *base = Kunit + (size_t)key0 * pitch;
#pragma unroll
    for (int j = 0; j < kLoadsPerWave; ++j) lds_dma16_at(base, off[j], lds + (wave * kLoadsPerWave + j) * 1024);
  }
  static constexpr int kFrags = DT == SPINDLE_F32 ? 16 : 8;        // 16-byte pieces of a row per lane group
  // MFMA operand j of staged row `row` for lane group g: one step of a 16-bit type, which is piece 2 j + g; four steps
  // of fp32, dimensions 8 j + 2 i + g, of which two pieces have every second one (a lane group could hold the pieces as
  // they are, but the sums would take the dimensions in another order, and scores of fp32 calls would differ by 2e-6).
  static __device__ __forceinline__ u4 piece(const char *buf, int row, int j, int g) {
    auto at = [&](int q) __attribute__((always_inline)) { return buf + row * kRowBytes + ((q ^ (row & (kPieces - 1))) << 4); };
    if constexpr (DT == SPINDLE_F32) {
      const uint32_t *x = reinterpret_cast<const uint32_t *>(at(2 * j)) + g, *y = reinterpret_cast<const uint32_t *>(at(2 * j + 1)) + g;
      return u4{x[0], x[2], y[0], y[2]};
    } else {
      return *reinterpret_cast<const u4 *>(at(2 * j + g));
    }
  }
  static __device__ __forceinline__ f16v mma(u4 a, u4 b, f16v c) {
    if constexpr (DT == SPINDLE_F32) {
#pragma unroll
      for (int i = 0; i < 4; ++i) c = M::mma(__uint_as_float(a[i]), __uint_as_float(b[i]), c);
      return c;
    } else {
      return M::mma(__builtin_bit_cast(typename M::frag, a), __builtin_bit_cast(typename M::frag, b), c);
    }
  }
  // The wave's 32 query rows (row group wr) into registers, through the second stage buffer.  Everything loaded to LDS
  // before has landed for every wave when this returns, and the buffer is free again.
  static __device__ __forceinline__ void queries(u4 (&qf)[kFrags], const char *Qunit, int R, const char *buf, uint32_t lds, int wr,
                                                 int wave, int lane) {
    constexpr int kAtOnce = 32 * WR < kStageKeys ? 32 * WR : kStageKeys;
#pragma unroll
    for (int q0 = 0; q0 < 32 * WR; q0 += kAtOnce) {
      load_queries(Qunit, q0, kAtOnce, R, lds, wave, lane);
      __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): this wave's part has landed
      __syncthreads();
      if (32 * wr >= q0 && 32 * wr < q0 + kAtOnce)     // wave-uniform
#pragma unroll
        for (int j = 0; j < kFrags; ++j) qf[j] = piece(buf, 32 * wr - q0 + (lane & 31), j, lane >> 5);
      __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): read
      __syncthreads();
    }
  }
  // Query rows q0 .. q0 + n - 1 of a unit of R (the last one again past them) into `lds` as a stage is.
  static __device__ __forceinline__ void load_queries(const char *Qunit, int q0, int n, int R, uint32_t lds, int wave, int lane) {
    for (int q = wave; q < n / kRowsPerLoad; q += kWaves) {
      const int r = q * kRowsPerLoad + lane / kPieces;
      const int piece = (lane % kPieces) ^ (r & (kPieces - 1));
      lds_dma16(Qunit + (size_t)min(q0 + r, R - 1) * kRowBytes + piece * 16, lds + q * 1024);
    }
  }
};

struct DeepParams {
  const char *K;       // [U][l][128] elements
  const char *Q;       // [U][R][128] elements (R = hn*lw rows, head-major)
  float2 *partial;     // [U][nchunks][Rpad] (max, sum) per chunk of keys, logits in base-2 units
  float *scores;       // [U][spitch] group-averaged accumulated attention
  int spitch;          // l_c rounded up to 4
  int *hist;           // [U][kBins] cleared here for deep_select (NULL: not needed)
  int l, lc, lw, hn, R, Rpad, nchunks;
  int stages;          // stages per block
  KvLayout lay;        // rows of K
  float sc2;           // scale * log2(e): logits are kept in base-2 units
  float inv_hn;
  int norm;
};

// (max, sum of exp2(. - max)) of two disjoint sets of logits
__device__ __forceinline__ void merge_stats(float &m, float &z, float m2, float z2) {
  const float mm = fmaxf(m, m2);
  if (mm == -INFINITY) return;                         // both empty
  z = z * __builtin_amdgcn_exp2f(m - mm) + z2 * __builtin_amdgcn_exp2f(m2 - mm);
  m = mm;
}

__device__ __forceinline__ uint32_t lds_address(const void *ptr) {
  return (uint32_t)(size_t)(__attribute__((address_space(3))) const char *)ptr;
}

// Pass 1.  Grid (chunks, units).  The matrix product is taken as keys x
// query rows, so a lane owns one query row (its column of the result) and the sixteen results
// in its registers are sixteen keys: the running (max, sum) of a row is two registers per lane
// and needs no exchange until the end of the block.
template <int DT, int WR, int KEYS>
__global__ __launch_bounds__((Geo<DT, WR, KEYS>::kThreads)) void deep_stats(DeepParams p) {
  typedef Geo<DT, WR, KEYS> S;
  typedef Mma<DT> M;
  constexpr int WK = S::kWaves / WR;
  constexpr int kTilesPerWave = S::kTiles / WK;
  constexpr bool kPrefetch = DT != SPINDLE_F32;        // the 64 one-register fragments of a float tile are read as they are used
  static_assert(kTilesPerWave >= 1, "every wave needs a tile of each stage");
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int u = blockIdx.y, chunk = blockIdx.x;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, c = lane & 31;
  const int wr = wave % WR, wk = wave / WR;
  if (chunk == 0 && p.hist) {                          // counters of this unit's selection
    for (int i = threadIdx.x; i < kBins; i += S::kThreads) p.hist[(size_t)u * kBins + i] = 0;
  }
  const int key_begin = chunk * p.stages * S::kStageKeys;
  int nst = (p.l - key_begin + S::kStageKeys - 1) / S::kStageKeys;
  nst = nst < p.stages ? nst : p.stages;
  const char *Kunit = p.K + kv_unit_offset(p.lay, u);
  const size_t kpitch = (size_t)p.lay.st;
  const char *Qunit = p.Q + (size_t)u * p.R * M::kRowBytes;
  const uint32_t lds0 = lds_address(smem);

  uint32_t koff[S::kLoadsPerWave];
  S::offsets(kpitch, wave, lane, koff);
  const bool narrow = kpitch * S::kStageKeys <= 0xFFFFFFFFull;   // lane offsets within a stage fit 32 bits
  auto stage_load = [&](int key0, uint32_t lds) {
    if (narrow && key0 + S::kStageKeys <= p.l) S::load_inside(Kunit, kpitch, key0, lds, wave, koff);
    else S::load(Kunit, kpitch, key0, p.l, lds, wave, lane);
  };
  stage_load(key_begin, lds0);

  // Query fragments stay in registers for the whole block.  They come through the second stage buffer (fp32: 128
  // rows at a time): read in fragment order, where lanes next to each other have different rows, the 64 KiB of 256
  // rows take a compute unit 4 us.
  u4 qf[S::kFrags];
  S::queries(qf, Qunit, p.R, smem + S::kStageBytes, lds0 + S::kStageBytes, wr, wave, lane);
  const int qrow = 32 * wr + c;
  const int klim = qrow < p.R ? p.lc + qrow % p.lw : -1;   // last key this lane's query row may attend to: query b of the window sits at l_c + b
  float m = -INFINITY, z = 0.f;

  for (int s = 0; s < nst; ++s) {
    const int k0 = key_begin + s * S::kStageKeys;
    if (s + 1 < nst) stage_load(k0 + S::kStageKeys, lds0 + ((s + 1) & 1) * S::kStageBytes);
    const char *buf = smem + (s & 1) * S::kStageBytes;
    const bool tail = k0 + S::kStageKeys > p.lc;       // causal mask / end of the sequence
    // The fragments of a tile are fetched from LDS together, those of the wave's next tile right
    // after the matrix instructions of the current one are issued, so that the LDS latency falls
    // into the vector work on the results (the other wave of the SIMD multiplies meanwhile).
    u4 kf[kPrefetch ? S::kFrags : 1];
    if (kPrefetch && k0 + wk * 32 < p.l) {
#pragma unroll
      for (int j = 0; j < S::kFrags; ++j) kf[kPrefetch ? j : 0] = S::piece(buf, wk * 32 + c, j, g);
    }
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
      const int ct = wk + t * WK;
      const int tk0 = k0 + ct * 32;
      if (tk0 >= p.l) continue;                        // wave-uniform
      f16v acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
      if (kPrefetch) {
#pragma unroll
        for (int j = 0; j < S::kFrags; ++j) acc = S::mma(kf[kPrefetch ? j : 0], qf[j], acc);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < kTilesPerWave && tk0 + WK * 32 < p.l) {
#pragma unroll
          for (int j = 0; j < S::kFrags; ++j) kf[kPrefetch ? j : 0] = S::piece(buf, (ct + WK) * 32 + c, j, g);
        }
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int j = 0; j < S::kFrags; ++j) acc = S::mma(S::piece(buf, ct * 32 + c, j, g), qf[j], acc);
      }
      if (!tail) {
        float hi = acc[0], lo = acc[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) hi = fmaxf(hi, acc[v]);
        if (p.sc2 < 0.f) {                             // uniform; a negative scale turns the order round
#pragma unroll
          for (int v = 1; v < 16; ++v) lo = fminf(lo, acc[v]);
          hi = lo;
        }
        const float mn = fmaxf(m, hi * p.sc2);
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(fmaf(acc[v], p.sc2, -mn));
        z = z * __builtin_amdgcn_exp2f(m - mn) + sum;
        m = mn;
      } else {
        float tv[16];
        float hi = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = tk0 + mma_row(v, g);
          tv[v] = key <= klim && key < p.l ? acc[v] * p.sc2 : -INFINITY;
          hi = fmaxf(hi, tv[v]);
        }
        const float mn = fmaxf(m, hi);
        if (mn > -INFINITY) {
          float sum = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) sum += __builtin_amdgcn_exp2f(tv[v] - mn);
          z = z * __builtin_amdgcn_exp2f(m - mn) + sum;
          m = mn;
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
  }

  // the two lane groups of a wave hold different keys of the same rows; then the WK waves of a
  // row group through LDS, in wave order
  float2 *red = reinterpret_cast<float2 *>(smem);      // [WK][32 * WR]
  {
    const float m2 = __shfl_xor(m, 32), z2 = __shfl_xor(z, 32);
    float mm = g ? m2 : m, zz = g ? z2 : z;            // same operand order in both lane groups
    merge_stats(mm, zz, g ? m : m2, g ? z : z2);
    if (g == 0) red[wk * (32 * WR) + qrow] = make_float2(mm, zz);
  }
  __syncthreads();
  const int row = threadIdx.x;
  if (row < 32 * WR) {
    float2 e = red[row];
#pragma unroll
    for (int j = 1; j < WK; ++j) {
      const float2 o = red[j * (32 * WR) + row];
      merge_stats(e.x, e.y, o.x, o.y);
    }
    p.partial[((size_t)u * p.nchunks + chunk) * p.Rpad + row] = e;
  }
}

// Pass 2.  Grid (chunks of context keys, units).  Here the product is taken as query rows x
// keys: a lane owns one key and its registers hold sixteen query rows, so the sum over the
// window queries and the heads of the group is a sum over the lane's own registers.  The
// weight of (row, key) is exp2(logit - c_row) with c_row = max + log2(sum) of the row.
template <int DT, int WR, int KEYS>
__global__ __launch_bounds__((Geo<DT, WR, KEYS>::kThreads)) void deep_accumulate(DeepParams p) {
  typedef Geo<DT, WR, KEYS> S;
  typedef Mma<DT> M;
  constexpr int WK = S::kWaves / WR;
  constexpr int kTilesPerWave = S::kTiles / WK;
  constexpr bool kPrefetch = DT != SPINDLE_F32;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  float *colpart = reinterpret_cast<float *>(smem + 2 * S::kStageBytes);      // [2][WR][kStageKeys]
  float *row_const = colpart + 2 * WR * S::kStageKeys;                          // [256]

  // The blocks go over the keys from the end, each compute-die's blocks over the ones it had in deep_stats (blocks are
  // dealt round-robin to the 8 dies): what the caches still hold of the last keys read is read first.  24 layers of
  // 8192 tokens, 402 MB of keys: 107 -> 97 us.
  const int nx = gridDim.x, total = nx * gridDim.y, id = blockIdx.y * nx + blockIdx.x;
  const int item = (id & 7) + 8 * ((total - (id & 7) + 7) / 8 - 1 - id / 8);
  const int u = item / nx, chunk = item % nx;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, c = lane & 31;
  const int wr = wave % WR, wk = wave / WR;
  const int key_begin = chunk * p.stages * S::kStageKeys;
  int nst = (p.lc - key_begin + S::kStageKeys - 1) / S::kStageKeys;            // only context keys get a score
  nst = nst < p.stages ? nst : p.stages;
  const char *Kunit = p.K + kv_unit_offset(p.lay, u);
  const size_t kpitch = (size_t)p.lay.st;
  const char *Qunit = p.Q + (size_t)u * p.R * M::kRowBytes;
  const uint32_t lds0 = lds_address(smem);

  uint32_t koff[S::kLoadsPerWave];
  S::offsets(kpitch, wave, lane, koff);
  const bool narrow = kpitch * S::kStageKeys <= 0xFFFFFFFFull;   // lane offsets within a stage fit 32 bits
  auto stage_load = [&](int key0, uint32_t lds) {
    if (narrow && key0 + S::kStageKeys <= p.l) S::load_inside(Kunit, kpitch, key0, lds, wave, koff);
    else S::load(Kunit, kpitch, key0, p.l, lds, wave, lane);
  };
  stage_load(key_begin, lds0);

  // max + log2(sum) of every query row from the per-chunk statistics of the first pass, merged
  // in chunk order by one thread per row (every block of the unit does the same sum in the same
  // order)
  for (int row = threadIdx.x; row < p.Rpad; row += S::kThreads) {
    const float2 *part = p.partial + (size_t)u * p.nchunks * p.Rpad + row;
    float mm = -INFINITY, zz = 0.f;
    for (int ch0 = 0; ch0 < p.nchunks; ch0 += 32) {   // 32 records in flight: one trip for 32 k keys
      float2 e[32];
#pragma unroll
      for (int j = 0; j < 32; ++j) e[j] = ch0 + j < p.nchunks ? part[(size_t)(ch0 + j) * p.Rpad] : make_float2(-INFINITY, 0.f);
#pragma unroll
      for (int j = 0; j < 32; ++j) merge_stats(mm, zz, e[j].x, e[j].y);
    }
    row_const[row] = row < p.R && zz > 0.f ? mm + log2f(zz) : INFINITY;        // rows of the padding weigh nothing
  }

  u4 qf[S::kFrags];
  S::queries(qf, Qunit, p.R, smem + S::kStageBytes, lds0 + S::kStageBytes, wr, wave, lane);   // as in deep_stats
  float cst[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) cst[v] = row_const[32 * wr + mma_row(v, g)];

  for (int s = 0; s < nst; ++s) {
    const int k0 = key_begin + s * S::kStageKeys;
    if (s + 1 < nst) stage_load(k0 + S::kStageKeys, lds0 + ((s + 1) & 1) * S::kStageBytes);
    const char *buf = smem + (s & 1) * S::kStageBytes;
    float *cp = colpart + (s & 1) * (WR * S::kStageKeys);
    u4 kf[kPrefetch ? S::kFrags : 1];    // as in deep_stats
    if (kPrefetch && k0 + wk * 32 < p.lc) {
#pragma unroll
      for (int j = 0; j < S::kFrags; ++j) kf[kPrefetch ? j : 0] = S::piece(buf, wk * 32 + c, j, g);
    }
#pragma unroll
    for (int t = 0; t < kTilesPerWave; ++t) {
      const int ct = wk + t * WK;
      if (k0 + ct * 32 >= p.lc) continue;              // wave-uniform
      f16v acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
      if (kPrefetch) {
#pragma unroll
        for (int j = 0; j < S::kFrags; ++j) acc = S::mma(qf[j], kf[kPrefetch ? j : 0], acc);
        __builtin_amdgcn_sched_barrier(0);
        if (t + 1 < kTilesPerWave && k0 + (ct + WK) * 32 < p.lc) {
#pragma unroll
          for (int j = 0; j < S::kFrags; ++j) kf[kPrefetch ? j : 0] = S::piece(buf, (ct + WK) * 32 + c, j, g);
        }
        __builtin_amdgcn_sched_barrier(0);
      } else {
#pragma unroll
        for (int j = 0; j < S::kFrags; ++j) acc = S::mma(qf[j], S::piece(buf, ct * 32 + c, j, g), acc);
      }
      float cs0 = 0.f, cs1 = 0.f;
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        cs0 += __builtin_amdgcn_exp2f(fmaf(acc[v], p.sc2, -cst[v]));
        cs1 += __builtin_amdgcn_exp2f(fmaf(acc[v + 1], p.sc2, -cst[v + 1]));
      }
      // the other sixteen rows of each block of 32 sit in the other lane group
      const uint32_t csb = __float_as_uint(cs0 + cs1);
      const auto both = __builtin_amdgcn_permlane32_swap(csb, csb, false, false);   // [0]: group 0's value, [1]: group 1's
      if (g == 0) cp[wr * S::kStageKeys + ct * 32 + c] = __uint_as_float(both[0]) + __uint_as_float(both[1]);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    for (int i = threadIdx.x; i < S::kStageKeys; i += S::kThreads) {   // fixed-order sum over the row groups
      const int a = k0 + i;
      if (a < p.lc) {
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < WR; ++j) sum += cp[j * S::kStageKeys + i];
        float v = sum * p.inv_hn;
        if (p.norm == SPINDLE_NORM_PAPER) v = v / (float)(p.l - a);
        p.scores[(size_t)u * p.spitch + a] = v;
      }
    }
  }
}

// ---------------------------------------------------------------- pool + top-k
struct SelectParams {
  const float *scores;   // [U][spitch]
  uint32_t *pooled;      // [U][lc] pooled scores as order-preserving keys
  float *scores_out;     // optional [U][lc]
  int *hist;             // [U][kBins], zero on entry
  const int32_t *budgets;
  int32_t *kept;         // [U][out_stride]
  int l, lc, lw, pool, budget, out_stride;
  int nfinish;           // workgroups per unit of deep_finish
  int spitch;            // floats per unit of `scores`, a multiple of 4
};

struct GatherParams {
  const char *K, *V;
  char *Ko, *Vo;
  const int32_t *kept;
  int l, out_stride, row_bytes;
  KvLayout lay;        // rows of K and V
};

// How many context tokens unit u keeps.
__device__ __forceinline__ int kept_context(const SelectParams &p, int u) {
  int budget = p.budgets ? p.budgets[u] : p.budget;
  if (budget < p.lw) budget = p.lw;
  int k = budget - p.lw;
  if (k > p.lc) k = p.lc;
  if (k > p.out_stride - p.lw) k = p.out_stride - p.lw;   // never write past the row pitch
  return k;
}

constexpr int kSelThreads = 1024;
constexpr int kSegLen = 2048;        // context positions per workgroup
constexpr int kHaloMax = 256;        // pooling radius up to which the raw scores of a segment sit in LDS
constexpr int kCandMax = 8192;       // scores sharing the threshold's bin that are ranked in LDS
constexpr int kRunsMax = 1024;       // runs that deep_finish counts apart
constexpr int kWaves = kSelThreads / 64, kBatch = 32;   // of deep_finish, steps of 64 keys that a wave has in flight
constexpr int kOneTripMax = kWaves * 64 * kBatch;

// base + how many of the bits are those of lanes below this one.
__device__ __forceinline__ int lanes_below(unsigned long long bits, int base) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bits >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bits, (uint32_t)base));
}

__device__ __forceinline__ uint32_t orderable(float f) {
  const uint32_t b = __float_as_uint(f);
  return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

// Counts, from the top, the digits of the keys `src[0 .. nsrc)` that match `prefix` above
// `bits_left`, and narrows (prefix, krem) by one digit of width w: afterwards the krem-th
// largest matching key still matches.  All threads of the block call it with the same arguments.
// Digits of ten bits where the keys may be in memory: two passes over them for 20 bits, not three (one unit of 524256 positions of which 100000
// are kept 349 us with digits of eight, 306 now, with scores that all tie 431 and 339); over those in LDS it is the same.
template <int kDigitBits>
__device__ void radix_step(const uint32_t *src, int nsrc, uint32_t &prefix, int &krem, int &bits_left, int *hist,
                           uint32_t *sh_prefix, int *sh_krem) {
  const int tid = threadIdx.x, lane = lane_id();
  const int w = bits_left < kDigitBits ? bits_left : kDigitBits, shift = bits_left - w;
  const uint32_t dmask = (1u << w) - 1u;
  static_assert(1 << kDigitBits <= kSelThreads, "a counter per thread");
  if (tid < 1 << kDigitBits) hist[tid] = 0;
  __syncthreads();
  constexpr int kAtOnce = 4;                           // independent keys per thread and trip
  for (int a0 = 0; a0 < nsrc; a0 += kAtOnce * kSelThreads) {
    uint32_t x[kAtOnce];
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const int a = a0 + q * kSelThreads + tid;
      x[q] = a < nsrc ? src[a] : 0u;
    }
#pragma unroll
    for (int q = 0; q < kAtOnce; ++q) {
      const int a = a0 + q * kSelThreads + tid;
      const bool in = a < nsrc && (bits_left == 32 || (x[q] >> bits_left) == (prefix >> bits_left));
      const int d = (int)((x[q] >> shift) & dmask);
      if (in) {
        // keys crowd into few digits: the digit of the first lane that takes part is counted
        // once for all lanes that share it
        const int d0 = __builtin_amdgcn_readfirstlane(d);
        const unsigned long long same = __ballot(d == d0);
        if (d != d0) atomicAdd(&hist[d], 1);
        else if (lane == __builtin_ctzll(same)) atomicAdd(&hist[d0], __popcll(same));
      }
    }
  }
  __syncthreads();
  if (tid < 64) {
    // lane t owns kPer counters; find the digit at which the count from the top reaches krem
    constexpr int kPer = (1 << kDigitBits) / 64;
    int hh[kPer], mine = 0;
#pragma unroll
    for (int j = 0; j < kPer; j += 4) {
      const int4 h = *reinterpret_cast<const int4 *>(hist + kPer * tid + j);
      hh[j] = h.x; hh[j + 1] = h.y; hh[j + 2] = h.z; hh[j + 3] = h.w;
      mine += h.x + h.y + h.z + h.w;
    }
    int above = mine;                                  // inclusive sum over lanes >= t
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int x = __shfl_down(above, o);
      if (tid + o < 64) above += x;
    }
    above -= mine;                                     // keys in counters of higher lanes
    int run = above;
#pragma unroll
    for (int j = kPer - 1; j >= 0; --j) {
      if (run < krem && krem <= run + hh[j]) {
        *sh_prefix = prefix | ((uint32_t)(kPer * tid + j) << shift);
        *sh_krem = krem - run;
      }
      run += hh[j];
    }
  }
  __syncthreads();
  prefix = *sh_prefix;
  krem = *sh_krem;
  bits_left = shift;
  __syncthreads();
}

// One workgroup per unit, everything on chip: the raw scores go to LDS, a lane pools four neighbouring positions at a
// time and puts their keys in the place of the scores; histogram of the top 12 bits, the k-th largest among the keys
// of its bin by comparing all of them, ordered compaction.
// Bound by latency and by the instructions of one compute unit; loops stay rolled, since a cold kernel also waits for
// its code (36 KB of it, unrolled with the keys in registers: 1.5 to 3 us more).  The segments of a unit over several
// workgroups (deep_select and deep_finish, which copies the rows as well) against this and deep_gather, the eviction call, us:
// one unit of 480 positions 24 and 18, eight of 4080 30 and 23, of 8176 32 and 28, of 12272 33 and 32, of 16368 36 and 35, one of
// 16368 31 and 30, 32 of 16368 67 and 67, 192 of 8176 201 and 187 (random keys; with scores that all tie 26 and 20, 31 and 23, 36 and
// 30, 40 and 35, 46 and 41, 42 and 38, 77 and 73, 204 and 188).
constexpr int kUnitMax = 16384, kUnitRadius = 8;
constexpr int kUnitStep = 4 * kSelThreads;             // positions of the workgroup per step
constexpr int kUnitLoads = kUnitMax / kUnitStep;
// Keys of one bin that are ranked by comparing all of them; more by radix passes over the unit's keys, 2 us or so.  Comparing a
// thousand takes 30: 8 units of 12272 positions with random scores 66 us up to 1024 and 33 up to 128, 32 of 16368 114 and 70, one
// of 2032 (a few more than 128) 23.7 up to 256 and 20.6.
constexpr int kUnitRank = 128;
constexpr int kCopies = 4;                             // of the histogram, by lane, so that equal digits collide less;
constexpr int kCopyPitch = kBins + 8;                  // in other banks
__host__ __device__ inline int unit_raw(int lc) { return (lc + kUnitStep - 1) / kUnitStep * kUnitStep + 2 * kUnitRadius; }
inline size_t unit_lds(int lc) { return ((size_t)unit_raw(lc) + kCopies * kCopyPitch) * sizeof(int); }

__global__ __launch_bounds__(kSelThreads) void deep_select_unit(SelectParams p) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ __attribute__((aligned(16))) uint32_t cand[kUnitRank + 4];
  __shared__ int wtotal[2][kSelThreads / 64];
  __shared__ __attribute__((aligned(16))) int hist256[256];
  __shared__ uint32_t sh_prefix;
  __shared__ int sh_krem, sh_ncand;
  constexpr int kWaves = kSelThreads / 64;
  const int u = blockIdx.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6, lc = p.lc;
  const float *raw = p.scores + (size_t)u * p.spitch;
  const int steps = (lc + kUnitStep - 1) / kUnitStep, run = steps * 256;   // of 256 positions; of a wave
  const int w0 = wave * run + 4 * lane;                // step i of a lane: positions w0 + 256 i ..
  float *rawl = reinterpret_cast<float *>(smem) + kUnitRadius;   // scores, then keys, by position; kUnitRadius more at both ends
  uint32_t *keys = reinterpret_cast<uint32_t *>(rawl);
  int *hist = reinterpret_cast<int *>(smem) + unit_raw(lc);
  {
    float4 v[kUnitLoads];
#pragma unroll
    for (int i = 0; i < kUnitLoads; ++i)
      if (i < steps && w0 + 256 * i < lc) v[i] = *reinterpret_cast<const float4 *>(raw + w0 + 256 * i);
    for (int i = tid; i < kCopies * kCopyPitch / 4; i += kSelThreads) reinterpret_cast<int4 *>(hist)[i] = make_int4(0, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < kUnitLoads; ++i)
      if (i < steps) {
        const int left = lc - (w0 + 256 * i);          // positions that exist
        v[i].x = left < 1 ? -INFINITY : v[i].x;
        v[i].y = left < 2 ? -INFINITY : v[i].y;
        v[i].z = left < 3 ? -INFINITY : v[i].z;
        v[i].w = left < 4 ? -INFINITY : v[i].w;
        *reinterpret_cast<float4 *>(rawl + w0 + 256 * i) = v[i];
      }
  }
  if (tid < kUnitRadius) rawl[tid - kUnitRadius] = rawl[kWaves * run + tid] = -INFINITY;
  if (tid == 0) sh_ncand = 0;
  const int k = kept_context(p, u), r = (p.pool - 1) / 2;
  int32_t *kept = p.kept + (size_t)u * p.out_stride;
  __syncthreads();

  // Pooling in place: a step is read before the one in front of it is written, and what the neighbouring waves write
  // is read before the barrier.
  {
    float4 f[5];                                       // positions a - 8 .. a + 11
    const float4 end0 = *reinterpret_cast<const float4 *>(rawl + (wave + 1) * run), end1 = *reinterpret_cast<const float4 *>(rawl + (wave + 1) * run + 4);
    auto read = [&](int i) __attribute__((always_inline)) {
      const float *at = rawl + w0 + 256 * i;
      f[2] = *reinterpret_cast<const float4 *>(at);
      if (r > 0) {                                     // uniform, as below
        f[1] = *reinterpret_cast<const float4 *>(at - 4);
        f[3] = *reinterpret_cast<const float4 *>(at + 4);
      }
      if (r > 4) {
        f[0] = *reinterpret_cast<const float4 *>(at - 8);
        f[4] = *reinterpret_cast<const float4 *>(at + 8);
      }
      if (i == steps - 1) {                            // (the next wave may have written there)
        if (lane == 63) { f[3] = end0; f[4] = end1; }
        if (lane == 62) f[4] = end0;
      }
    };
    read(0);
    __syncthreads();
    const bool wide = p.scores_out && (lc & 3) == 0 && (reinterpret_cast<uintptr_t>(p.scores_out) & 15) == 0;
    int *own = hist + (lane & (kCopies - 1)) * kCopyPitch;
#pragma unroll 1
    for (int i = 0; i < steps; ++i) {
      const int a = w0 + 256 * i;
      const float *v = reinterpret_cast<const float *>(f);
      float mx[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) mx[j] = fmaxf(-INFINITY, v[8 + j]);
#pragma unroll
      for (int d = 1; d <= kUnitRadius; ++d)
        if (d <= r) {
#pragma unroll
          for (int j = 0; j < 4; ++j) mx[j] = fmaxf(mx[j], fmaxf(v[8 + j - d], v[8 + j + d]));
        }
      u4 x;                                            // 0 past the end
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = a + j < lc ? orderable(mx[j]) : 0u;
      if (wide) {
        if (a < lc) *reinterpret_cast<float4 *>(p.scores_out + (size_t)u * lc + a) = make_float4(mx[0], mx[1], mx[2], mx[3]);
      } else if (p.scores_out) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (a + j < lc) p.scores_out[(size_t)u * lc + a + j] = mx[j];
      }
      int n = 1;                                       // pooled neighbours are often equal: one addition for a run of them
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j < 3 && x[j] >> 20 == x[j < 3 ? j + 1 : 3] >> 20) {
          ++n;
        } else {
          if (x[j]) atomicAdd(&own[x[j] >> 20], n);
          n = 1;
        }
      }
      if (i + 1 < steps) read(i + 1);
      // every lane's reads in front of any lane's store, and the store in front of later reads: LDS keeps the order of one
      // wave's accesses, the fences (no instruction) keep the compiler from changing it
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      *reinterpret_cast<u4 *>(keys + a) = x;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  }
  for (int b = tid; b < p.lw; b += kSelThreads) kept[k + b] = lc + b;
  for (int j = k + p.lw + tid; j < p.out_stride; j += kSelThreads) kept[j] = -1;
  if (k == 0) return;
  if (k >= lc) {
    for (int a = tid; a < lc; a += kSelThreads) kept[a] = a;
    return;
  }
  __syncthreads();

  // threshold bin: thread t owns four bins, from the top, so that counts add up along the threads
  {
    const int bin0 = kBins - 4 - 4 * tid;
    int4 h = make_int4(0, 0, 0, 0);
    for (int c = 0; c < kCopies; ++c) {
      const int4 y = *reinterpret_cast<const int4 *>(hist + c * kCopyPitch + bin0);
      h.x += y.x; h.y += y.y; h.z += y.z; h.w += y.w;
    }
    const int hh[4] = {h.w, h.z, h.y, h.x}, mine = h.x + h.y + h.z + h.w, incl = lanes_up_to(mine);
    if (lane == 63) wtotal[0][wave] = incl;
    __syncthreads();
    int seen = incl - mine;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) seen += w < wave ? wtotal[0][w] : 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (seen < k && k <= seen + hh[j]) {
        sh_prefix = (uint32_t)(bin0 + 3 - j) << 20;
        sh_krem = k - seen;
      }
      seen += hh[j];
    }
  }
  __syncthreads();
  uint32_t prefix = sh_prefix;                         // to become the key of the k-th largest pooled score
  int krem = sh_krem;                                  // how many keys equal to it are taken
  const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll 1
  for (int i = 0; i < steps; ++i) {
    const u4 x = *reinterpret_cast<const u4 *>(keys + w0 + 256 * i);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = x[j] >> 20 == prefix >> 20 && x[j] != 0;
      const unsigned long long mk = __ballot(in);
      if (mk) {                                        // wave-uniform
        int at = 0;
        if (lane == __builtin_ctzll(mk)) at = atomicAdd(&sh_ncand, __popcll(mk));
        at = __shfl(at, __builtin_ctzll(mk)) + __popcll(mk & below);
        if (in && at < kUnitRank) cand[at] = x[j];
      }
    }
  }
  __syncthreads();
  const int ncand = sh_ncand;
  if (ncand <= kUnitRank) {
    if (wave * 64 < ncand) {
      const uint32_t own = tid < ncand ? cand[tid] : 0u;
      int gt = 0, eq = 0;
      for (int j = 0; j < ncand; j += 4) {
        const u4 y = *reinterpret_cast<const u4 *>(cand + j);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          gt += j + q < ncand && y[q] > own;
          eq += j + q < ncand && y[q] == own;
        }
      }
      if (tid < ncand && gt < krem && krem <= gt + eq) {
        sh_prefix = own;
        sh_krem = krem - gt;
      }
    }
    __syncthreads();
    prefix = sh_prefix;
    krem = sh_krem;
  } else {
    int bits_left = 20;
    while (bits_left > 0) radix_step<8>(keys, kWaves * run, prefix, krem, bits_left, hist256, &sh_prefix, &sh_krem);
  }

  // ordered compaction: everything above the threshold, then the first `krem` equal to it; both counts in one word
  auto count = [&](const u4 &x) __attribute__((always_inline)) {
    int n = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) n += (x[j] > prefix ? 1 << 16 : 0) + (x[j] == prefix ? 1 : 0);
    return n;
  };
  int total = 0;
#pragma unroll 1
  for (int i = 0; i < steps; ++i) total += count(*reinterpret_cast<const u4 *>(keys + w0 + 256 * i));
  total = lanes_up_to(total);
  if (lane == 63) wtotal[1][wave] = total;
  __syncthreads();
  int gt_seen = 0, eq_seen = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    gt_seen += w < wave ? wtotal[1][w] >> 16 : 0;
    eq_seen += w < wave ? wtotal[1][w] & 0xFFFF : 0;
  }
#pragma unroll 1
  for (int i = 0; i < steps; ++i) {
    const u4 x = *reinterpret_cast<const u4 *>(keys + w0 + 256 * i);
    const int own = count(x), incl = lanes_up_to(own);
    int gt = gt_seen + ((incl - own) >> 16), eq = eq_seen + ((incl - own) & 0xFFFF);
    if (own)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (x[j] > prefix) {
          kept[gt + (eq < krem ? eq : krem)] = w0 + 256 * i + j;
          ++gt;
        } else if (x[j] == prefix) {
          if (eq < krem) kept[gt + eq] = w0 + 256 * i + j;
          ++eq;
        }
      }
    const int all = __builtin_amdgcn_readlane(incl, 63);
    gt_seen += all >> 16;
    eq_seen += all & 0xFFFF;
  }
}

// Units of more than kUnitMax context positions or pooled over more than 2 kUnitRadius + 1 of them, grid (segments, units)
// of two launches.  In the first every workgroup pools its segment of the raw scores, stores the pooled scores as keys and
// adds its 4096-bin histogram to the unit's.
__global__ __launch_bounds__(kSelThreads) void deep_select(SelectParams p) {
  __shared__ float rawl[kSegLen + 2 * kHaloMax];
  __shared__ int hist[kBins];
  const int seg = blockIdx.x, u = blockIdx.y, tid = threadIdx.x, lane = lane_id();
  const int lc = p.lc;
  const float *raw = p.scores + (size_t)u * p.spitch;
  uint32_t *pooled = p.pooled + (size_t)u * lc;
  int *ghist = p.hist + (size_t)u * kBins;

  for (int i = tid; i < kBins; i += kSelThreads) hist[i] = 0;
  const int a_begin = seg * kSegLen;
  const int a_end = a_begin + kSegLen < lc ? a_begin + kSegLen : lc;
  const int r = (p.pool - 1) / 2;
  const bool in_lds = r <= kHaloMax;
  const int h_begin = a_begin - r < 0 ? 0 : a_begin - r;
  const int h_end = a_end + r > lc ? lc : a_end + r;
  if (in_lds)
    for (int a = h_begin + tid; a < h_end; a += kSelThreads) rawl[a - h_begin] = raw[a];
  __syncthreads();
  for (int a = a_begin + tid; a < a_end; a += kSelThreads) {
    const int lo = a - r < 0 ? 0 : a - r, hi = a + r >= lc ? lc - 1 : a + r;
    float mx = -INFINITY;
    if (in_lds) for (int j = lo; j <= hi; ++j) mx = fmaxf(mx, rawl[j - h_begin]);
    else for (int j = lo; j <= hi; ++j) mx = fmaxf(mx, raw[j]);
    const uint32_t x = orderable(mx);
    pooled[a] = x;
    if (p.scores_out) p.scores_out[(size_t)u * lc + a] = mx;
    const int d = (int)(x >> 20);
    const int d0 = __builtin_amdgcn_readfirstlane(d);
    const unsigned long long same = __ballot(d == d0);
    if (d != d0) atomicAdd(&hist[d], 1);
    else if (lane == __builtin_ctzll(same)) atomicAdd(&hist[d0], __popcll(same));
  }
  __syncthreads();
  for (int i = tid; i < kBins; i += kSelThreads) {
    const int v = hist[i];
    if (v) __hip_atomic_fetch_add(&ghist[i], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Every workgroup works out what the whole unit's selection comes to, threshold bin from the histogram, exact value of the
// k-th largest key among the keys of that bin, then writes its share of the kept positions, as many as every other, and copies
// their rows of K and V.  (By segments of the context, the one that holds most of what is kept copies it alone: the divisor of
// Eq. 3 has similar keys keep the end of the context.  Calls that keep 2048 random keys, 8 units of 32736 positions 64 us by segments and 48
// by shares, 32 units 156 and 118; without the divisor, positions all over, 48 and 50, 126 and 118.)
// Bound by latency.  The keys are read once: where a run's kept positions start follows from how many of it are above the bin
// and from those in the bin, which are in LDS by run, and only the runs that hold some of the share are looked at again (three
// reads: 8 units of 131040 positions 143 us, now 119, one of 524256 231, now 128).
// Ranking the keys of the bin by comparing all of them, as deep_select_unit does, takes 40 us where there are a thousand.
// Where the workgroups of all units would not run at once (finish_blocks), one per unit selects and deep_gather copies (kCopies = false).
template <bool kCopies, bool kOneTrip>
__global__ __launch_bounds__(kSelThreads) void deep_finish(SelectParams p, GatherParams q) {
  __shared__ __attribute__((aligned(16))) int hist[1024];
  __shared__ __attribute__((aligned(16))) uint32_t cand[kCandMax];
  __shared__ int wsum[kWaves], run_gt[kRunsMax], run_eq[kRunsMax];
  __shared__ uint32_t sh_prefix;
  __shared__ int sh_krem, sh_ncand;
  const int blk = blockIdx.x, u = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int lc = p.lc;
  const uint32_t *pooled = p.pooled + (size_t)u * lc;
  const int *ghist = p.hist + (size_t)u * kBins;
  int32_t *kept = p.kept + (size_t)u * p.out_stride;
  const int k = kept_context(p, u);
  const int share = (k + p.nfinish - 1) / p.nfinish;   // (kCopies: kCandMax at most)
  const int r0 = min(k, blk * share), r1 = min(k, r0 + share);   // the workgroup's kept positions

  // The unit's keys in runs, dealt to the waves in turn: of thirty-two steps of 64 positions, all loads of which are in flight
  // together, or a few times that, and shorter ones where every wave has one: then its keys stay in registers for all uses.
  const int run = kOneTrip ? (((lc + kWaves - 1) / kWaves) + 63) & ~63 : 64 * kBatch * ((lc - 1) / (64 * kBatch * kRunsMax) + 1);
  const int nruns = (lc + run - 1) / max(run, 1);
  uint32_t x[kBatch];
  auto load_keys = [&](int b0, int end) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kBatch; ++i) {
      const int a = b0 + 64 * i + lane;
      x[i] = a < end ? pooled[a] : 0u;
    }
  };
  uint32_t prefix = 0;                                 // key of the k-th largest pooled score
  int krem = k;                                        // how many keys equal to it are taken
  uint32_t *mine = cand;                               // [share] positions r0 .. r1 - 1, behind the candidates' last use
  if (k > 0 && k < lc) {
    if (kOneTrip) load_keys(wave * run, min(lc, (wave + 1) * run));
    // threshold bin: thread t owns four bins, from the top, so that counts add up along the threads
    {
      const int bin0 = kBins - 4 - 4 * tid;
      const int4 h = *reinterpret_cast<const int4 *>(ghist + bin0);
      const int hh[4] = {h.w, h.z, h.y, h.x}, own = h.x + h.y + h.z + h.w, incl = lanes_up_to(own);
      if (lane == 63) wsum[wave] = incl;
      __syncthreads();
      int seen = incl - own;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) seen += w < wave ? wsum[w] : 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (seen < k && k <= seen + hh[j]) {
          sh_prefix = (uint32_t)(bin0 + 3 - j) << 20;
          sh_krem = k - seen;
        }
        seen += hh[j];
      }
      if (tid == 0) sh_ncand = 0;
      __syncthreads();
      prefix = sh_prefix;
      krem = sh_krem;
    }
    // First use: the keys of the threshold's bin, ranked in LDS when they fit (a few hundred as a rule), else where they are,
    // those of a run together; and how many of a run are in higher bins.
    const uint32_t last = prefix | 0xFFFFFu;           // of the bin
    for (int r = wave; r < nruns; r += kWaves) {
      const int end = min(lc, (r + 1) * run);
      int above = 0, at = 0, n = 0;
      for (int b0 = r * run; b0 < end; b0 += 64 * kBatch) {
        if (!kOneTrip) load_keys(b0, end);
        int own = 0, higher = 0;                       // (keys past the end are 0, in the lowest bin, which no score has)
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          higher += x[i] > last;
          own += x[i] >= prefix;
        }
        own -= higher;
        const int incl = lanes_up_to(higher << 16 | own), all = __builtin_amdgcn_readlane(incl, 63);
        n = all & 0xFFFF;
        above += all >> 16;
        if (n) {
          if (lane == 0) at = atomicAdd(&sh_ncand, n);
          at = __builtin_amdgcn_readfirstlane(at);
          int to = at + (incl & 0xFFFF) - own;
          if (own)
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
              if (x[i] - prefix <= 0xFFFFFu) {
                if (to < kCandMax) cand[to] = x[i];
                ++to;
              }
        }
        if (kOneTrip) break;
      }
      if (lane == 0) {
        run_gt[r] = above;
        run_eq[r] = (int)((uint32_t)at << 12 | (uint32_t)n);   // where they are, if all fit and the run is one trip
      }
      if (kOneTrip) break;
    }
    __syncthreads();
    const int ncand = sh_ncand;
    const uint32_t *src = ncand <= kCandMax ? cand : pooled;
    const int nsrc = ncand <= kCandMax ? ncand : lc;
    int bits_left = 20;
    while (bits_left > 0) radix_step<10>(src, nsrc, prefix, krem, bits_left, hist, &sh_prefix, &sh_krem);
    // ordered compaction: everything above the threshold, the first `krem` equal to it.  Counts of the runs first, of all of them
    // from their candidates where these are in LDS, else of 64 at a time up to the last that the workgroup needs;
    const bool listed = ncand <= kCandMax && run <= 64 * kBatch && prefix != 0;
    int gt_before = 0, eq_before = 0;
    for (int s0 = 0; s0 < nruns; ) {
      const int s1 = listed ? nruns : min(nruns, s0 + 64);
      for (int r = s0 + wave; r < s1; r += kWaves) {
        int ngt = 0, neq = 0;
        if (listed) {
          const uint32_t rec = (uint32_t)run_eq[r];
          const int at = (int)(rec >> 12), n = (int)(rec & 0xFFFu);
          for (int i = lane; i < n; i += 64) {
            ngt += cand[at + i] > prefix;
            neq += cand[at + i] == prefix;
          }
        } else {
          const int end = min(lc, (r + 1) * run);
          for (int b0 = r * run; b0 < end; b0 += 64 * kBatch) {
            if (!kOneTrip) load_keys(b0, end);
            int here = b0 + lane;
            asm("" : "+v"(here));                      // (the comparisons of the loads are not kept in 64 scalar registers)
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
              const bool in = here + 64 * i < end;
              ngt += in && x[i] > prefix;
              neq += in && x[i] == prefix;
            }
            if (kOneTrip) break;
          }
        }
        ngt = lanes_up_to(ngt);
        neq = lanes_up_to(neq);
        if (lane == 63) {
          run_gt[r] = (listed ? run_gt[r] : 0) + ngt;
          run_eq[r] = neq;
        }
        if (kOneTrip) break;
      }
      __syncthreads();
      // then the places of those runs that hold some of the workgroup's own, by ballots over 64 positions.
      for (int c0 = s0; c0 < s1; c0 += 64) {
        const int g = c0 + lane < s1 ? run_gt[c0 + lane] : 0, e = c0 + lane < s1 ? run_eq[c0 + lane] : 0;
        const int ig = lanes_up_to(g) + gt_before, ie = lanes_up_to(e) + eq_before;   // with the run itself
        const int from = ig - g + min(ie - e, krem), to = ig + min(ie, krem);
        unsigned long long todo = __ballot(from < to && from < r1 && to > r0) & (0x0001000100010001ull << wave);
        static_assert(kWaves == 16, "every sixteenth run is the wave's");
        for (; todo; todo &= todo - 1) {
          const int nth = __builtin_ctzll(todo), r = c0 + nth, end = min(lc, (r + 1) * run);
          const int gt0 = __builtin_amdgcn_readlane(ig - g, nth), eq0 = __builtin_amdgcn_readlane(ie - e, nth);
          const int eq1 = __builtin_amdgcn_readlane(ie, nth);
          // (of the keys equal to the threshold a run has all taken, or none, but for one run)
          const bool some = prefix + 1u <= 1u || (eq0 < krem && eq1 > krem);
          const uint32_t least = prefix + (eq0 >= krem);
          int seen = gt0 + min(eq0, krem) - r0, eq_seen = eq0;
          for (int b0 = r * run; b0 < end; b0 += 64 * kBatch) {
            if (!kOneTrip) load_keys(b0, end);
            int here = b0 + lane;
            asm("" : "+v"(here));
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
              const int a = here + 64 * i;
              bool take = x[i] >= least;
              if (some) {
                const bool eq = a < end && x[i] == prefix;
                const unsigned long long meq = __ballot(eq);
                take = x[i] > prefix || (eq && lanes_below(meq, eq_seen) < krem);
                eq_seen += __popcll(meq);
              }
              const unsigned long long taken = __ballot(take);
              const int at = lanes_below(taken, seen);
              if (take && (unsigned)at < (unsigned)(r1 - r0)) {
                if (kCopies) mine[at] = (uint32_t)a;
                else kept[r0 + at] = a;
              }
              seen += __popcll(taken);
            }
            if (kOneTrip) break;
          }
          if (kOneTrip) break;
        }
        if (kOneTrip) break;
        gt_before = __builtin_amdgcn_readlane(ig, 63);
        eq_before = __builtin_amdgcn_readlane(ie, 63);
      }
      s0 = s1;
      if (kOneTrip || gt_before + min(eq_before, krem) >= r1) break;
    }
  } else {
    for (int i = tid; i < r1 - r0; i += kSelThreads) {
      if (kCopies) mine[i] = (uint32_t)(r0 + i);
      else kept[r0 + i] = r0 + i;
    }
  }
  if constexpr (!kCopies) {
    for (int b = tid; b < p.out_stride - k; b += kSelThreads) kept[k + b] = b < p.lw ? lc + b : -1;
    return;
  }
  __syncthreads();
  // their rows, and of the window and the padding behind the kept positions the workgroup's share
  const int tpr = q.row_bytes / 16, per = kSelThreads / tpr, t = tid % tpr;
  const size_t in = kv_unit_offset(q.lay, u) + t * 16, out = (size_t)u * p.out_stride * q.row_bytes + t * 16;
  const int nkept = r1 - r0, behind = p.out_stride - k, share_behind = (behind + p.nfinish - 1) / p.nfinish;
  const int nbehind = max(0, min(behind - blk * share_behind, share_behind));
  for (int i0 = tid / tpr; i0 < nkept + nbehind; i0 += 2 * per) {
    u4 kv[2], vv[2];
    int to[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int i = i0 + j * per;
      to[j] = -1;
      kv[j] = vv[j] = u4{0, 0, 0, 0};
      if (i >= nkept + nbehind) continue;
      int idx;
      if (i < nkept) {
        to[j] = r0 + i;
        idx = (int)mine[i];
      } else {
        const int b = blk * share_behind + i - nkept;  // of the window, then of the padding
        to[j] = k + b;
        idx = b < p.lw ? lc + b : -1;
      }
      if (t == 0) kept[to[j]] = idx;
      if (idx >= 0) {
        kv[j] = *reinterpret_cast<const u4 *>(q.K + in + (size_t)idx * (size_t)q.lay.st);
        if (q.V) vv[j] = *reinterpret_cast<const u4 *>(q.V + in + (size_t)idx * (size_t)q.lay.st);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (to[j] >= 0) {
        *reinterpret_cast<u4 *>(q.Ko + out + (size_t)to[j] * q.row_bytes) = kv[j];
        if (q.Vo) *reinterpret_cast<u4 *>(q.Vo + out + (size_t)to[j] * q.row_bytes) = vv[j];
      }
  }
}

// ---------------------------------------------------------------- gather
__global__ __launch_bounds__(256) void deep_gather(GatherParams p) {
  const int tpr = p.row_bytes / 16;
  const int rows_per_block = 256 / tpr;
  const int u = blockIdx.y;
  const int j = blockIdx.x * rows_per_block + threadIdx.x / tpr;
  const int t = threadIdx.x % tpr;
  if (j >= p.out_stride) return;
  const int idx = p.kept[(size_t)u * p.out_stride + j];
  const size_t dst = ((size_t)u * p.out_stride + j) * p.row_bytes + t * 16;
  const size_t src = kv_unit_offset(p.lay, u) + (size_t)(idx < 0 ? 0 : idx) * (size_t)p.lay.st + t * 16;
  u4 kv = {0, 0, 0, 0}, vv = {0, 0, 0, 0};
  if (idx >= 0) {
    kv = *reinterpret_cast<const u4 *>(p.K + src);
    if (p.V) vv = *reinterpret_cast<const u4 *>(p.V + src);
  }
  *reinterpret_cast<u4 *>(p.Ko + dst) = kv;
  if (p.Vo) *reinterpret_cast<u4 *>(p.Vo + dst) = vv;
}

// ---------------------------------------------------------------- host side
struct DeepLayout {
  float2 *partial;
  float *scores;
  uint32_t *pooled;
  int *hist;
  int keys, stages, nchunks;   // keys per stage, stages per block
  size_t bytes;
};

// Keys per stage and stages per block: whatever ends first if 256 blocks run at a time.  A stage of 64 KiB takes about
// 3.4 us, whatever its size some 0.1 of that more (the barrier), a block 1.2 of it (launch, query fragments, first stage,
// merges): many blocks are as bad as a last round of few.  Statistics, weights and the rest of the call on fp16
// keys, us: 24 layers of 8192 tokens with 4 stages per block 282, with 6 276, with 8 (three whole rounds) 253; 32 heads of 32768
// tokens 251, 236 and 227.
// Every block of the second pass merges the statistics of all chunks of its unit, 32 in flight: 0.3 of a stage for each
// 32 of them (a stage of fp32 keys takes four times as long).  It keeps one or two units from being cut into 256 chunks:
// one of 8192 tokens with 256 query rows 39 us by 256 chunks of 32 keys, 27 by 64 of 128; 32768 tokens 53 and 48, two units of
// 8192 31 and 27; 32 query rows 32 and 21.  Over 1 to 192 units of 512 to 131072 tokens with 32, 128 and 256 query rows the
// choice is 2.6 % off the best of all stage sizes and counts on average, 19 % at most; without this term 7.4 % and 51 %.  (More than
// one block of small stages fits a compute unit; counting them so did not choose better.)
constexpr int kBlocksAtOnce = 256;

void choose_stages(int U, int l, int dtype, int *keys, int *stages) {
  const int full = dtype == SPINDLE_F32 ? 128 : 256;
  const double merge = dtype == SPINDLE_F32 ? 0.08 : 0.3;
  double best = INFINITY;
  for (int k = full; k >= 32; k /= 2) {
    const int n = (l + k - 1) / k;
    for (int s = 1; s <= kMaxStagesPerBlock; ++s) {
      const int chunks = (n + s - 1) / s;
      const long rounds = ((long)U * chunks + kBlocksAtOnce - 1) / kBlocksAtOnce;
      const double t = (double)rounds * (s * ((double)k / full + 0.1) + 1.2) + merge * ((chunks + 31) / 32);
      if (t < best) {
        best = t;
        *keys = k;
        *stages = s;
      }
    }
  }
}

DeepLayout deep_layout(void *ws, int U, int l, int lw, int Rpad, int dtype) {
  Carver cv(ws);
  DeepLayout L;
  choose_stages(U, l, dtype, &L.keys, &L.stages);
  L.nchunks = (l + L.stages * L.keys - 1) / (L.stages * L.keys);
  const int lc = l - lw;
  L.partial = cv.take<float2>((size_t)U * L.nchunks * Rpad);
  L.scores = cv.take<float>((size_t)U * (lc > 0 ? (lc + 3) & ~3 : 4));
  L.pooled = cv.take<uint32_t>((size_t)U * (lc > 0 ? lc : 1));
  L.hist = cv.take<int>((size_t)U * kBins);
  L.bytes = cv.total();
  return L;
}

// Workgroups per unit of deep_finish.  Each reads all keys of its unit, so there are no more of them than run at once on half
// of the chip (the call may run beside others': three layers of 32768 tokens in a pipeline, all of it against half, 2057 and 2059, on
// another day 2030 and 2019 us; alone, 16 units of 32736 positions 68 and 69), and as many as have LDS for their places.  Then the copies
// come along for nothing: 16 units of 32736 positions 69 us (74 by one workgroup each and a launch for the copies), 3 of 99987 62
// (101), one of 524256 128 (280).  More wait for each other, and what they read grows with the
// square of the context: 8 of 524256 519 us, as many as segments 1040.  More than four per segment gain nothing.
constexpr int kFinishBlocks = 128;

int finish_blocks(int U, int nseg) {
  const int each = kFinishBlocks / U;
  static_assert(kCandMax >= 4 * kSegLen, "a share of what is kept fits");
  return each < (nseg + 3) / 4 ? 1 : (each < 4 * nseg ? each : 4 * nseg);
}

int padded_rows(int R) { return R <= 64 ? 64 : (R <= 128 ? 128 : 256); }

template <int DT, int WR, int KEYS>
spindle_status launch_passes(const DeepParams &p, int U, hipStream_t st) {
  typedef Geo<DT, WR, KEYS> S;
  // two stages; the statistics of the waves, or the sums of the row groups over two stages and a constant per row
  size_t smem_stats = 2 * (size_t)S::kStageBytes;
  if (smem_stats < (size_t)S::kThreads * sizeof(float2)) smem_stats = (size_t)S::kThreads * sizeof(float2);
  const size_t smem_acc = 2 * (size_t)S::kStageBytes + (2 * WR * S::kStageKeys + 256) * sizeof(float);
  static LdsLimit lim_stats, lim_acc;                  // one pair per instantiation; the sizes are constants of it
  if (spindle_status e = allow_lds(lim_stats, reinterpret_cast<const void *>(&deep_stats<DT, WR, KEYS>), smem_stats)) return e;
  if (spindle_status e = allow_lds(lim_acc, reinterpret_cast<const void *>(&deep_accumulate<DT, WR, KEYS>), smem_acc)) return e;
  { ProfScope ps("deep_stats", st);
  hipLaunchKernelGGL((deep_stats<DT, WR, KEYS>), dim3(p.nchunks, U), dim3(S::kThreads), smem_stats, st, p); }
  if (p.lc > 0) {
    const int per = p.stages * S::kStageKeys;
    ProfScope ps("deep_accumulate", st);
    hipLaunchKernelGGL((deep_accumulate<DT, WR, KEYS>), dim3((p.lc + per - 1) / per, U), dim3(S::kThreads), smem_acc, st, p);
  }
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}

template <int DT, int WR>
spindle_status launch_rows(const DeepParams &p, int keys, int U, hipStream_t st) {
  if (keys == 32) return launch_passes<DT, WR, 32>(p, U, st);
  if (keys == 64) return launch_passes<DT, WR, 64>(p, U, st);
  if (keys == 128) return launch_passes<DT, WR, 128>(p, U, st);
  if constexpr (DT != SPINDLE_F32) return launch_passes<DT, WR, 256>(p, U, st);
  SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED, "%d keys per stage", keys);
}

void launch_gather(const GatherParams &p, int U, hipStream_t st) {
  const int rows_per_block = 256 / (p.row_bytes / 16);
  ProfScope ps("deep_gather", st);
  hipLaunchKernelGGL(deep_gather, dim3((p.out_stride + rows_per_block - 1) / rows_per_block, U), dim3(256), 0, st, p);
}

template <int DT>
spindle_status launch_dtype(const DeepParams &p, int keys, int U, hipStream_t st) {
  if (p.Rpad == 64) return launch_rows<DT, 2>(p, keys, U, st);
  if (p.Rpad == 128) return launch_rows<DT, 4>(p, keys, U, st);
  return launch_rows<DT, 8>(p, keys, U, st);
}

}  // namespace
}  // namespace spindle

using namespace spindle;

extern "C" spindle_status spindle_deep_workspace_bytes(const spindle_kv_desc *desc, int32_t window,
                                                       size_t *bytes) {
  spindle_status s = check_desc(desc);
  if (s != SPINDLE_OK) return s;
  if (!bytes) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "bytes is NULL");
  if (window < 1 || window > desc->seq_len) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "window must be in [1, seq_len]");
  if (desc->group_size < 1 || (int64_t)window * desc->group_size > 256)
    SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED, "window * group_size must be in [1, 256]");
  const int U = desc->batch * desc->n_kv_heads;
  *bytes = deep_layout(nullptr, U, desc->seq_len, window, padded_rows(window * desc->group_size), desc->dtype).bytes;
  return SPINDLE_OK;
}

extern "C" spindle_status spindle_compress_deep(const spindle_kv_desc *desc, const void *K, const void *V,
                                                const void *Qw, int32_t window, int32_t pool_kernel,
                                                float scale, int32_t norm, int32_t budget,
                                                const int32_t *budgets, int32_t out_stride,
                                                int32_t *kept_idx, void *K_out, void *V_out,
                                                float *scores_out, void *workspace,
                                                size_t workspace_bytes, void *stream) {
  size_t need = 0;
  spindle_status s = spindle_deep_workspace_bytes(desc, window, &need);
  if (s != SPINDLE_OK) return s;
  if (!K || !Qw || !kept_idx || !K_out) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "K, Qw, kept_idx and K_out are required");
  if ((V == nullptr) != (V_out == nullptr)) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "V and V_out must both be given or both NULL");
  if (pool_kernel < 1 || (pool_kernel & 1) == 0) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "pool_kernel must be odd and >= 1");
  if (norm != SPINDLE_NORM_PAPER && norm != SPINDLE_NORM_NONE) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "unknown norm mode %d", norm);
  if (!(scale == scale) || fabsf(scale) > 3.0e38f) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "scale must be finite");
  const int l = desc->seq_len, lw = window, lc = l - lw;
  if (!budgets && budget < lw) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "budget (%d) must be >= window (%d)", budget, lw);
  if (out_stride < lw || (!budgets && out_stride < (budget < l ? budget : l)))
    SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "out_stride (%d) is smaller than the kept-token count", out_stride);
  if (!workspace || workspace_bytes < need || (reinterpret_cast<uintptr_t>(workspace) & 255))
    SPINDLE_FAIL(SPINDLE_ERR_WORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)", need, workspace_bytes);
  const uintptr_t al = reinterpret_cast<uintptr_t>(K) | reinterpret_cast<uintptr_t>(V) |
                       reinterpret_cast<uintptr_t>(Qw) | reinterpret_cast<uintptr_t>(K_out) |
                       reinterpret_cast<uintptr_t>(V_out);
  if (al & 15) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");

  hipStream_t st = static_cast<hipStream_t>(stream);
  const int U = desc->batch * desc->n_kv_heads;
  const int R = lw * desc->group_size, Rpad = padded_rows(R);
  DeepLayout L = deep_layout(workspace, U, l, lw, Rpad, desc->dtype);

  DeepParams p;
  KvLayout lay;
  s = kv_layout(desc, &lay);
  if (s != SPINDLE_OK) return s;
  p.K = static_cast<const char *>(K);
  p.lay = lay;
  p.Q = static_cast<const char *>(Qw);
  p.partial = L.partial;
  p.scores = L.scores;
  p.spitch = (lc + 3) & ~3;
  const bool by_unit = lc > 0 && lc <= kUnitMax && pool_kernel <= 2 * kUnitRadius + 1;
  p.hist = by_unit ? nullptr : L.hist;
  p.l = l; p.lc = lc; p.lw = lw; p.hn = desc->group_size; p.R = R; p.Rpad = Rpad;
  p.stages = L.stages;
  p.nchunks = L.nchunks;
  p.sc2 = scale * kLog2e;
  p.inv_hn = 1.0f / (float)desc->group_size;
  p.norm = norm;
  if (desc->dtype == SPINDLE_F16) s = launch_dtype<SPINDLE_F16>(p, L.keys, U, st);
  else if (desc->dtype == SPINDLE_BF16) s = launch_dtype<SPINDLE_BF16>(p, L.keys, U, st);
  else s = launch_dtype<SPINDLE_F32>(p, L.keys, U, st);
  if (s != SPINDLE_OK) return s;

  SelectParams sp;
  sp.scores = L.scores; sp.pooled = L.pooled; sp.scores_out = scores_out;
  sp.hist = L.hist;
  sp.budgets = budgets; sp.kept = kept_idx;
  sp.l = l; sp.lc = lc; sp.lw = lw; sp.pool = pool_kernel; sp.budget = budget; sp.out_stride = out_stride;
  sp.spitch = p.spitch;
  GatherParams gp;
  gp.K = static_cast<const char *>(K); gp.V = static_cast<const char *>(V);
  gp.Ko = static_cast<char *>(K_out); gp.Vo = static_cast<char *>(V_out);
  gp.kept = kept_idx; gp.l = l; gp.out_stride = out_stride;
  gp.row_bytes = kHeadDim * dtype_bytes(desc->dtype);
  gp.lay = lay;
  if (by_unit) {
    static LdsLimit lim;
    if ((s = allow_lds(lim, reinterpret_cast<const void *>(&deep_select_unit), unit_lds(kUnitMax))) != SPINDLE_OK) return s;
    { ProfScope ps("deep_select", st);
    hipLaunchKernelGGL(deep_select_unit, dim3(U), dim3(kSelThreads), unit_lds(lc), st, sp); }
    launch_gather(gp, U, st);
  } else {
    const int nseg = lc > 0 ? (lc + kSegLen - 1) / kSegLen : 1;
    sp.nfinish = finish_blocks(U, nseg);
    { ProfScope ps("deep_select", st);
    hipLaunchKernelGGL(deep_select, dim3(nseg, U), dim3(kSelThreads), 0, st, sp); }
    { ProfScope ps("deep_finish", st);
    auto *finish = sp.nfinish > 1 ? (lc <= kOneTripMax ? deep_finish<true, true> : deep_finish<true, false>)
                                  : (lc <= kOneTripMax ? deep_finish<false, true> : deep_finish<false, false>);
    hipLaunchKernelGGL(finish, dim3(sp.nfinish, U), dim3(kSelThreads), 0, st, sp, gp); }
    if (sp.nfinish == 1) launch_gather(gp, U, st);
  }
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}
