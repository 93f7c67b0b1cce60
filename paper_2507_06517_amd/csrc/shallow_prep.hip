// Magnitudes (Eq. 8), unit vectors and sketches of the codebook path's tokens.
#include "shallow.h"

namespace spindle {
namespace {

// Counters, counts and marks zero, n_codes = -1 ("not finished"), codebooks zero: every thread of the launch writes
// its share.  (As a launch of its own it took 3 to 6 us of every call, most of it the launch.)  A short problem with a
// large table has blocks behind its tokens that do nothing else, as many as leave a thread kClearPieces pieces, and no more
// than the chip has compute units: the call for 64 fp16 tokens with tables of 16384 and 65536 rows 69 and 160 us by the
// block of the tokens alone, 35 and 39 with them (1024 blocks: 8 problems of 512 tokens and 32768 rows 76 -> 80).
constexpr int kClearPieces = 8, kClearBlocks = 256;
__device__ __forceinline__ void begin_call(const ShallowParams &p, size_t nzero, size_t cpieces) {
  const size_t stride = (size_t)gridDim.x * gridDim.y * 256;
  const size_t i0 = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x;
  uint32_t *z = reinterpret_cast<uint32_t *>(p.counters);
  for (size_t i = i0; i < nzero; i += stride) z[i] = 0u;
  for (int t = 0; t < p.UT / p.U; ++t) {
    for (size_t i = i0; i < (size_t)p.U; i += stride) p.n_codes[t][i] = -1;
    u4 *c = reinterpret_cast<u4 *>(p.C[t]);               // 16-byte aligned, a multiple of 16 bytes per row
    for (size_t i = i0; i < cpieces; i += stride) c[i] = u4{0, 0, 0, 0};
  }
}

// 64 tokens per block.  kSketch: also the tokens' sketches (shallow.h).  The rotation is a 128-point
// Walsh-Hadamard transform, 32 coordinates per thread: five stages in registers, two across the
// four threads of a token by quad permutations.  It spreads what a vector has in a few coordinates
// over all of them, so that the 60 kept ones carry their share of every vector's norm.
// It is the first kernel of a call and also writes what must hold before the others (begin_call).
template <int DT, bool kSketch>
__global__ __launch_bounds__(256) void shallow_prep(ShallowParams p, size_t nzero, size_t cpieces) {
  typedef typename Elem<DT>::type T;
  constexpr int kRows = 64;
  constexpr int row_bytes = kHeadDim * sizeof(T);
  constexpr int lds_row = row_bytes + 16;
  constexpr int tpr = row_bytes / 16;
  __shared__ __attribute__((aligned(16))) char tile_in[kRows * lds_row];
  constexpr bool kUnit = DT == SPINDLE_F32;            // unit vectors and their remainders
  __shared__ __attribute__((aligned(16))) char tile_out[kUnit ? kRows * kLdsRow : 16];
  __shared__ double row_inv[kRows];
  __shared__ float row_factor[kRows];
  const int ut = blockIdx.y, t = ut / p.U;
  const int row0 = blockIdx.x * kRows;
  begin_call(p, nzero, cpieces);
  if (row0 >= p.n) return;                             // a block that only clears
  for (int i = threadIdx.x; i < kRows * tpr; i += 256) {
    const int r = i / tpr, ch = i % tpr;
    u4 v = {0, 0, 0, 0};
    if (row0 + r < p.n) v = *reinterpret_cast<const u4 *>(x_row(p, ut, row0 + r) + ch * 16);
    *reinterpret_cast<u4 *>(tile_in + r * lds_row + ch * 16) = v;
  }
  __syncthreads();
  if (threadIdx.x < kRows && row0 + threadIdx.x < p.n) {
    const int r = threadIdx.x;
    constexpr int per = 16 / sizeof(T);
    double ss = 0.0;
    for (int ch = 0; ch < tpr; ++ch) {
      const u4 v = *reinterpret_cast<const u4 *>(tile_in + r * lds_row + ch * 16);
      const T *e = reinterpret_cast<const T *>(&v);
#pragma unroll
      for (int i = 0; i < per; ++i) {
        const double x = (double)Elem<DT>::to_float(e[i]);
        ss += x * x;
      }
    }
    const double m = sqrt(ss);
    const size_t idx = (size_t)ut * p.n + row0 + r;
    p.m64[idx] = m;
    p.mag[t][(size_t)(ut % p.U) * p.n + row0 + r] = (float)m;
    row_inv[r] = m > 0.0 ? (double)kUnitScale / m : 0.0;
    // NaN: the products of the row may leave the range of fp32, shallow_rows decides its pairs in
    // double precision.  Rows that hold a NaN or an infinity go the same way: their products are NaN with
    // a sign that depends on the order of the operands, so the two ends of a pair could decide
    // differently, and the merge needs a symmetric relation.
    float inv = 0.f;
    if (m != 0.0) {
      const bool usual = DT == SPINDLE_F32 ? m > 0x1p-100 && m < 0x1p100 : m > 0x1p-40 && m < 0x1p55;
      inv = !usual ? NAN : DT == SPINDLE_F32 ? 1.f / kUnitScale : (float)(1.0 / m);
    }
    row_factor[r] = inv;
    if (!kSketch) p.invp[idx] = inv;                 // (positions are tokens)
    p.perm[idx] = (uint16_t)(row0 + r);
    p.iperm[idx] = (uint16_t)(row0 + r);
  } else if (threadIdx.x < kRows) {
    row_inv[threadIdx.x] = 0.0;                      // rows past the end of the sequence
  }
  __syncthreads();
  if (kUnit || kSketch) {
    // four threads per row: unit vector (x 2^10), of fp32 inputs rounded to fp16
    const int r = threadIdx.x >> 2, part = threadIdx.x & 3;
    constexpr int per = 16 / sizeof(T);
    const double inv64 = row_inv[r];
    const float inv = (float)inv64;
    float u[32];
#pragma unroll
    for (int c = 0; c < tpr / 4; ++c) {
      const int ch = part * (tpr / 4) + c;
      const u4 v = *reinterpret_cast<const u4 *>(tile_in + r * lds_row + ch * 16);
      const T *e = reinterpret_cast<const T *>(&v);
#pragma unroll
      for (int i = 0; i < per; ++i) {
        const float x = Elem<DT>::to_float(e[i]) * inv;
        u[c * per + i] = x;
        if (kUnit) reinterpret_cast<_Float16 *>(tile_out + r * kLdsRow)[ch * per + i] = (_Float16)x;
      }
    }
    if (DT == SPINDLE_F32 && row0 + r < p.n) {
      // what the rounding to fp16 took off, x 2^11
      _Float16 *xl = p.Xl + ((size_t)ut * p.n + row0 + r) * kHeadDim + part * 32;
#pragma unroll
      for (int i = 0; i < 32; i += 8) {
        h8 lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) lo[j] = (_Float16)((u[i + j] - (float)(_Float16)u[i + j]) * 2048.f);
        *reinterpret_cast<h8 *>(xl + i) = lo;
      }
    }
    if (kSketch) {
#pragma unroll
      for (int h = 1; h < 32; h *= 2)
#pragma unroll
        for (int i = 0; i < 32; ++i)
          if ((i & h) == 0) {
            const float a = u[i], b = u[i + h];
            u[i] = a + b;
            u[i + h] = a - b;
          }
      const float s1 = part & 1 ? -1.f : 1.f, s2 = part & 2 ? -1.f : 1.f;
#pragma unroll
      for (int i = 0; i < 32; ++i)                     // quad_perm [1,0,3,2]
        u[i] = fmaf(s1, u[i], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u[i]), 0xB1, 0xF, 0xF, true)));
#pragma unroll
      for (int i = 0; i < 32; ++i)                     // quad_perm [2,3,0,1]
        u[i] = fmaf(s2, u[i], __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(u[i]), 0x4E, 0xF, 0xF, true)));
      constexpr float kNorm = kSketchScale / (kUnitScale * 11.3137085f);   // / sqrt(128)
      float rest = 0.f;
#pragma unroll
      for (int i = 15; i < 32; ++i) rest = fmaf(u[i], u[i], rest);
      rest += __shfl_xor(rest, 1);
      rest += __shfl_xor(rest, 2);
      const double m2 = inv64;                         // 1024 / m
      const bool fine = m2 == 0.0 || (m2 > 0x1p-89 && m2 < 0x1p109);
      uint32_t w[4] = {0, 0, 0, 0};
      float q2 = 0.f;                                  // squared distance of the integers from what they stand for
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float s = (i < 15 ? u[i] : 0.5f * sqrtf(rest)) * kNorm;
        const float q = fminf(fmaxf(rintf(s), -127.f), 127.f);
        q2 = fmaf(s - q, s - q, q2);
        w[i >> 2] |= ((uint32_t)(int)q & 0xFFu) << (8 * (i & 3));
      }
      q2 += __shfl_xor(q2, 1);
      q2 += __shfl_xor(q2, 2);
      if (row0 + r < p.n) {
        const size_t idx = (size_t)ut * p.n + row0 + r;
        u4 piece = {w[0], w[1], w[2], w[3]};
        if (!fine) piece = u4{0, 0, 0, 0};
        *reinterpret_cast<u4 *>(p.sk0 + idx * kSketchBytes + part * 16) = piece;
        if (part == 0) p.inv_err[idx] = make_float2(row_factor[r], fine ? sqrtf(q2) * (1.f / kSketchScale) : -1.f);
      }
    }
  }
  if (!kUnit) return;
  __syncthreads();
  for (int i = threadIdx.x; i < kRows * 16; i += 256) {
    const int r = i / 16, ch = i % 16;
    if (row0 + r < p.n)
      *reinterpret_cast<u4 *>(reinterpret_cast<char *>(p.Xh) + ((size_t)ut * p.n + row0 + r) * 256 + ch * 16) =
          *reinterpret_cast<const u4 *>(tile_out + r * kLdsRow + ch * 16);
  }
}

}  // namespace

spindle_status launch_prep(const ShallowParams &p, size_t nzero, size_t cpieces, hipStream_t st) {
  const size_t clear = ((size_t)(p.UT / p.U) * cpieces / kClearPieces + 255) / 256;   // blocks, of the whole call
  const int tokens = (p.n + 63) / 64, wide = (int)(((clear < kClearBlocks ? clear : kClearBlocks) + p.UT - 1) / p.UT);
  const dim3 pgrid(tokens > wide ? tokens : wide, p.UT);
#define SPINDLE_PREP(DT)                                                                                          \
  do {                                                                                                            \
    if (p.scan) hipLaunchKernelGGL((shallow_prep<DT, true>), pgrid, dim3(256), 0, st, p, nzero, cpieces);         \
    else hipLaunchKernelGGL((shallow_prep<DT, false>), pgrid, dim3(256), 0, st, p, nzero, cpieces);               \
  } while (0)
  ProfScope ps("shallow_prep", st);
  if (p.dtype == SPINDLE_F16) SPINDLE_PREP(SPINDLE_F16);
  else if (p.dtype == SPINDLE_BF16) SPINDLE_PREP(SPINDLE_BF16);
  else SPINDLE_PREP(SPINDLE_F32);
#undef SPINDLE_PREP
  return SPINDLE_OK;
}

}  // namespace spindle
