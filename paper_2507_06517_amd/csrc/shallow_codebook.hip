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
    reinterpret_cast<u4 *>(reinterpret_cast<T *>(p.C[t]) + ((size_t)u * p.cap + e) * kHeadDim)[piece] = out;
  }
}

// ---------------------------------------------------------------- codebook cap
// A token whose entry was cut goes to the stored entry of highest cosine (Eq. 4), lowest
// entry index on ties, decided as the double-precision evaluation decides it.
//
// shallow_assign finds, per cut token, the few entries that can be that maximum: fp16
// matrix-core cosines (the unit vectors of shallow_prep) against all stored entries, off
// from the exact value by less than kGuard.  With F the largest approximate cosine of a
// token, the exact maximum has an approximate value >= F - 2 kGuard, and so has every entry
// that ties with it.  Each lane keeps, for its token and its half of the entries, the
// running maximum and the entries seen within 2 kGuard of it (the list restarts whenever the
// maximum jumps by more than that, so it stays short).  shallow_assign_exact evaluates the
// surviving entries in double precision; a token whose list ran full is left to
// shallow_overflow, the exhaustive search.
constexpr int kAssignThreads = 256;

__global__ __launch_bounds__(kAssignThreads, 2) void shallow_assign(ShallowParams p) {
  typedef Mma<SPINDLE_F16> M;
  __shared__ __attribute__((aligned(1024))) char stage[2 * kStageBytes];
  const int ut = blockIdx.y, n = p.n;
  const int nov = (int)p.ovf_cnt[ut];
  const int slot0 = blockIdx.x * kAssignThreads;
  if (slot0 >= nov) return;
  const int kept = p.n_codes[ut / p.U][ut % p.U];     // = cap whenever tokens were cut
  if (kept <= 0) return;
  const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5, c = lane & 31;
  const char *Xh = reinterpret_cast<const char *>(p.Xh) + (size_t)ut * n * 256;
  const uint32_t *ovf = p.ovf + (size_t)ut * n;
  const int *rank_vert = p.rank_vert + (size_t)ut * n;
  const float band2 = 2.f * kGuard * kUnitScale * kUnitScale;

  // the wave's 64 cut tokens: MFMA B operand (matrix columns = lanes)
  int slot[2];
  bool valid[2];
  M::frag af[2][M::kSteps];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    slot[cb] = slot0 + 64 * wave + 32 * cb + c;
    valid[cb] = slot[cb] < nov;
    const int tok = valid[cb] ? (int)ovf[slot[cb]] : 0;
#pragma unroll
    for (int ks = 0; ks < M::kSteps; ++ks) af[cb][ks] = valid[cb] ? M::load(Xh + (size_t)tok * 256, ks, g) : M::zero();
  }
  // staged entry 16*g + v of a tile is fed to matrix row 8*(v/4) + 4*g + v%4 (as in shallow_rows)
  const int prow = 16 * ((c >> 2) & 1) + 4 * (c >> 3) + (c & 3);
  int soff[M::kSteps];
#pragma unroll
  for (int ks = 0; ks < M::kSteps; ++ks)
    soff[ks] = prow * 256 + (((2 * ks + g) ^ ((prow & 7) | ((prow & 16) >> 1))) << 4);
  // loads of a 64-entry stage: wave w, load q covers rows (4 w + q) * 4 + lane / 16
  int srow[4];
  uint32_t spiece[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    srow[q] = (wave * 4 + q) * 4 + (lane >> 4);
    spiece[q] = (uint32_t)((((lane & 15) ^ ((srow[q] & 7) | ((srow[q] & 16) >> 1))) << 4));
  }
  const uint32_t stage_lds = (uint32_t)(size_t)(__attribute__((address_space(3))) char *)stage;
  const int nstages = (kept + kStageCols - 1) / kStageCols;
  int tokq[4];                                       // tokens of the entries the next load brings in
  auto fetch_tokens = [&](int s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int j = s * kStageCols + srow[q];
      tokq[q] = j < kept ? rank_vert[j] : 0;         // rows past the last entry are masked below
    }
  };
  auto dma = [&](int bufsel) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      lds_dma16_at(Xh, (uint32_t)tokq[q] * 256u + spiece[q], stage_lds + bufsel * kStageBytes + (wave * 4 + q) * 1024);
  };
  float runmax[2] = {-INFINITY, -INFINITY};
  int cnt[2] = {0, 0};
  uint2 *cand = p.ccand + (size_t)ut * n * 2 * kCandCap;
  auto collect = [&](f16v a, int cb, int j0) {
    if (j0 + 32 > kept) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (j0 + 16 * g + v >= kept) a[v] = -INFINITY;
    }
    float t = a[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) t = fmaxf(t, a[v]);
    const float nm = fmaxf(runmax[cb], t);
    if (nm > runmax[cb] + band2) cnt[cb] = 0;         // everything collected so far is out of reach
    runmax[cb] = nm;
    const float thr = nm - band2;
    // bit v of `hits`: a[v] >= thr, from the sign of a[v] - thr (sixteen tests and branches, one per
    // value, cost several times the matrix instructions of the tile; hits are rare)
    uint32_t miss = 0;
#pragma unroll
    for (int v = 15; v >= 0; --v) miss = __builtin_amdgcn_alignbit(miss, __float_as_uint(a[v] - thr), 31);
    uint32_t hits = valid[cb] ? ~miss & 0xFFFFu : 0u;
    if (hits) {
      uint2 *list = cand + ((size_t)slot[cb] * 2 + g) * kCandCap;
      do {
        const int v = __builtin_ctz(hits);
        hits &= hits - 1;
        float val = a[0];
#pragma unroll
        for (int u = 1; u < 16; ++u) val = v == u ? a[u] : val;
        if (cnt[cb] < kCandCap) list[cnt[cb]] = make_uint2((uint32_t)(j0 + 16 * g + v), __float_as_uint(val));
        ++cnt[cb];
      } while (hits);
    }
  };

  fetch_tokens(0);
  dma(0);
  if (nstages > 1) fetch_tokens(1);
  for (int s = 0; s < nstages; ++s) {
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0): stage s has landed
    __syncthreads();                                  // ... for every wave; the other buffer is free
    if (s + 1 < nstages) {
      dma((s + 1) & 1);
      if (s + 2 < nstages) fetch_tokens(s + 2);
    }
#pragma unroll
    for (int ct = 0; ct < 2; ++ct) {
      const int j0 = s * kStageCols + 32 * ct;
      if (j0 >= kept) break;
      f16v acc0, acc1;
#pragma unroll
      for (int v = 0; v < 16; ++v) { acc0[v] = 0.f; acc1[v] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < M::kSteps; ++ks) {
        const M::frag f = *reinterpret_cast<const M::frag *>(stage + (s & 1) * kStageBytes + ct * 32 * 256 + soff[ks]);
        acc0 = M::mma(f, af[0][ks], acc0);
        acc1 = M::mma(f, af[1][ks], acc1);
      }
      collect(acc0, 0, j0);
      collect(acc1, 1, j0);
    }
  }
  float2 *cstat = p.cstat + (size_t)ut * n * 2;
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
    if (valid[cb]) cstat[(size_t)slot[cb] * 2 + g] = make_float2(runmax[cb], __int_as_float(cnt[cb]));
}

__global__ __launch_bounds__(256) void shallow_assign_exact(ShallowParams p) {
  const int ut = blockIdx.y, n = p.n;
  const int nov = (int)p.ovf_cnt[ut];
  const uint32_t *ovf = p.ovf + (size_t)ut * n;
  const int *rank_vert = p.rank_vert + (size_t)ut * n;
  const float2 *cstat = p.cstat + (size_t)ut * n * 2;
  const uint2 *cand = p.ccand + (size_t)ut * n * 2 * kCandCap;
  const float band2 = 2.f * kGuard * kUnitScale * kUnitScale;
  for (int s = blockIdx.x * 256 + threadIdx.x; s < nov; s += gridDim.x * 256) {
    const int a = (int)ovf[s];
    const float2 st0 = cstat[(size_t)s * 2], st1 = cstat[(size_t)s * 2 + 1];
    const int c0 = __float_as_int(st0.y), c1 = __float_as_int(st1.y);
    if (c0 > kCandCap || c1 > kCandCap) {              // a list ran full: exhaustive search
      p.ovf_left[atomicAdd(p.ovf_count, 1u)] = ((uint32_t)ut << 16) | (uint32_t)a;
      continue;
    }
    const float thr = fmaxf(st0.x, st1.x) - band2;
    double bv = -INFINITY;
    int bj = 0x7FFFFFFF;
    for (int h = 0; h < 2; ++h) {
      const int ch = h ? c1 : c0;
      for (int i = 0; i < ch; ++i) {
        const uint2 e = cand[((size_t)s * 2 + h) * kCandCap + i];
        if (__uint_as_float(e.y) >= thr) {
          const int j = (int)e.x;
          const double cv = cos64(p, ut, a, rank_vert[j]);
          if (cv > bv || (cv == bv && j < bj)) { bv = cv; bj = j; }
        }
      }
    }
    if (bj == 0x7FFFFFFF) {                            // no approximate cosine is a number: a NaN or an infinity in the token
      p.ovf_left[atomicAdd(p.ovf_count, 1u)] = ((uint32_t)ut << 16) | (uint32_t)a;
      continue;
    }
    p.ref[ut / p.U][(size_t)(ut % p.U) * n + a] = bj;
  }
}

// One block per token left over: highest cosine among all stored entries.
__global__ __launch_bounds__(256) void shallow_overflow(ShallowParams p) {
  __shared__ double sh_v[256];
  __shared__ int sh_j[256];
  const unsigned count = *p.ovf_count;
  for (unsigned i = blockIdx.x; i < count; i += gridDim.x) {
    const uint32_t e = p.ovf_left[i];
    const int ut = (int)(e >> 16), a = (int)(e & 0xFFFFu);
    const int *rank_vert = p.rank_vert + (size_t)ut * p.n;
    double bv = -INFINITY;
    int bj = 0x7FFFFFFF;
    for (int j = threadIdx.x; j < p.cap; j += 256) {
      const double cv = cos64(p, ut, a, rank_vert[j]);
      if (cv > bv) { bv = cv; bj = j; }
    }
    sh_v[threadIdx.x] = bv;
    sh_j[threadIdx.x] = bj;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (threadIdx.x < o) {
        const double ov = sh_v[threadIdx.x + o];
        const int oj = sh_j[threadIdx.x + o];
        if (ov > sh_v[threadIdx.x] || (ov == sh_v[threadIdx.x] && oj < sh_j[threadIdx.x])) {
          sh_v[threadIdx.x] = ov;
          sh_j[threadIdx.x] = oj;
        }
      }
      __syncthreads();
    }
    if (threadIdx.x == 0) p.ref[ut / p.U][(size_t)(ut % p.U) * p.n + a] = sh_j[0] == 0x7FFFFFFF ? 0 : sh_j[0];
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
  { ProfScope ps("shallow_assign", st);
  hipLaunchKernelGGL(shallow_assign, dim3((n + kAssignThreads - 1) / kAssignThreads, p.UT), dim3(kAssignThreads), 0, st, p);
  int ax = (n + 255) / 256;
  hipLaunchKernelGGL(shallow_assign_exact, dim3(ax < 64 ? ax : 64, p.UT), dim3(256), 0, st, p); }
  { ProfScope ps("shallow_overflow", st);
  hipLaunchKernelGGL(shallow_overflow, dim3(2048), dim3(256), 0, st, p); }
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}

}  // namespace spindle
