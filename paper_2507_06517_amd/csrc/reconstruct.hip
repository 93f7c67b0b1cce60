// Codebook reconstruction, Eq. 14: x~_a = C[r_a] * m_a.
#include "common.h"

namespace spindle {
namespace {

// A thread takes the same 16-byte piece of kRowsAtOnce rows, so that their references, entries and stores are in flight
// together.  An output that the second-level caches don't hold anyway is streamed past them, which leaves them to the
// codebook; a smaller one stays there for the kernel that reads it.  Bound by the writes: K and V of 8 heads of 32768
// fp16 tokens to buffers no cache holds 47 us with one row per thread (and a division by the length in each) and
// ordinary stores, 30 now: 4.6 TB/s of algorithmic bytes, what a large copy reaches.
constexpr int kRebuildThreads = 256, kRowsAtOnce = 4;
constexpr size_t kStreamBytes = 32u << 20;       // the second-level caches of the 8 dies together

template <int DT, bool kStream>
__global__ __launch_bounds__(kRebuildThreads) void reconstruct_kernel(const char *C, const int32_t *ref, const float *mag,
                                                                      char *out, int n, int cap, int units) {
  typedef typename Elem<DT>::type T;
  constexpr int per = 16 / sizeof(T);           // elements per 16-byte chunk
  constexpr int tpr = kHeadDim / per;           // threads per row
  constexpr int rows = kRebuildThreads / tpr;   // of the block at a time
  const int ch = threadIdx.x % tpr;
  for (int u = blockIdx.y; u < units; u += gridDim.y) {
    const int row0 = blockIdx.x * (rows * kRowsAtOnce) + threadIdx.x / tpr;
    int r[kRowsAtOnce];
    float m[kRowsAtOnce];
    u4 v[kRowsAtOnce];
#pragma unroll
    for (int k = 0; k < kRowsAtOnce; ++k) {
      const bool on = row0 + k * rows < n;
      r[k] = on ? ref[(size_t)u * n + row0 + k * rows] : -1;
      m[k] = on ? mag[(size_t)u * n + row0 + k * rows] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < kRowsAtOnce; ++k) {
      v[k] = u4{0, 0, 0, 0};
      if (r[k] >= 0 && r[k] < cap) v[k] = *reinterpret_cast<const u4 *>(C + (((size_t)u * cap + r[k]) * kHeadDim) * sizeof(T) + ch * 16);
    }
#pragma unroll
    for (int k = 0; k < kRowsAtOnce; ++k) {
      if (row0 + k * rows >= n) continue;
      u4 o = {0, 0, 0, 0};
      if (r[k] >= 0 && r[k] < cap) {
        const T *e = reinterpret_cast<const T *>(&v[k]);
        T *w = reinterpret_cast<T *>(&o);
#pragma unroll
        for (int i = 0; i < per; ++i) w[i] = Elem<DT>::from_float(Elem<DT>::to_float(e[i]) * m[k]);
      }
      u4 *to = reinterpret_cast<u4 *>(out + ((size_t)u * n + row0 + k * rows) * kHeadDim * sizeof(T) + ch * 16);
      if (kStream) __builtin_nontemporal_store(o, to);
      else *to = o;
    }
  }
}

template <int DT>
void launch_reconstruct(const char *C, const int32_t *ref, const float *mag, char *out, int n, int cap, int units, hipStream_t st) {
  constexpr int per_block = kRebuildThreads / (kHeadDim * dtype_bytes(DT) / 16) * kRowsAtOnce;
  const dim3 grid((n + per_block - 1) / per_block, units < 65535 ? units : 65535);
  if ((size_t)units * n * kHeadDim * dtype_bytes(DT) > kStreamBytes)
    hipLaunchKernelGGL((reconstruct_kernel<DT, true>), grid, dim3(kRebuildThreads), 0, st, C, ref, mag, out, n, cap, units);
  else
    hipLaunchKernelGGL((reconstruct_kernel<DT, false>), grid, dim3(kRebuildThreads), 0, st, C, ref, mag, out, n, cap, units);
}

}  // namespace
}  // namespace spindle

using namespace spindle;

extern "C" spindle_status spindle_reconstruct(int32_t units, int32_t seq_len, int32_t head_dim, int32_t dtype,
                                              int32_t max_codes, const void *C, const int32_t *ref,
                                              const float *mag, void *out, void *stream) {
  if (units < 1 || seq_len < 1 || max_codes < 1) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "units, seq_len and max_codes must be >= 1");
  if (head_dim != kHeadDim) SPINDLE_FAIL(SPINDLE_ERR_UNSUPPORTED, "head_dim must be 128, got %d", head_dim);
  if (!C || !ref || !mag || !out) SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "C, ref, mag and out are required");
  if ((reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(out)) & 15)
    SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const char *Cc = static_cast<const char *>(C);
  char *oc = static_cast<char *>(out);
  if (dtype == SPINDLE_F32) {
    launch_reconstruct<SPINDLE_F32>(Cc, ref, mag, oc, seq_len, max_codes, units, st);
  } else if (dtype == SPINDLE_F16) {
    launch_reconstruct<SPINDLE_F16>(Cc, ref, mag, oc, seq_len, max_codes, units, st);
  } else if (dtype == SPINDLE_BF16) {
    launch_reconstruct<SPINDLE_BF16>(Cc, ref, mag, oc, seq_len, max_codes, units, st);
  } else {
    SPINDLE_FAIL(SPINDLE_ERR_INVALID_ARG, "unknown dtype %d", dtype);
  }
  SPINDLE_HIP(hipGetLastError());
  return SPINDLE_OK;
}
