// Static min-max calibration and symmetrization factors (OutlierTune
// Sec. 3.2: z = (max + min) / 2 per activation channel; App. A: min-max
// calibration of the activation scale, offline).
//
// Device layout of the running state: minmax[0, K) = per-channel minima,
// minmax[K, 2K) = maxima, both fp32 (the inputs are fp16, so exact).
// Minimum and maximum are order-independent, so the state is the same
// whatever the launch shape and however the rows are split across calls.
#include <math.h>

#include "ot_common.h"

namespace ot {
namespace detail {

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = 64;

// Float atomics through the integer order of IEEE bit patterns: for
// non-negative floats the signed-int order is the float order, for negative
// floats the unsigned order is the reverse of it.  -0 must be mapped to +0
// by the caller.
__device__ inline void atomic_min_f32(float *addr, float v) {
  if (v >= 0.0f)
    atomicMin(reinterpret_cast<int *>(addr), __float_as_int(v));
  else
    atomicMax(reinterpret_cast<unsigned int *>(addr), __float_as_uint(v));
}

__device__ inline void atomic_max_f32(float *addr, float v) {
  if (v >= 0.0f)
    atomicMax(reinterpret_cast<int *>(addr), __float_as_int(v));
  else
    atomicMin(reinterpret_cast<unsigned int *>(addr), __float_as_uint(v));
}

// A quiet NaN whose bit pattern, read as a signed int, is above every finite
// float and +inf: once stored into a maximum slot no later update replaces it.
constexpr int kPoison = 0x7FC00000;

__global__ __launch_bounds__(kThreads) void calib_reset_kernel(float *minmax, int64_t K) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k < K) {
    minmax[k] = INFINITY;
    minmax[K + k] = -INFINITY;
  }
}

// grid.x: channel blocks of kThreads channels, grid.y: row blocks (strided
// when there are more than 4096).  Each thread owns one channel and scans
// blocks of kRowsPerBlock rows (coalesced: a wave
// reads 64 consecutive fp16 of a row), then publishes one atomic min and max.
__global__ __launch_bounds__(kThreads) void calib_minmax_kernel(const uint16_t *__restrict__ x,
                                                                int64_t rows, int64_t K,
                                                                float *__restrict__ minmax) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k >= K) return;
  float lo = INFINITY, hi = -INFINITY;
  bool bad = false;
  for (int64_t r0 = (int64_t)blockIdx.y * kRowsPerBlock; r0 < rows;
       r0 += (int64_t)gridDim.y * kRowsPerBlock) {
    const int64_t r1 = r0 + kRowsPerBlock < rows ? r0 + kRowsPerBlock : rows;
    for (int64_t r = r0; r < r1; ++r) {
      const float v = half_bits_to_float(x[r * K + k]) + 0.0f;  // -0 -> +0
      bad |= !isfinite(v);
      lo = fminf(lo, v);
      hi = fmaxf(hi, v);
    }
  }
  if (bad) {
    atomicMax(reinterpret_cast<int *>(&minmax[K + k]), kPoison);
    return;
  }
  atomic_min_f32(&minmax[k], lo);
  atomic_max_f32(&minmax[K + k], hi);
}

// Rows of whole 16-byte chunks (any other width or alignment takes the kernel
// above).  Bound by HBM: 2 bytes per value, where one 2-byte load per lane and
// row kept too few bytes in flight: 2048 x 5120 (21 MB) 22.8 us there, 9.7
// here.  A wave takes 512 channels, 8 per lane, and kRowsAhead rows at a time
// (all their loads first), keeps minima and maxima as packed fp16 (the inputs
// are fp16, so exact) and the largest magnitude's bits (inf and NaN are 0x7c00
// and up); the workgroup's waves meet in LDS, so each channel takes one
// atomic min and max per workgroup.
constexpr int kWaves = 4;
constexpr int kWaveChannels = 512;
constexpr int kRowsAhead = 8;
constexpr int64_t kGridTarget = 1024;

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(64 * kWaves) void calib_minmax_rows_kernel(
    const uint16_t *__restrict__ x, int64_t rows, int64_t K, float *__restrict__ minmax) {
  __shared__ v4u part[3][kWaves][64];  // minima, maxima, magnitudes
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c0 = (int64_t)blockIdx.x * kWaveChannels;  // first channel
  const int64_t k0 = c0 + lane * 8;
  const h2 inf2 = {(_Float16)INFINITY, (_Float16)INFINITY};
  h2 lo[4], hi[4];
  us2 mag[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    lo[i] = inf2;
    hi[i] = -inf2;
    mag[i] = us2{0, 0};
  }
  if (k0 < K) {
    const int64_t step = (int64_t)gridDim.y * kWaves * kRowsAhead;
    for (int64_t r0 = ((int64_t)blockIdx.y * kWaves + wave) * kRowsAhead; r0 < rows; r0 += step) {
      v4u v[kRowsAhead];
#pragma unroll
      for (int u = 0; u < kRowsAhead; ++u) {
        // past the last row: the last row once more, which changes nothing
        const int64_t r = r0 + u < rows ? r0 + u : rows - 1;
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(x + r * K + k0));
      }
#pragma unroll
      for (int u = 0; u < kRowsAhead; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const unsigned word = v[u][i];
          const h2 w = __builtin_bit_cast(h2, word);
          lo[i] = __builtin_elementwise_min(lo[i], w);
          hi[i] = __builtin_elementwise_max(hi[i], w);
          mag[i] = __builtin_elementwise_max(mag[i],
                                             __builtin_bit_cast(us2, word & 0x7fff7fffu));
        }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    part[0][wave][lane][i] = __builtin_bit_cast(unsigned, lo[i]);
    part[1][wave][lane][i] = __builtin_bit_cast(unsigned, hi[i]);
    part[2][wave][lane][i] = __builtin_bit_cast(unsigned, mag[i]);
  }
  __syncthreads();
  const uint16_t *p = reinterpret_cast<const uint16_t *>(part);
  constexpr int kPlane = kWaves * kWaveChannels;
  for (int c = threadIdx.x; c < kWaveChannels && c0 + c < K; c += 64 * kWaves) {
    float l = INFINITY, h = -INFINITY;
    unsigned m = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      l = fminf(l, half_bits_to_float(p[w * kWaveChannels + c]));
      h = fmaxf(h, half_bits_to_float(p[kPlane + w * kWaveChannels + c]));
      m = max(m, (unsigned)p[2 * kPlane + w * kWaveChannels + c]);
    }
    const int64_t k = c0 + c;
    if (m >= 0x7c00u) {
      atomicMax(reinterpret_cast<int *>(&minmax[K + k]), kPoison);
    } else {
      atomic_min_f32(&minmax[k], l + 0.0f);      // -0 -> +0
      atomic_max_f32(&minmax[K + k], h + 0.0f);
    }
  }
}

// Finalize of a synchronous calibration call: every workgroup looks the whole
// state over (2 K floats, from the L2) and writes its channels' z, s, 1/s only
// if all of it is finite; otherwise it raises *status (host memory).  One
// launch and one synchronization where the state used to be copied to the
// host, looked over there and finalized by a launch of its own.
constexpr int kFinishThreads = 1024;

__device__ inline void finalize_channel(const float *__restrict__ minmax, int64_t K, int64_t k,
                                        int qa, int symmetrize, float *__restrict__ z,
                                        float *__restrict__ s, float *__restrict__ inv_s);

__global__ __launch_bounds__(kFinishThreads) void calib_finish_kernel(
    const float *__restrict__ minmax, int64_t K, int qa, float *__restrict__ z,
    float *__restrict__ s, float *__restrict__ inv_s, int *__restrict__ status) {
  bool bad = false;
#pragma unroll 8
  for (int64_t i = threadIdx.x; i < 2 * K; i += kFinishThreads) bad |= !isfinite(minmax[i]);
  if (__syncthreads_or(bad)) {
    if (threadIdx.x == 0)
      __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return;
  }
  const int64_t k = (int64_t)blockIdx.x * kFinishThreads + threadIdx.x;
  if (k < K) finalize_channel(minmax, K, k, qa, 1, z, s, inv_s);
}

// z, s, inv_s from the state, in fp64 with one rounding to fp32 each.
// symmetrize != 0: Sec. 3.2's z = (hi + lo) / 2, s = ((hi - lo) / 2) / qa.
// symmetrize == 0 (the ablation of Sec. 4.4): z = 0, s = max(|lo|, |hi|) / qa.
__device__ inline void finalize_channel(const float *__restrict__ minmax, int64_t K, int64_t k,
                                        int qa, int symmetrize, float *__restrict__ z,
                                        float *__restrict__ s, float *__restrict__ inv_s) {
  const double lo = (double)minmax[k];
  const double hi = (double)minmax[K + k];
  // exact: both are fp16 values
  const double half = symmetrize ? (hi - lo) / 2.0 : fmax(fabs(lo), fabs(hi));
  float sk = (float)(half / (double)qa);
  if (sk == 0.0f) sk = 1.0f;
  z[k] = symmetrize ? (float)((hi + lo) / 2.0) : 0.0f;
  s[k] = sk;
  inv_s[k] = (float)(1.0 / (double)sk);
}

__global__ __launch_bounds__(kThreads) void calib_finalize_kernel(const float *__restrict__ minmax,
                                                                  int64_t K, int qa,
                                                                  int symmetrize,
                                                                  float *__restrict__ z,
                                                                  float *__restrict__ s,
                                                                  float *__restrict__ inv_s) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k < K) finalize_channel(minmax, K, k, qa, symmetrize, z, s, inv_s);
}

unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace detail

using namespace detail;

hipError_t launch_calib_reset(float *minmax, int64_t K, hipStream_t st) {
  calib_reset_kernel<<<blocks_for(K, kThreads), kThreads, 0, st>>>(minmax, K);
  return hipGetLastError();
}

hipError_t launch_calib_minmax(const uint16_t *x, int64_t rows, int64_t K, float *minmax,
                               hipStream_t st) {
  if (K % 8 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0) {
    // enough workgroups for every CU several times over, and no more: each
    // costs two atomics per channel
    const int64_t gx = (K + kWaveChannels - 1) / kWaveChannels;
    int64_t gy = (rows + kWaves * kRowsAhead - 1) / (kWaves * kRowsAhead);
    const int64_t most = (kGridTarget + gx - 1) / gx;
    if (gy > most) gy = most;
    calib_minmax_rows_kernel<<<dim3((unsigned)gx, (unsigned)gy), 64 * kWaves, 0, st>>>(x, rows, K,
                                                                                      minmax);
    return hipGetLastError();
  }
  unsigned gy = blocks_for(rows, kRowsPerBlock);
  dim3 grid(blocks_for(K, kThreads), gy < 4096 ? gy : 4096);
  calib_minmax_kernel<<<grid, kThreads, 0, st>>>(x, rows, K, minmax);
  return hipGetLastError();
}

bool calib_finish_ok(int64_t K) { return K <= 65536; }

hipError_t launch_calib_finish(const float *minmax, int64_t K, int qa, float *z, float *s,
                               float *inv_s, int *status, hipStream_t st) {
  calib_finish_kernel<<<blocks_for(K, kFinishThreads), kFinishThreads, 0, st>>>(minmax, K, qa, z, s,
                                                                               inv_s, status);
  return hipGetLastError();
}

hipError_t launch_calib_finalize(const float *minmax, int64_t K, int qa, int symmetrize, float *z,
                                 float *s, float *inv_s, hipStream_t st) {
  calib_finalize_kernel<<<blocks_for(K, kThreads), kThreads, 0, st>>>(minmax, K, qa, symmetrize, z,
                                                                      s, inv_s);
  return hipGetLastError();
}

}  // namespace ot
