// Offline weight and bias transform of OutlierTune:
//   Sec. 3.1 Eq. (e):  W_s[n, k] = W[n, k] * s_k   (activation scale folded
//                      into the weights along the input channels)
//   Eq. (f):           per-output-channel quantization of W_s with a
//                      min-max scale sW_n = max_k |W_s[n, k]| / qw
//   Sec. 3.2 Eq. (g):  compensated bias b'_n = sum_k z_k W[n, k] + b_n
//   Implementation paragraph: done once, before inference.
// and, for the per-token linears (out, fc2; Eq. (c), (h)), the same
// per-output-channel quantization of W itself with the bias b + z.
//
// The general kernels (any K and alignment): one workgroup per output channel
// n, W read twice.  fold_rows_kernel below takes whole 16-byte chunks.
// Pass 1 reduces max |W_s| and the
// bias sum in fp64 (each product is exact in fp64: 24 x 11 significand
// bits); pass 2 writes the codes with a correctly rounded fp64 division.
// The max is order-free, so sW and Wq are exact; the fp64 bias sum is a
// fixed tree, so b' is deterministic but may differ from a sequential sum in
// its last fp32 place.
#include <math.h>

#include "ot_common.h"

namespace ot {
namespace detail {

constexpr int kThreads = 256;

// One output channel's scale and bias; a non-finite one (NaN for a row with
// non-finite weights) also raises *status (host memory, where given).
__device__ inline void finish_row(int64_t n, int bad, float sw, float bias,
                                  float *__restrict__ sW, float *__restrict__ bprime,
                                  int *__restrict__ status) {
  if (bad) sw = __builtin_nanf("");
  sW[n] = sw;
  bprime[n] = bias;
  if (status != nullptr && (!isfinite(sw) || !isfinite(bias)))
    __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// s == nullptr means s = 1 (no activation scale to fold: the per-token
// path), z == nullptr means z = 0; zres (nullable, [N]) is added to the bias
// (Eq. (h): the shift of a symmetrized residual stream).
__global__ __launch_bounds__(kThreads) void fold_kernel(const uint16_t *__restrict__ W,
                                                        const uint16_t *__restrict__ b,
                                                        const float *__restrict__ zres,
                                                        int64_t K, int qw,
                                                        const float *__restrict__ z,
                                                        const float *__restrict__ s,
                                                        int8_t *__restrict__ Wq,
                                                        float *__restrict__ sW,
                                                        float *__restrict__ bprime,
                                                        int *__restrict__ status) {
  __shared__ double red_max[kThreads];
  __shared__ double red_sum[kThreads];
  __shared__ int red_bad[kThreads];
  __shared__ double row_scale;

  const int64_t n = blockIdx.x;
  const uint16_t *w = W + n * K;
  const int t = threadIdx.x;

  double m = 0.0, acc = 0.0;
  int bad = 0;
  for (int64_t k = t; k < K; k += kThreads) {
    const double wk = (double)half_bits_to_float(w[k]);
    bad |= !isfinite(wk);
    const double ws = s ? (double)s[k] * wk : wk;  // Eq. (e), exact
    m = fmax(m, fabs(ws));
    if (z) acc += (double)z[k] * wk;  // exact product, fp64 sum
  }
  red_max[t] = m;
  red_sum[t] = acc;
  red_bad[t] = bad;
  __syncthreads();
  for (int off = kThreads / 2; off > 0; off >>= 1) {
    if (t < off) {
      red_max[t] = fmax(red_max[t], red_max[t + off]);
      red_sum[t] = red_sum[t] + red_sum[t + off];
      red_bad[t] |= red_bad[t + off];
    }
    __syncthreads();
  }
  if (t == 0) {
    float sw = (float)(red_max[0] / (double)qw);
    if (sw == 0.0f) sw = 1.0f;
    const double bn = b ? (double)half_bits_to_float(b[n]) : 0.0;
    finish_row(n, red_bad[0], sw, (float)(red_sum[0] + bn + (zres ? (double)zres[n] : 0.0)), sW,
               bprime, status);
    row_scale = (double)sw;
  }
  __syncthreads();
  const double sc = row_scale;
  const double lim = (double)qw;
  int8_t *q = Wq + n * K;
  for (int64_t k = t; k < K; k += kThreads) {
    const double wk = (double)half_bits_to_float(w[k]);
    const double ws = s ? (double)s[k] * wk : wk;
    const double r = fmin(fmax(rint(ws / sc), -lim), lim);
    q[k] = (int8_t)(int)r;
  }
}

// Asymmetric weights (the "Int8" setting): per output channel n of W_s,
//   lo, hi = min(min_k W_s, 0), max(max_k W_s, 0);  sW = fp32((hi - lo) / L)
//   zW = clip(rne(-lo / sW), 0, L);  c = clip(rne(W_s / sW) + zW, 0, L)
// with L = 2^bits - 1 (Eq. (a) with a zero point).  Codes and zero point
// are stored shifted by 2^(bits-1) (signed int8 for the matrix cores).
__global__ __launch_bounds__(kThreads) void fold_asym_kernel(
    const uint16_t *__restrict__ W, const uint16_t *__restrict__ b, int64_t K, int w_bits,
    const float *__restrict__ z, const float *__restrict__ s, int8_t *__restrict__ Wq,
    float *__restrict__ sW, int32_t *__restrict__ zW, float *__restrict__ bprime,
    int *__restrict__ status) {
  __shared__ double red_min[kThreads];
  __shared__ double red_max[kThreads];
  __shared__ double red_sum[kThreads];
  __shared__ int red_bad[kThreads];
  __shared__ double row_scale, row_zero;

  const int64_t n = blockIdx.x;
  const uint16_t *w = W + n * K;
  const int t = threadIdx.x;
  const double L = (double)((1 << w_bits) - 1);
  const int half = 1 << (w_bits - 1);

  double lo = 0.0, hi = 0.0, acc = 0.0;  // the range always holds 0
  int bad = 0;
  for (int64_t k = t; k < K; k += kThreads) {
    const double wk = (double)half_bits_to_float(w[k]);
    bad |= !isfinite(wk);
    const double ws = (double)s[k] * wk;  // Eq. (e), exact
    lo = fmin(lo, ws);
    hi = fmax(hi, ws);
    acc += (double)z[k] * wk;  // exact product, fp64 sum
  }
  red_min[t] = lo;
  red_max[t] = hi;
  red_sum[t] = acc;
  red_bad[t] = bad;
  __syncthreads();
  for (int off = kThreads / 2; off > 0; off >>= 1) {
    if (t < off) {
      red_min[t] = fmin(red_min[t], red_min[t + off]);
      red_max[t] = fmax(red_max[t], red_max[t + off]);
      red_sum[t] = red_sum[t] + red_sum[t + off];
      red_bad[t] |= red_bad[t + off];
    }
    __syncthreads();
  }
  if (t == 0) {
    float sw = (float)((red_max[0] - red_min[0]) / L);
    if (sw == 0.0f) sw = 1.0f;
    const double zp = fmin(fmax(rint(-red_min[0] / (double)sw), 0.0), L);
    const double bn = b ? (double)half_bits_to_float(b[n]) : 0.0;
    finish_row(n, red_bad[0], sw, (float)(red_sum[0] + bn), sW, bprime, status);
    zW[n] = (int32_t)zp - half;
    row_scale = (double)sw;
    row_zero = zp;
  }
  __syncthreads();
  const double sc = row_scale, zp = row_zero;
  int8_t *q = Wq + n * K;
  for (int64_t k = t; k < K; k += kThreads) {
    const double ws = (double)s[k] * (double)half_bits_to_float(w[k]);
    const double c = fmin(fmax(rint(ws / sc) + zp, 0.0), L);
    q[k] = (int8_t)((int)c - half);
  }
}

// ---------------------------------------------------------------------------
// Rows of whole 16-byte chunks: W read once, several rows per workgroup
// ---------------------------------------------------------------------------
// Bound by HBM (2 bytes in, 1 out per weight) where the general kernel is
// bound by its fp64 divisions, 2-byte loads and 1-byte stores: 20480 x 5120,
// per-channel, 395 us there, 75 us here (315 MB, 4.2 TB/s; 58 us per-token,
// which needs no products).
//
// A workgroup takes R output channels and holds their weights in registers
// (thread t the 8-weight chunks t, t + T, ..., CPT of them) between the
// row reductions and the codes.  R rows share each chunk's s and z, which
// otherwise cost four times the L2 traffic of the weights.
//
// Reductions in fp64 as in the general kernel (exact products, so sW and
// the codes are the same; b' sums in another fixed order).
//
// Codes.  The code is rne(fl64(ws / sc)).  q = fl32(fl32(s w) fl32(1 / sc))
// is within |q| 3.01 2^-24 of ws / sc (three roundings), at most 2.3e-5 for
// |q| <= 127 and 4.6e-5 for <= 255, and fl64's own rounding is far smaller.
// Where q lies farther than 3e-5 (7e-5) from a half-integer, the nearest
// integer of all three is the same; the others (6 weights in 10^5) take
// the fp64 division.  Rows whose scale is outside 2^-100 .. 2^100 (products
// could leave fp32's range) take it throughout.
enum FoldMode { kFoldChannel = 0, kFoldToken = 1, kFoldAsym = 2 };

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

__device__ inline float half_at(const v4u &x, int e) {
  return half_bits_to_float((uint16_t)(x[e >> 1] >> (16 * (e & 1))));
}

struct OpMax {
  __device__ static double f(double a, double b) { return fmax(a, b); }
};
struct OpMin {
  __device__ static double f(double a, double b) { return fmin(a, b); }
};
struct OpSum {
  __device__ static double f(double a, double b) { return a + b; }
};

// Wave reduction of R values at once: the lanes split the values between
// them while they halve, so lane l ends with value l / (64 / R).
template <class Op, int R>
__device__ inline double wave_reduce(const double (&v)[R], int lane) {
  static_assert(R == 1 || R == 2 || R == 4, "rows per workgroup");
  double a;
  int off;
  if constexpr (R == 4) {
    const bool up = lane & 32;
    const double k0 = up ? v[2] : v[0], k1 = up ? v[3] : v[1];
    const double s0 = up ? v[0] : v[2], s1 = up ? v[1] : v[3];
    const double a0 = Op::f(k0, __shfl_xor(s0, 32)), a1 = Op::f(k1, __shfl_xor(s1, 32));
    const bool up2 = lane & 16;
    a = Op::f(up2 ? a1 : a0, __shfl_xor(up2 ? a0 : a1, 16));
    off = 8;
  } else if constexpr (R == 2) {
    const bool up = lane & 32;
    a = Op::f(up ? v[1] : v[0], __shfl_xor(up ? v[0] : v[1], 32));
    off = 16;
  } else {
    a = v[0];
    off = 32;
  }
  for (; off >= 1; off >>= 1) a = Op::f(a, __shfl_xor(a, off));
  return a;
}

__device__ inline float lane_value(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

template <int MODE, int CPT, int R, int MAXT>
__global__ __launch_bounds__(MAXT) void fold_rows_kernel(
    const uint16_t *__restrict__ W, const uint16_t *__restrict__ b, const float *__restrict__ zres,
    int64_t N, int K, int bits, const float *__restrict__ z, const float *__restrict__ s,
    int8_t *__restrict__ Wq, float *__restrict__ sW, int32_t *__restrict__ zW,
    float *__restrict__ bprime, int *__restrict__ status) {
  __shared__ double red[3][MAXT / 64][R];
  __shared__ unsigned red_bits[MAXT / 64][R];
  const int T = blockDim.x, t = threadIdx.x, lane = t & 63, wave = t >> 6, nwaves = T >> 6;
  const int nchunks = K / 8;
  const int64_t row0 = (int64_t)blockIdx.x * R;

  v4u x[R][CPT];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      const int ch = t + j * T;
      x[r][j] = ch < nchunks && row0 + r < N
                    ? __builtin_nontemporal_load(
                          reinterpret_cast<const v4u *>(W + (row0 + r) * K + (int64_t)ch * 8))
                    : v4u{0u, 0u, 0u, 0u};
    }

  // ---- row reductions -----------------------------------------------------------
  double hi[R], lo[R], acc[R];
  us2 mag[R];  // largest |w| as fp16 bits: order as integers, >= 0x7c00 non-finite
#pragma unroll
  for (int r = 0; r < R; ++r) {
    hi[r] = lo[r] = acc[r] = 0.0;
    mag[r] = us2{0, 0};
  }
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int ch = t + j * T;
    if (ch >= nchunks) continue;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        mag[r] = __builtin_elementwise_max(
            mag[r], __builtin_bit_cast(us2, x[r][j][i] & 0x7fff7fffu));
    if constexpr (MODE != kFoldToken) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4 s4 = reinterpret_cast<const float4 *>(s + (int64_t)ch * 8)[h];
        const float4 z4 = reinterpret_cast<const float4 *>(z + (int64_t)ch * 8)[h];
        const float sv[4] = {s4.x, s4.y, s4.z, s4.w}, zv[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const double sd = (double)sv[e], zd = (double)zv[e];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double wd = (double)half_at(x[r][j], 4 * h + e);
            const double ws = sd * wd;  // Eq. (e), exact
            if constexpr (MODE == kFoldAsym) {
              hi[r] = fmax(hi[r], ws);
              lo[r] = fmin(lo[r], ws);
            } else {
              hi[r] = fmax(hi[r], fabs(ws));
            }
            acc[r] = fma(zd, wd, acc[r]);  // exact product, fp64 sum
          }
        }
      }
    }
  }
  // lane l of a wave ends with row l / (64 / R)
  constexpr int kLanes = 64 / R;
  {
    double h1 = 0.0, l1 = 0.0, a1 = 0.0;
    if constexpr (MODE != kFoldToken) {
      h1 = wave_reduce<OpMax, R>(hi, lane);
      a1 = wave_reduce<OpSum, R>(acc, lane);
    }
    if constexpr (MODE == kFoldAsym) l1 = wave_reduce<OpMin, R>(lo, lane);
    double md[R];  // fp16 bit patterns are exact as doubles
#pragma unroll
    for (int r = 0; r < R; ++r) md[r] = (double)(mag[r][0] > mag[r][1] ? mag[r][0] : mag[r][1]);
    const double m1 = wave_reduce<OpMax, R>(md, lane);
    if (lane % kLanes == 0) {
      red[0][wave][lane / kLanes] = h1;
      red[1][wave][lane / kLanes] = a1;
      red[2][wave][lane / kLanes] = l1;
      red_bits[wave][lane / kLanes] = (unsigned)m1;
    }
  }
  __syncthreads();

  // ---- each row's scale, zero point and bias (lane l: row l mod R) -----------------
  const int q = MODE == kFoldAsym ? (1 << bits) - 1 : (1 << (bits - 1)) - 1;  // L or qw
  const int half = MODE == kFoldAsym ? 1 << (bits - 1) : 0;
  const int lr = lane % R;
  double h = 0.0, l = 0.0, a = 0.0;
  unsigned mb = 0;
  for (int w = 0; w < nwaves; ++w) {
    h = fmax(h, red[0][w][lr]);
    a += red[1][w][lr];
    l = fmin(l, red[2][w][lr]);
    mb = max(mb, red_bits[w][lr]);
  }
  if constexpr (MODE == kFoldToken) h = (double)half_bits_to_float((uint16_t)mb);
  float sw = (float)((MODE == kFoldAsym ? h - l : h) / (double)q);
  if (sw == 0.0f) sw = 1.0f;
  const float zp =
      MODE == kFoldAsym ? (float)fmin(fmax(rint(-l / (double)sw), 0.0), (double)q) : 0.f;
  // 0 where every code of the row takes the fp64 division
  const float inv = sw > 0x1p-100f && sw < 0x1p100f ? (float)(1.0 / (double)sw) : 0.f;
  if (t < R && row0 + t < N) {
    const int64_t n = row0 + t;
    const double bn = b ? (double)half_bits_to_float(b[n]) : 0.0;
    finish_row(n, mb >= 0x7c00u, sw, (float)(a + bn + (zres ? (double)zres[n] : 0.0)), sW, bprime,
               status);
    if constexpr (MODE == kFoldAsym) zW[n] = (int32_t)zp - half;
  }

  // ---- codes -----------------------------------------------------------------------
  const float margin = MODE == kFoldAsym ? 0.5f - 7e-5f : 0.5f - 3e-5f;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int ch = t + j * T;
    if (ch >= nchunks) continue;
    float sv[8];
    if constexpr (MODE != kFoldToken) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const float4 s4 = reinterpret_cast<const float4 *>(s + (int64_t)ch * 8)[g];
        sv[4 * g] = s4.x; sv[4 * g + 1] = s4.y; sv[4 * g + 2] = s4.z; sv[4 * g + 3] = s4.w;
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (row0 + r >= N) continue;
      const float inv_r = lane_value(inv, r), sw_r = lane_value(sw, r), zp_r = lane_value(zp, r);
      const float top = (float)q - zp_r, bottom = MODE == kFoldAsym ? -zp_r : -(float)q;
      // adding 1.5 * 2^23 rounds to an integer whose low byte is in the
      // sum's; the shift of an asymmetric code is added along
      const float magic = 12582912.0f + (zp_r - (float)half);
      uint32_t code[8];
      bool unsure = inv_r == 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float w = half_at(x[r][j], e);
        const float ws = MODE == kFoldToken ? w : sv[e] * w;
        const float u = __builtin_amdgcn_fmed3f(ws * inv_r, bottom, top);
        const float v = u + magic;
        unsure |= fabsf(u - (v - magic)) > margin;
        code[e] = __float_as_uint(v);
      }
      if (unsure) {
        const double sc = (double)sw_r;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const double wd = (double)half_at(x[r][j], e);
          const double ws = MODE == kFoldToken ? wd : (double)sv[e] * wd;
          const double c = fmin(fmax(rint(ws / sc), (double)bottom), (double)top);
          code[e] = (uint32_t)((int)c + (MODE == kFoldAsym ? (int)zp_r - half : 0));
        }
      }
      const uint32_t lo4 = __builtin_amdgcn_perm(code[1], code[0], 0x0c0c0400u) |
                           __builtin_amdgcn_perm(code[3], code[2], 0x04000c0cu);
      const uint32_t hi4 = __builtin_amdgcn_perm(code[5], code[4], 0x0c0c0400u) |
                           __builtin_amdgcn_perm(code[7], code[6], 0x04000c0cu);
      *reinterpret_cast<uint2 *>(Wq + (row0 + r) * K + (int64_t)ch * 8) = make_uint2(lo4, hi4);
    }
  }
}

// Rows of whole 16-byte chunks, every pointer aligned for the vector accesses,
// and a row that a workgroup's registers hold.
constexpr int64_t kMaxRowsK = 65536;
static bool rows_kernel_ok(const uint16_t *W, int64_t K, const float *z, const float *s,
                           const int8_t *Wq) {
  const uintptr_t p16 = reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(z) |
                        reinterpret_cast<uintptr_t>(s);
  return K % 8 == 0 && K <= kMaxRowsK && p16 % 16 == 0 &&
         reinterpret_cast<uintptr_t>(Wq) % 8 == 0;
}

template <int MODE, int CPT, int R, int MAXT>
hipError_t launch_rows(const uint16_t *W, const uint16_t *b, const float *zres, int64_t N,
                       int64_t K, int bits, const float *z, const float *s, int8_t *Wq, float *sW,
                       int32_t *zW, float *bprime, int *status, hipStream_t st) {
  const int threads = (int)((K / 8 + CPT * 64 - 1) / (CPT * 64)) * 64;
  if (threads > MAXT) return hipErrorInvalidValue;
  fold_rows_kernel<MODE, CPT, R, MAXT><<<(unsigned)((N + R - 1) / R), threads, 0, st>>>(
      W, b, zres, N, (int)K, bits, z, s, Wq, sW, zW, bprime, status);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_rows_k(const uint16_t *W, const uint16_t *b, const float *zres, int64_t N,
                         int64_t K, int bits, const float *z, const float *s, int8_t *Wq,
                         float *sW, int32_t *zW, float *bprime, int *status, hipStream_t st) {
  // Workgroups of 3 or 4 waves where the registers allow (20480 x 5120,
  // per-channel: 3 waves of 4 rows 75 us, 5 waves of 4 rows 117, 10 waves
  // 102), two rows past K = 8192 (16384: 85 us, four rows 90-99).
  if (K <= 6144)
    return launch_rows<MODE, 3, 4, 256>(W, b, zres, N, K, bits, z, s, Wq, sW, zW, bprime, status,
                                        st);
  if (K <= 8192)
    return launch_rows<MODE, 4, 4, 256>(W, b, zres, N, K, bits, z, s, Wq, sW, zW, bprime, status,
                                        st);
  if (K > 16384 && K <= 20480)  // 8 waves: 86 us against 111 with 5 waves of 8 chunks
    return launch_rows<MODE, 5, 2, 512>(W, b, zres, N, K, bits, z, s, Wq, sW, zW, bprime, status,
                                        st);
  if (K <= 32768)
    return launch_rows<MODE, 8, 2, 512>(W, b, zres, N, K, bits, z, s, Wq, sW, zW, bprime, status,
                                        st);
  return launch_rows<MODE, 8, 1, 1024>(W, b, zres, N, K, bits, z, s, Wq, sW, zW, bprime, status,
                                       st);
}

}  // namespace detail

using namespace detail;

hipError_t launch_fold(const uint16_t *W, const uint16_t *b, int64_t N, int64_t K, int w_bits,
                       const float *z, const float *s, int8_t *Wq, float *sW, float *bprime,
                       int *status, hipStream_t st) {
  if (rows_kernel_ok(W, K, z, s, Wq))
    return launch_rows_k<kFoldChannel>(W, b, nullptr, N, K, w_bits, z, s, Wq, sW, nullptr, bprime,
                                       status, st);
  fold_kernel<<<(unsigned)N, kThreads, 0, st>>>(W, b, nullptr, K, (1 << (w_bits - 1)) - 1, z, s,
                                                Wq, sW, bprime, status);
  return hipGetLastError();
}

// Per-token linear (Eq. (c), (h)): sW_n = max_k |W[n, k]| / qw, codes of W
// itself, b'_n = b_n + zres_n.
hipError_t launch_fold_per_token(const uint16_t *W, const uint16_t *b, const float *zres,
                                 int64_t N, int64_t K, int w_bits, int8_t *Wq, float *sW,
                                 float *bprime, int *status, hipStream_t st) {
  if (rows_kernel_ok(W, K, nullptr, nullptr, Wq))
    return launch_rows_k<kFoldToken>(W, b, zres, N, K, w_bits, nullptr, nullptr, Wq, sW, nullptr,
                                     bprime, status, st);
  fold_kernel<<<(unsigned)N, kThreads, 0, st>>>(W, b, zres, K, (1 << (w_bits - 1)) - 1, nullptr,
                                                nullptr, Wq, sW, bprime, status);
  return hipGetLastError();
}

hipError_t launch_fold_asym(const uint16_t *W, const uint16_t *b, int64_t N, int64_t K,
                            int w_bits, const float *z, const float *s, int8_t *Wq, float *sW,
                            int32_t *zW, float *bprime, int *status, hipStream_t st) {
  if (rows_kernel_ok(W, K, z, s, Wq))
    return launch_rows_k<kFoldAsym>(W, b, nullptr, N, K, w_bits, z, s, Wq, sW, zW, bprime, status,
                                    st);
  fold_asym_kernel<<<(unsigned)N, kThreads, 0, st>>>(W, b, K, w_bits, z, s, Wq, sW, zW, bprime,
                                                     status);
  return hipGetLastError();
}

}  // namespace ot
