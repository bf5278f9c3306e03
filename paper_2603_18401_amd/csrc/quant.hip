// Storage formats of the reduced-precision matching path: FP32 descriptor
// rows to BF16 (round to nearest even) or to OCP FP8-E4M3FN codes with one
// FP32 scale per row (s = amax / 448, 1 for an all-zero row; code =
// round-to-nearest-even of x / s, saturated at 448), and the norm of each
// row's rounding error.
//
// All four kernels are bound by memory.  Rows of 128 values whose arrays are
// aligned for it (every descriptor the library matches) take half a wavefront
// each, four values per lane in one 16-byte load, kRowsInFlight rows of a
// half-wavefront in flight, one row's conversion on the hardware's FP8
// instructions; other widths, and arrays that are not aligned, one wavefront
// per row and a value per lane.  500003 rows of 128, before -> now: to BF16
// 98 -> 57 us, to FP8 171 -> 57 us, rounding error of BF16 rows
// 120 -> 84 us, of FP8 rows 185 -> 64 us.  (These follow one another on the
// same rows, part of which is still in the memory-side cache then: the bytes
// alone, at the 4.9 TB/s of a large copy from and to HBM, are 78, 66, 79 and
// 66 us.  After 1 GiB of other writes, some of which are still to be written
// back, the four take 102, 98, 117 and 108 us, and a 256 MB copy 132.)
#include "device_common.h"
#include "launch.h"

namespace epm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr float kFp8Max = 448.0f;

__device__ __forceinline__ uint16_t to_bf16(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;  // NaN
  return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
}

// E4M3FN: 1 sign, 4 exponent (bias 7), 3 mantissa bits; subnormals step 2^-9
__device__ __forceinline__ uint8_t to_e4m3(float v) {
  const uint32_t sign = __float_as_uint(v) >> 31;
  const float a = fminf(fabsf(v), kFp8Max);
  uint32_t code;
  if (a < 0.015625f) {  // 2^-6: subnormal range (8 encodes the smallest normal)
    code = (uint32_t)rintf(a * 512.0f);
  } else {
    const uint32_t ua = __float_as_uint(a);
    int e = (int)(ua >> 23) - 127;
    const uint32_t m = ua & 0x7FFFFFu;
    uint32_t keep = m >> 20;
    const uint32_t rem = m & 0xFFFFFu;
    if (rem > 0x80000u || (rem == 0x80000u && (keep & 1u))) ++keep;
    if (keep == 8u) {
      keep = 0u;
      ++e;
    }
    code = ((uint32_t)(e + 7) << 3) | keep;
    if (code > 0x7Eu) code = 0x7Eu;  // 448, the largest finite value
  }
  return (uint8_t)(code | (sign << 7));
}

__device__ __forceinline__ float wave_max(float v) {
  #pragma unroll
  for (int off = 1; off < kWave; off <<= 1) v = fmaxf(v, __shfl_xor(v, off));
  return v;
}

// ------------------------------------------------ rows of 128, aligned
constexpr int kRowLanes = 32;      // lanes per row, four values each
constexpr int kRowsInFlight = 4;   // rows per half-wavefront
constexpr int kVecRows = kThreads / kRowLanes * kRowsInFlight;  // rows per workgroup

bool aligned_to(const void* p, uintptr_t n) { return (reinterpret_cast<uintptr_t>(p) & (n - 1)) == 0; }

// Four E4M3 codes: the hardware rounds to nearest even as to_e4m3 does, which
// saturates first (a NaN becomes 448 with its sign).
__device__ __forceinline__ float e4m3_range(float v) {
  return __builtin_copysignf(fminf(fabsf(v), kFp8Max), v);
}

__device__ __forceinline__ uint32_t to_e4m3x4(float a, float b, float c, float d) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_range(a), e4m3_range(b), 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(e4m3_range(c), e4m3_range(d), w, true);
  return (uint32_t)w;
}

// Row r's first piece for this lane, row kRowsInFlight pieces apart.
__device__ __forceinline__ int64_t vec_row(int u) {
  return (int64_t)blockIdx.x * kVecRows + u * (kThreads / kRowLanes) + threadIdx.x / kRowLanes;
}

__global__ __launch_bounds__(kThreads) void k_quant_bf16_rows(const float4* __restrict__ src,
                                                              int64_t rows,
                                                              uint2* __restrict__ dst) {
  const int l = threadIdx.x & (kRowLanes - 1);
  float4 x[kRowsInFlight];
  #pragma unroll
  for (int u = 0; u < kRowsInFlight; ++u)
    if (vec_row(u) < rows) x[u] = src[vec_row(u) * kRowLanes + l];
  #pragma unroll
  for (int u = 0; u < kRowsInFlight; ++u) {
    if (vec_row(u) >= rows) return;
    dst[vec_row(u) * kRowLanes + l] =
        make_uint2((uint32_t)to_bf16(x[u].x) | ((uint32_t)to_bf16(x[u].y) << 16),
                   (uint32_t)to_bf16(x[u].z) | ((uint32_t)to_bf16(x[u].w) << 16));
  }
}

__global__ __launch_bounds__(kThreads) void k_quant_fp8_rows(const float4* __restrict__ src,
                                                             int64_t rows,
                                                             uint32_t* __restrict__ dst,
                                                             float* __restrict__ scale) {
  const int l = threadIdx.x & (kRowLanes - 1);
  float4 x[kRowsInFlight];
  #pragma unroll
  for (int u = 0; u < kRowsInFlight; ++u)
    x[u] = vec_row(u) < rows ? src[vec_row(u) * kRowLanes + l] : make_float4(0.f, 0.f, 0.f, 0.f);
  #pragma unroll
  for (int u = 0; u < kRowsInFlight; ++u) {
    float amax = fmaxf(fmaxf(fabsf(x[u].x), fabsf(x[u].y)), fmaxf(fabsf(x[u].z), fabsf(x[u].w)));
    #pragma unroll
    for (int off = 1; off < kRowLanes; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    float s = amax / kFp8Max;
    if (!(s > 0.0f)) s = 1.0f;
    if (vec_row(u) >= rows) return;
    dst[vec_row(u) * kRowLanes + l] = to_e4m3x4(x[u].x / s, x[u].y / s, x[u].z / s, x[u].w / s);
    if (l == 0) scale[vec_row(u)] = s;
  }
}

template <int FMT>
__global__ __launch_bounds__(kThreads) void k_round_err_rows(const float4* __restrict__ src,
                                                             int64_t rows,
                                                             const void* __restrict__ codes,
                                                             const float* __restrict__ scale,
                                                             float* __restrict__ err) {
  const int l = threadIdx.x & (kRowLanes - 1);
  float4 x[kRowsInFlight];
  uint2 c[kRowsInFlight];
  float s[kRowsInFlight];
  #pragma unroll
  for (int u = 0; u < kRowsInFlight; ++u) {
    const int64_t r = vec_row(u) < rows ? vec_row(u) : rows - 1;
    x[u] = src[r * kRowLanes + l];
    if (FMT == 0) c[u] = static_cast<const uint2*>(codes)[r * kRowLanes + l];
    else c[u].x = static_cast<const uint32_t*>(codes)[r * kRowLanes + l];
    s[u] = FMT == 1 ? scale[r] : 1.0f;
  }
  #pragma unroll
  for (int u = 0; u < kRowsInFlight; ++u) {
    const float xs[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
    float y[4];
    if (FMT == 0) {
      y[0] = __uint_as_float(c[u].x << 16);
      y[1] = __uint_as_float(c[u].x & 0xFFFF0000u);
      y[2] = __uint_as_float(c[u].y << 16);
      y[3] = __uint_as_float(c[u].y & 0xFFFF0000u);
    } else {
      const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)c[u].x, false);
      const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)c[u].x, true);
      y[0] = lo[0];
      y[1] = lo[1];
      y[2] = hi[0];
      y[3] = hi[1];
      // 0x7F is no code of epm_quantize: read as the next value after 448
      #pragma unroll
      for (int k = 0; k < 4; ++k)
        if (y[k] != y[k]) y[k] = (c[u].x >> (8 * k + 7)) & 1u ? -480.0f : 480.0f;
    }
    double acc = 0.0;
    #pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double d = (double)xs[k] - (FMT == 1 ? (double)y[k] * (double)s[u] : (double)y[k]);
      acc += d * d;
    }
    #pragma unroll
    for (int off = 1; off < kRowLanes; off <<= 1) acc += __shfl_xor(acc, off);
    if (l == 0 && vec_row(u) < rows) err[vec_row(u)] = (float)(sqrt(acc) * (1.0 + 1e-6)) + 1e-30f;
  }
}

// ------------------------------------------------ any width
__global__ __launch_bounds__(kThreads) void k_quant_bf16(const float* __restrict__ src,
                                                         int64_t n, uint16_t* __restrict__ dst) {
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kThreads)
    dst[i] = to_bf16(src[i]);
}

__global__ __launch_bounds__(kThreads) void k_quant_fp8(const float* __restrict__ src,
                                                        int64_t rows, int dim,
                                                        uint8_t* __restrict__ dst,
                                                        float* __restrict__ scale) {
  const int lane = lane_id();
  for (int64_t r = (int64_t)blockIdx.x * kWaves + wave_id(); r < rows;
       r += (int64_t)gridDim.x * kWaves) {
    const float* x = src + r * dim;
    float amax = 0.0f;
    for (int k = lane; k < dim; k += kWave) amax = fmaxf(amax, fabsf(x[k]));
    amax = wave_max(amax);
    float s = amax / kFp8Max;
    if (!(s > 0.0f)) s = 1.0f;
    for (int k = lane; k < dim; k += kWave) dst[r * dim + k] = to_e4m3(x[k] / s);
    if (lane == 0) scale[r] = s;
  }
}

// Norm of each row's rounding error, err[r] >= |x_r - dequant(code_r)|
// (FP64 sums, inflated by 1e-6 for their rounding): the tight per-row term
// that the reduced-precision bounds can use in place of the format's
// worst case.  One wavefront per row.
template <int FMT>
__global__ __launch_bounds__(kThreads) void k_round_err(const float* __restrict__ src,
                                                        int64_t rows, int dim,
                                                        const void* __restrict__ codes,
                                                        const float* __restrict__ scale,
                                                        float* __restrict__ err) {
  const int lane = lane_id();
  for (int64_t r = (int64_t)blockIdx.x * kWaves + wave_id(); r < rows;
       r += (int64_t)gridDim.x * kWaves) {
    double acc = 0.0;
    const double s = FMT == 1 ? (double)scale[r] : 1.0;
    for (int k = lane; k < dim; k += kWave) {
      double y;
      if (FMT == 0) {
        y = (double)__uint_as_float((uint32_t)static_cast<const uint16_t*>(codes)[r * dim + k] << 16);
      } else {
        const uint32_t c = static_cast<const uint8_t*>(codes)[r * dim + k];
        const uint32_t e = (c >> 3) & 15u, m = c & 7u;
        double v = e == 0 ? (double)m * 0.001953125
                          : (double)__uint_as_float(((e + 120u) << 23) | (m << 20));
        y = ((c & 0x80u) ? -v : v) * s;
      }
      const double d = (double)src[r * dim + k] - y;
      acc += d * d;
    }
    #pragma unroll
    for (int off = 1; off < kWave; off <<= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) err[r] = (float)(sqrt(acc) * (1.0 + 1e-6)) + 1e-30f;
  }
}

}  // namespace

hipError_t launch_round_err(const float* src, int64_t rows, int dim, int fmt, const void* codes,
                            const float* scale, float* err, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const int64_t vblocks = (rows + kVecRows - 1) / kVecRows;
  if (dim == 128 && vblocks <= INT32_MAX && aligned_to(src, 16) && aligned_to(codes, fmt == 0 ? 8 : 4)) {
    const float4* x = reinterpret_cast<const float4*>(src);
    if (fmt == 0)
      hipLaunchKernelGGL((k_round_err_rows<0>), dim3((unsigned)vblocks), dim3(kThreads), 0, s, x,
                         rows, codes, scale, err);
    else
      hipLaunchKernelGGL((k_round_err_rows<1>), dim3((unsigned)vblocks), dim3(kThreads), 0, s, x,
                         rows, codes, scale, err);
    return hipGetLastError();
  }
  int64_t blocks = (rows + kWaves - 1) / kWaves;
  if (blocks > 65536) blocks = 65536;
  if (fmt == 0)
    hipLaunchKernelGGL((k_round_err<0>), dim3((unsigned)blocks), dim3(kThreads), 0, s, src, rows,
                       dim, codes, scale, err);
  else
    hipLaunchKernelGGL((k_round_err<1>), dim3((unsigned)blocks), dim3(kThreads), 0, s, src, rows,
                       dim, codes, scale, err);
  return hipGetLastError();
}

hipError_t launch_quantize(const float* src, int64_t rows, int dim, int fmt, void* dst,
                           float* scale, hipStream_t s) {
  if (rows == 0) return hipSuccess;
  const int64_t vblocks = (rows + kVecRows - 1) / kVecRows;
  if (dim == 128 && vblocks <= INT32_MAX && aligned_to(src, 16) && aligned_to(dst, fmt == 0 ? 8 : 4)) {
    const float4* x = reinterpret_cast<const float4*>(src);
    if (fmt == 0)
      hipLaunchKernelGGL(k_quant_bf16_rows, dim3((unsigned)vblocks), dim3(kThreads), 0, s, x, rows,
                         static_cast<uint2*>(dst));
    else
      hipLaunchKernelGGL(k_quant_fp8_rows, dim3((unsigned)vblocks), dim3(kThreads), 0, s, x, rows,
                         static_cast<uint32_t*>(dst), scale);
    return hipGetLastError();
  }
  if (fmt == 0) {
    const int64_t n = rows * dim;
    int64_t blocks = (n + kThreads - 1) / kThreads;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_quant_bf16, dim3((unsigned)blocks), dim3(kThreads), 0, s, src, n,
                       static_cast<uint16_t*>(dst));
  } else {
    int64_t blocks = (rows + kWaves - 1) / kWaves;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_quant_fp8, dim3((unsigned)blocks), dim3(kThreads), 0, s, src, rows,
                       dim, static_cast<uint8_t*>(dst), scale);
  }
  return hipGetLastError();
}

}  // namespace epm
