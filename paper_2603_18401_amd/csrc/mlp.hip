// Learned per-keypoint tolerance (the paper's future-work item of Sec. 6):
// a 6 -> 64 -> 64 -> 1 ReLU network maps image-2 keypoint attributes to
// eps_j = clamp(softplus(z), 0.5, 8) px, trained with a pinball (quantile)
// loss on point-line residuals (Eq. 3) of the method's own matches.
//
//   k_eps_features   per keypoint: (scale, response, orientation, x^, y^,
//                    log1p(min(|p - e2| / diag, 1000)))
//   k_eps_infer      BF16 weights (rounded on the device from the FP32
//                    masters), FP32 activations and accumulation
//   k_eps_grad       FP32 forward + backward of a minibatch; every workgroup
//                    owns a fixed slice of the batch and writes its partial
//                    gradient, so the sums have a fixed order
//   k_eps_reduce     partial gradients summed over workgroups in order
//   k_eps_adam       Adam update, one thread per parameter
//   k_residuals      point-line distance (FP64, same evaluation as the
//                    candidate test) of each query's selected match
//
// Parameter vector (4673 floats): W1 [64][6], b1 [64], W2 [64][64], b2 [64],
// w3 [64], b3; matrices row-major with one row per output unit.
#include "device_common.h"
#include "launch.h"
#include "mfma_bounds.h"

namespace epm {

namespace {

constexpr int kIn = 6, kH = 64;
constexpr int kOffW1 = 0, kOffB1 = kOffW1 + kH * kIn, kOffW2 = kOffB1 + kH,
              kOffB2 = kOffW2 + kH * kH, kOffW3 = kOffB2 + kH, kOffB3 = kOffW3 + kH;
constexpr int kParams = kOffB3 + 1;
static_assert(kParams == kEpsParams, "parameter layout");
constexpr float kEpsMin = 0.5f, kEpsMax = 8.0f;
constexpr double kDistClip = 1000.0;

__device__ __forceinline__ float softplus_f(float z) {
  return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));  // NaN stays NaN
}

__device__ __forceinline__ float sigmoid_f(float z) {
  return z >= 0.0f ? 1.0f / (1.0f + expf(-z)) : expf(z) / (1.0f + expf(z));
}

// float -> nearest bfloat16 (ties to even), as a float
__device__ __forceinline__ float bf16_round(float x) {
  const uint32_t u = __float_as_uint(x);
  const uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
  return __uint_as_float(r);
}

// ---------------------------------------------------------------- features
constexpr int kFeatThreads = 256;

__global__ __launch_bounds__(kFeatThreads) void k_eps_features(const EpsPair* __restrict__ pairs,
                                                               const int64_t* __restrict__ kstart,
                                                               int num_pairs, int64_t n2,
                                                               const float* __restrict__ kp2,
                                                               const float* __restrict__ attrs,
                                                               float* __restrict__ out) {
  const int64_t j = (int64_t)blockIdx.x * kFeatThreads + threadIdx.x;
  if (j >= n2) return;
  const EpsPair P = pairs[find_pair(kstart, num_pairs, j)];
  const double x = kp2[2 * j], y = kp2[2 * j + 1];
  double rel = kDistClip;
  if (P.finite) {
    const double d = hypot(x - P.ex, y - P.ey);
    rel = fmin(d / P.diag, kDistClip);
  }
  const double half = 0.5 * P.w;
  float* o = out + 6 * j;
  o[0] = attrs[3 * j];
  o[1] = attrs[3 * j + 1];
  o[2] = attrs[3 * j + 2];
  o[3] = (float)((x - half) / half);
  o[4] = (float)((y - 0.5 * P.h) / half);
  o[5] = (float)log1p(rel);
}

// --------------------------------------------------------------- inference
// The 6-64-64 layers on the BF16 matrix cores, exactly: the weights are BF16
// values, and an FP32 activation is the sum of three BF16 values (8 + 8 + 8
// significant bits, by truncation: x = hi + mid + lo with nothing left over),
// so W x = W hi + W mid + W lo with every product exact and FP32
// accumulation, as in FP32 arithmetic (error against 64 bits 1.1e-7 either
// way).  A wavefront takes 64 keypoints, 16 at a time: v_mfma_f32_16x16x32,
// rows = units, columns = keypoints; the three parts of the six features and
// a constant 1 (the bias) fill one 32-deep product, and layer 1's result
// (units 16 t + 4 g + r of keypoint l & 15, g = l >> 4) is layer 2's operand
// as it stands, its weights read in that order once per wavefront.  28
// products of 16 cycles per 16 keypoints; the vector arithmetic of the splits
// and the output layer bounds it.  One thread per keypoint with the weights
// broadcast from LDS took 332 us for 2 M keypoints; this takes 72 us.
constexpr int kInferThreads = 256;
constexpr int kInferWaves = kInferThreads / kWave;
constexpr int kInferBlocks = 768;  // three per CU: the weights are staged once per workgroup
// Features and weights from these sizes on (or not finite) are left to the
// plain evaluation, whose infinities and overflows a split does not
// reproduce; below them no product or sum of the network can overflow.
constexpr float kInferBigX = 1e9f, kInferBigW = 1e6f;

// max(x, 0) of a value that is not NaN, as integers: one instruction, where
// fmaxf quiets its operand first
__device__ __forceinline__ float relu_finite(float x) {
  return __int_as_float(max(__float_as_int(x), 0));
}

__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {  // upper halves of both
  return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

__device__ __forceinline__ float bf16_trunc(float x) {
  return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
}

// Eight values as three BF16 operands whose sum they are.
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&part)[3]) {
  uint32_t w[3][4];
  #pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float a = x[2 * k], b = x[2 * k + 1];
    const float a1 = a - bf16_trunc(a), b1 = b - bf16_trunc(b);
    const float a2 = a1 - bf16_trunc(a1), b2 = b1 - bf16_trunc(b1);
    w[0][k] = bf16_pair(a, b);
    w[1][k] = bf16_pair(a1, b1);
    w[2][k] = bf16_pair(a2, b2);
  }
  #pragma unroll
  for (int p = 0; p < 3; ++p)
    part[p] = __builtin_bit_cast(bf16x8, make_uint4(w[p][0], w[p][1], w[p][2], w[p][3]));
}

// The network's z by one thread, left to right (weights in LDS): kPlainRows
// units of the second layer side by side, four inputs of each at a time, so
// that the first layer is worked out twice in all and no more registers are
// held than beside the matrix form (with the whole first layer in registers
// the kernel loses a wavefront per SIMD).  What bounds it: the weights' LDS
// reads.  2 M keypoints with one in every 64 that comes here take 487 us (1961
// with the first layer worked out anew for every unit; a kernel of its own,
// one thread per keypoint, takes 275), without any 74.
constexpr int kPlainRows = 32;
__device__ float infer_plain(const float* w, const float (&x)[kIn]) {
  float z = w[kOffB3];
  #pragma unroll 1
  for (int r0 = 0; r0 < kH; r0 += kPlainRows) {
    float a[kPlainRows];
    #pragma unroll
    for (int r = 0; r < kPlainRows; ++r) a[r] = w[kOffB2 + r0 + r];
    #pragma unroll 1
    for (int u = 0; u < kH; u += 4) {
      float h[4];
      #pragma unroll
      for (int e = 0; e < 4; ++e) {
        h[e] = w[kOffB1 + u + e];
        #pragma unroll
        for (int c = 0; c < kIn; ++c) h[e] = fmaf(w[kOffW1 + (u + e) * kIn + c], x[c], h[e]);
        h[e] = fmaxf(h[e], 0.0f);
      }
      #pragma unroll
      for (int r = 0; r < kPlainRows; ++r) {
        static_assert(kOffW2 % 4 == 0 && kH % 4 == 0, "aligned quadruples");
        const float4 k = *reinterpret_cast<const float4*>(w + kOffW2 + (r0 + r) * kH + u);
        a[r] = fmaf(k.x, h[0], a[r]);
        a[r] = fmaf(k.y, h[1], a[r]);
        a[r] = fmaf(k.z, h[2], a[r]);
        a[r] = fmaf(k.w, h[3], a[r]);
      }
    }
    #pragma unroll
    for (int r = 0; r < kPlainRows; ++r) z = fmaf(w[kOffW3 + r0 + r], fmaxf(a[r], 0.0f), z);
  }
  return z;
}

__global__ __launch_bounds__(kInferThreads, 2) void k_eps_infer(const float* __restrict__ feat,
                                                             int64_t n,
                                                             const float* __restrict__ params,
                                                             float* __restrict__ eps) {
  __shared__ __attribute__((aligned(16))) float w[kParams];
  __shared__ uint4 parts[kInferWaves][3][kWave];  // a wavefront's split features
  const int lane = lane_id(), wave = wave_id();
  const int c = lane & 15, g = lane >> 4;
  bool odd = false;  // a weight out of the range
  for (int p = threadIdx.x; p < kParams; p += kInferThreads) {
    w[p] = bf16_round(params[p]);
    odd |= !(fabsf(w[p]) < kInferBigW);
  }
  const bool plain_all = __syncthreads_or(odd) != 0;
  // operands: element e of lane (c, g) is k = 8 g + e
  bf16x8 w1[4], w2[4][2];
  f32x4 b2[4], w3[4];
  #pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int u = 16 * t + c;
    float v[8];
    #pragma unroll
    for (int e = 0; e < 8; ++e)
      v[e] = g == 3 || e > kIn ? 0.0f : (e < kIn ? w[kOffW1 + u * kIn + e] : w[kOffB1 + u]);
    w1[t] = __builtin_bit_cast(bf16x8, make_uint4(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]),
                                                  bf16_pair(v[4], v[5]), bf16_pair(v[6], v[7])));
    #pragma unroll
    for (int s = 0; s < 2; ++s) {
      #pragma unroll
      for (int e = 0; e < 8; ++e)  // unit 16 (2 s + e / 4) + 4 g + e % 4
        v[e] = w[kOffW2 + u * kH + 16 * (2 * s + e / 4) + 4 * g + e % 4];
      w2[t][s] = __builtin_bit_cast(bf16x8, make_uint4(bf16_pair(v[0], v[1]), bf16_pair(v[2], v[3]),
                                                       bf16_pair(v[4], v[5]), bf16_pair(v[6], v[7])));
    }
    #pragma unroll
    for (int r = 0; r < 4; ++r) {
      b2[t][r] = w[kOffB2 + 16 * t + 4 * g + r];
      w3[t][r] = w[kOffW3 + 16 * t + 4 * g + r];
    }
  }
  const float b3 = w[kOffB3];
  const f32x4 zero = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
  const int64_t step = (int64_t)gridDim.x * kInferThreads;
  for (int64_t j0 = ((int64_t)blockIdx.x * kInferWaves + wave) * kWave; j0 < n; j0 += step) {
    const int64_t j = j0 + lane;
    float x[kIn];
    bool fine = true;
    #pragma unroll
    for (int k = 0; k < kIn; ++k) {
      x[k] = j < n ? feat[kIn * j + k] : 0.0f;
      fine &= fabsf(x[k]) < kInferBigX;
    }
    {
      const float v[8] = {x[0], x[1], x[2], x[3], x[4], x[5], 1.0f, 0.0f};
      bf16x8 part[3];
      split8(v, part);
      #pragma unroll
      for (int p = 0; p < 3; ++p) parts[wave][p][lane] = __builtin_bit_cast(uint4, part[p]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float z = 0.0f;
    #pragma unroll
    for (int q = 0; q < 4; ++q) {  // keypoints j0 + 16 q ..
      const uint4 raw = parts[wave][g < 3 ? g : 0][16 * q + c];
      const bf16x8 xin = __builtin_bit_cast(bf16x8, g < 3 ? raw : make_uint4(0u, 0u, 0u, 0u));
      f32x4 h[4];
      #pragma unroll
      for (int t = 0; t < 4; ++t) {
        h[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[t], xin, zero, 0, 0, 0);
        #pragma unroll
        for (int r = 0; r < 4; ++r) h[t][r] = relu_finite(h[t][r]);
      }
      f32x4 a[4] = {b2[0], b2[1], b2[2], b2[3]};
      #pragma unroll
      for (int s = 0; s < 2; ++s) {
        const float v[8] = {h[2 * s][0], h[2 * s][1], h[2 * s][2], h[2 * s][3],
                            h[2 * s + 1][0], h[2 * s + 1][1], h[2 * s + 1][2], h[2 * s + 1][3]};
        bf16x8 part[3];
        split8(v, part);
        #pragma unroll
        for (int p = 0; p < 3; ++p)
          #pragma unroll
          for (int t = 0; t < 4; ++t)
            a[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2[t][s], part[p], a[t], 0, 0, 0);
      }
      float zp = 0.0f;
      #pragma unroll
      for (int t = 0; t < 4; ++t)
        #pragma unroll
        for (int r = 0; r < 4; ++r) zp = fmaf(w3[t][r], relu_finite(a[t][r]), zp);
      zp += __shfl_xor(zp, 16);
      zp += __shfl_xor(zp, 32);
      z = g == q ? zp + b3 : z;  // lane 16 q + c keeps keypoint 16 q + c
    }
    // (a keypoint's tolerance does not depend on the others of its wavefront)
    if (plain_all || !fine) z = infer_plain(w, x);
    if (j < n) eps[j] = fminf(fmaxf(softplus_f(z), kEpsMin), kEpsMax);
    __builtin_amdgcn_wave_barrier();  // the parts are read before they are written again
  }
}

// ---------------------------------------------------------------- training
// Forward and backward on the FP32 matrix cores, 16 samples per wavefront
// and step.  What bounds it: 13.2 k multiply-adds per sample, 11 us for a
// batch of 65536 at the card's FP32 MFMA rate, beside about 600 vector
// instructions per step; two wavefronts per SIMD (one with every weight in
// registers measured 37 us) let one's vector work run behind the other's
// products.  The gradients and activations never leave the registers; only
// the two operands made of W2 are read from LDS, laid out lane by lane.
// v_mfma_f32_16x16x4: lane l supplies A[l & 15][l >> 4] and B[l >> 4][l & 15]
// and gets rows 4 (l >> 4) + r, r = 0..3, of column l & 15.  With c = l & 15
// and g = l >> 4:
//   * "T" results (rows = units, columns = samples): the lane holds units
//     16 t + 4 g + r of sample c, which is the next product's B operand (or,
//     exchanged, its A operand) as it stands when that product's k-th step
//     takes units 16 t + 4 g + r, g = 0..3 -- only the weights have to be
//     read in that order;
//   * "N" results (rows = samples, columns = units): the lane holds unit
//     16 t + c of samples 4 g + r, which is both operands of the products
//     over the samples (the weight gradients).
// Layer 1 is computed in both forms (16 of the 224 products per step), the
// second layer's mask is carried from T to N in ballots, and D1 comes out in
// N form from the T operand.  The biases b1 ride along as a seventh feature
// of constant 1.  Before (LDS rows, 64 samples x 4 lanes, vector FMAs):
// 179 us at 65536 samples; now 31 us (kernel trace; 29 at least).
constexpr int kGradThreads = 512;
constexpr int kPass = 128;  // samples per workgroup and step
constexpr int kGroup = 16;  // samples per wavefront and step
// a small batch is spread over more workgroups than its steps would fill
constexpr int kBlockSamples = 64;
constexpr int kGradWaves = kGradThreads / kWave;
static_assert(kGradWaves * kGroup == kPass, "one group per wavefront");
constexpr int kTiles = kH / 16;  // 16-unit tiles of a hidden layer
static_assert(kTiles == 4 && kIn + 1 <= 8, "operand layout of the network");

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sample base + (l & 15): its slot, and its feature row, -1 for none (indices
// outside the caller's arrays make the sample count as absent).
struct GradRow {
  int64_t slot, fi;
};

__device__ __forceinline__ GradRow load_row(const EpsGradArgs& A, int64_t base, int64_t end) {
  const int64_t sid = base + (lane_id() & 15);
  GradRow s;
  s.slot = sid < end ? (int64_t)A.sample_idx[sid] : -1;
  s.fi = -1;
  if (s.slot >= 0 && s.slot < A.num_slots) {
    s.fi = A.feat_index ? A.feat_index[s.slot] : s.slot;
    if (s.fi >= A.num_rows) s.fi = -1;
  }
  return s;
}

// A group's inputs: the sample's target and its features g and 4 + g (the
// seventh is the constant 1), and feature l & 15 of samples 4 g + r.
struct GradIn {
  float x0, x1, y, xn[4];
  bool valid;
};

__device__ __forceinline__ GradIn load_group(const EpsGradArgs& A, const GradRow& s) {
  const int lane = lane_id(), c = lane & 15, g = lane >> 4;
  GradIn in;
  in.valid = s.fi >= 0;
  in.y = in.valid ? A.target[s.slot] : 0.0f;
  const float* x = A.features + kIn * s.fi;
  in.x0 = in.valid ? x[g] : 0.0f;
  in.x1 = in.valid && g < kIn - 4 ? x[4 + g] : (g == kIn - 4 ? 1.0f : 0.0f);
  #pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int64_t fr = __shfl(s.fi, 4 * g + r);
    in.xn[r] = fr >= 0 && c < kIn ? A.features[kIn * fr + c] : (c == kIn ? 1.0f : 0.0f);
  }
  return in;
}

__global__ __launch_bounds__(kGradThreads, 2) void k_eps_grad(EpsGradArgs A) {
  // the weights on the way in, the wavefronts' gradients on the way out
  __shared__ float w[kParams + 1];
  // W2 as the two products' operands, lane by lane (element r of the float4
  // is k-step 4 t + r): [o][t] W2[16 o + c][16 t + 4 g + r], and
  // [t][u] W2[16 t + 4 g + r][16 u + c]
  __shared__ float4 w2f[kTiles][kTiles][kWave], w2b[kTiles][kTiles][kWave];
  __shared__ float part[kGradWaves / 2][kParams + 1];
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int c = lane & 15, g = lane >> 4;
  const int64_t chunk = (A.batch + gridDim.x - 1) / gridDim.x;
  const int64_t begin = (int64_t)blockIdx.x * chunk;
  const int64_t end = begin + chunk < A.batch ? begin + chunk : A.batch;
  int64_t base = begin + wave * kGroup;
  GradIn in = load_group(A, load_row(A, base, end));
  GradRow row = load_row(A, base + kPass, end);
  for (int p = tid; p < kParams; p += kGradThreads) w[p] = A.params[p];
  __syncthreads();
  for (int p = tid; p < kTiles * kTiles * kWave; p += kGradThreads) {
    const int x = p / (kTiles * kWave), y = p / kWave % kTiles;
    const float* f = w + kOffW2 + (16 * x + c) * kH + 16 * y + 4 * g;
    w2f[x][y][lane] = make_float4(f[0], f[1], f[2], f[3]);
    const float* b = w + kOffW2 + (16 * x + 4 * g) * kH + 16 * y + c;
    w2b[x][y][lane] = make_float4(b[0], b[kH], b[2 * kH], b[3 * kH]);
  }
  __syncthreads();

  float w1a[kTiles], w1b[kTiles], w3n[kTiles];  // W1 and b1 by unit c, feature g / 4 + g; w3
  f32x4 w3t[kTiles];                            // w3 of units 16 t + 4 g + r
  #pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    const int u = 16 * t + c;
    w1a[t] = w[kOffW1 + u * kIn + g];
    w1b[t] = g < kIn - 4 ? w[kOffW1 + u * kIn + 4 + g] : (g == kIn - 4 ? w[kOffB1 + u] : 0.0f);
    w3n[t] = w[kOffW3 + u];
    #pragma unroll
    for (int r = 0; r < 4; ++r) w3t[t][r] = w[kOffW3 + 16 * t + 4 * g + r];
  }
  const float b3 = w[kOffB3];
  const f32x4 zero = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 g1[kTiles], g2[kTiles][kTiles];  // dW1 (column 6: db1), dW2
  float gb2[kTiles], g3[kTiles][4];      // db2 by unit c; dw3 by sample and unit
  float gb3 = 0.0f, loss = 0.0f;
  #pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    g1[t] = zero;
    gb2[t] = 0.0f;
    #pragma unroll
    for (int o = 0; o < kTiles; ++o) g2[t][o] = zero;
    #pragma unroll
    for (int r = 0; r < 4; ++r) g3[t][r] = 0.0f;
  }

  while (base < end) {  // uniform in the wavefront
    // the operands are read from LDS in every step: held over the loop they
    // would not fit beside the gradients
    asm volatile("" ::: "memory");
    // the next group's inputs and the rows of the one after it are loaded
    // behind this one's products
    const GradIn ahead = load_group(A, row);
    row = load_row(A, base + 2 * kPass, end);
    // layer 1 in both forms
    f32x4 h1t[kTiles], h1n[kTiles];
    #pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      h1t[t] = mfma4(w1b[t], in.x1, mfma4(w1a[t], in.x0, zero));
      h1n[t] = mfma4(in.x1, w1b[t], mfma4(in.x0, w1a[t], zero));
      #pragma unroll
      for (int r = 0; r < 4; ++r) {
        h1t[t][r] = fmaxf(0.0f, h1t[t][r]);
        h1n[t][r] = fmaxf(0.0f, h1n[t][r]);
      }
    }
    // layer 2 and z
    f32x4 h2[kTiles];
    #pragma unroll
    for (int o = 0; o < kTiles; ++o) {
      const float* b2 = w + kOffB2 + 16 * o + 4 * g;
      h2[o] = (f32x4){b2[0], b2[1], b2[2], b2[3]};
    }
    #pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      f32x4 k[kTiles];
      #pragma unroll
      for (int o = 0; o < kTiles; ++o) k[o] = __builtin_bit_cast(f32x4, w2f[o][t][lane]);
      #pragma unroll
      for (int r = 0; r < 4; ++r)
        #pragma unroll
        for (int o = 0; o < kTiles; ++o) h2[o] = mfma4(k[o][r], h1t[t][r], h2[o]);
    }
    float zp = 0.0f;
    #pragma unroll
    for (int o = 0; o < kTiles; ++o)
      #pragma unroll
      for (int r = 0; r < 4; ++r) {
        h2[o][r] = fmaxf(0.0f, h2[o][r]);
        zp = fmaf(w3t[o][r], h2[o][r], zp);
      }
    zp += __shfl_xor(zp, 16);
    zp += __shfl_xor(zp, 32);
    const float z = zp + b3;
    const float yhat = softplus_f(z);
    const float uu = in.y - yhat;
    float dz = 0.0f;
    if (in.valid) {
      if (g == 0) loss += uu >= 0.0f ? A.q * uu : (A.q - 1.0f) * uu;
      const float dyhat = (yhat >= in.y ? 1.0f - A.q : -A.q) * A.inv_batch;
      dz = dyhat * sigmoid_f(z);
    }
    if (g == 0) gb3 += dz;
    float dzn[4];  // of samples 4 g + r
    #pragma unroll
    for (int r = 0; r < 4; ++r) dzn[r] = __shfl(dz, 4 * g + r);
    // D2 in both forms
    f32x4 d2t[kTiles], d2n[kTiles];
    #pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      uint64_t live[4];  // bit 16 g + c of live[r]: unit 16 t + 4 g + r of sample c
      #pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool on = h2[t][r] > 0.0f;
        live[r] = ballot(on);
        g3[t][r] = fmaf(dz, h2[t][r], g3[t][r]);
        d2t[t][r] = on ? dz * w3t[t][r] : 0.0f;
      }
      // this lane's unit 16 t + c, samples 4 g .. 4 g + 3
      const uint64_t lo = c & 1 ? live[1] : live[0], hi = c & 1 ? live[3] : live[2];
      const uint32_t bits = (uint32_t)((c & 2 ? hi : lo) >> (16 * (c >> 2) + 4 * g));
      #pragma unroll
      for (int r = 0; r < 4; ++r) {
        d2n[t][r] = (bits >> r) & 1u ? dzn[r] * w3n[t] : 0.0f;
        gb2[t] += d2n[t][r];
      }
    }
    // D1 = D2 W2, masked
    f32x4 d1n[kTiles];
    #pragma unroll
    for (int u = 0; u < kTiles; ++u) d1n[u] = zero;
    #pragma unroll
    for (int t = 0; t < kTiles; ++t) {
      f32x4 k[kTiles];
      #pragma unroll
      for (int u = 0; u < kTiles; ++u) k[u] = __builtin_bit_cast(f32x4, w2b[t][u][lane]);
      #pragma unroll
      for (int r = 0; r < 4; ++r)
        #pragma unroll
        for (int u = 0; u < kTiles; ++u) d1n[u] = mfma4(d2t[t][r], k[u][r], d1n[u]);
    }
    #pragma unroll
    for (int u = 0; u < kTiles; ++u)
      #pragma unroll
      for (int r = 0; r < 4; ++r) d1n[u][r] = h1n[u][r] > 0.0f ? d1n[u][r] : 0.0f;
    // the weight gradients over the samples
    #pragma unroll
    for (int r = 0; r < 4; ++r)
      #pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        #pragma unroll
        for (int u = 0; u < kTiles; ++u) g2[t][u] = mfma4(d2n[t][r], h1n[u][r], g2[t][u]);
        g1[t] = mfma4(d1n[t][r], in.xn[r], g1[t]);
      }
    in = ahead;
    base += kPass;
  }

  // the wavefront's sums: units 16 t + 4 g + r by column c of the MFMA
  // results, the rest reduced over the lanes that share a unit
  #pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    gb2[t] += __shfl_xor(gb2[t], 16);
    gb2[t] += __shfl_xor(gb2[t], 32);
    #pragma unroll
    for (int r = 0; r < 4; ++r)
      #pragma unroll
      for (int off = 1; off < 16; off <<= 1) g3[t][r] += __shfl_xor(g3[t][r], off);
  }
  #pragma unroll
  for (int off = 1; off < 16; off <<= 1) {
    gb3 += __shfl_xor(gb3, off);
    loss += __shfl_xor(loss, off);
  }
  // wavefront w + 4 adds its sums to those of wavefront w
  constexpr int kHalf = kGradWaves / 2;
  float* mine = part[wave % kHalf];
  for (int half = 0; half < 2; ++half) {
    if (wave / kHalf == half) {
      const auto put = [&](int p, float v) { mine[p] = half == 0 ? v : mine[p] + v; };
      #pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        if (g == 0) put(kOffB2 + 16 * t + c, gb2[t]);
        #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ut = 16 * t + 4 * g + r;
          if (c < kIn) put(kOffW1 + ut * kIn + c, g1[t][r]);
          if (c == kIn) put(kOffB1 + ut, g1[t][r]);
          #pragma unroll
          for (int u = 0; u < kTiles; ++u) put(kOffW2 + ut * kH + 16 * u + c, g2[t][u][r]);
          if (c == 0) put(kOffW3 + ut, g3[t][r]);
        }
      }
      if (lane == 0) {
        put(kOffB3, gb3);
        put(kParams, loss);
      }
    }
    __syncthreads();
  }
  float* out = A.partials + (int64_t)blockIdx.x * (kParams + 1);
  for (int p = tid; p <= kParams; p += kGradThreads) {
    float v = part[0][p];
    #pragma unroll
    for (int k = 1; k < kHalf; ++k) v += part[k][p];
    out[p] = v;
  }
}

// The workgroups' partial gradients summed in a fixed order: 64 parameters
// per workgroup (256-byte rows), their partials split over the wavefronts,
// each of which has a row of loads in flight at once.  4.8 MB at 256
// partials.  One thread per parameter walking all partials took 60 us, two
// dependent loads at a time; this takes 4.6 us (kernel trace).
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(kReduceWaves * kWave) void k_eps_reduce(
    const float* __restrict__ partials, int blocks, float inv_batch, float* __restrict__ grad,
    float* __restrict__ loss) {
  __shared__ float sums[kReduceWaves][kWave];
  const int lane = lane_id(), wave = wave_id();
  const int p = (int)blockIdx.x * kWave + lane;
  constexpr int kFly = kEpsGradMaxBlocks / kReduceWaves;  // partials per wavefront at most
  const int per = (blocks + kReduceWaves - 1) / kReduceWaves;
  float v[kFly];
  #pragma unroll
  for (int k = 0; k < kFly; ++k) {
    const int b = wave * per + k;
    v[k] = k < per && b < blocks && p <= kParams ? partials[(int64_t)b * (kParams + 1) + p] : 0.0f;
  }
  float a = 0.0f;
  #pragma unroll
  for (int k = 0; k < kFly; ++k) a += v[k];
  sums[wave][lane] = a;
  __syncthreads();
  if (wave != 0 || p > kParams) return;
  a = sums[0][lane];
  #pragma unroll
  for (int k = 1; k < kReduceWaves; ++k) a += sums[k][lane];
  if (p < kParams) grad[p] = a;
  else if (loss) *loss = a * inv_batch;
}

__global__ void k_eps_adam(float* __restrict__ theta, float* __restrict__ m,
                           float* __restrict__ v, const float* __restrict__ grad, float lr,
                           float beta1, float beta2, float eps, float c1, float c2) {
  const int p = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (p >= kParams) return;
  const float g = grad[p];
  const float mm = beta1 * m[p] + (1.0f - beta1) * g;
  const float vv = beta2 * v[p] + (1.0f - beta2) * g * g;
  m[p] = mm;
  v[p] = vv;
  theta[p] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

// --------------------------------------------------------------- residuals
__global__ __launch_bounds__(256) void k_residuals(const PairDev* __restrict__ pairs,
                                                   const int64_t* __restrict__ qstart,
                                                   int num_pairs, int64_t n1,
                                                   const float* __restrict__ kp1,
                                                   const float* __restrict__ kp2,
                                                   const int32_t* __restrict__ best,
                                                   float* __restrict__ residual,
                                                   int64_t* __restrict__ feat_index) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n1) return;
  const PairDev& pd = pairs[find_pair(qstart, num_pairs, i)];
  const int32_t j = best[i];
  if (j < 0 || j >= pd.n) {
    residual[i] = -1.0f;
    if (feat_index) feat_index[i] = -1;
    return;
  }
  double a, b, c;
  epipolar_line(pd.F, kp1[2 * i], kp1[2 * i + 1], a, b, c);
  const int64_t g = pd.k_begin + j;
  const double num = fabs(__dadd_rn(__dadd_rn(__dmul_rn(a, (double)kp2[2 * g]),
                                              __dmul_rn(b, (double)kp2[2 * g + 1])), c));
  const double den = __dsqrt_rn(__dadd_rn(__dmul_rn(a, a), __dmul_rn(b, b)));
  residual[i] = (float)__ddiv_rn(num, den);
  if (feat_index) feat_index[i] = g;
}

}  // namespace

hipError_t launch_eps_features(const EpsPair* pairs, const int64_t* kstart, int num_pairs,
                               int64_t n2, const float* kp2, const float* attrs, float* out,
                               hipStream_t s) {
  if (n2 == 0) return hipSuccess;
  const int64_t blocks = (n2 + kFeatThreads - 1) / kFeatThreads;
  hipLaunchKernelGGL(k_eps_features, dim3((unsigned)blocks), dim3(kFeatThreads), 0, s, pairs,
                     kstart, num_pairs, n2, kp2, attrs, out);
  return hipGetLastError();
}

hipError_t launch_eps_infer(const float* feat, int64_t n, const float* params, float* eps,
                            hipStream_t s) {
  if (n == 0) return hipSuccess;
  int64_t blocks = (n + kInferThreads - 1) / kInferThreads;
  if (blocks > kInferBlocks) blocks = kInferBlocks;
  hipLaunchKernelGGL(k_eps_infer, dim3((unsigned)blocks), dim3(kInferThreads), 0, s, feat, n,
                     params, eps);
  return hipGetLastError();
}

int eps_grad_blocks(int64_t batch) {
  const int64_t b = (batch + kBlockSamples - 1) / kBlockSamples;
  return (int)(b < kEpsGradMaxBlocks ? (b > 0 ? b : 1) : kEpsGradMaxBlocks);
}

hipError_t launch_eps_grad(const EpsGradArgs& a, float* grad, float* loss, hipStream_t s) {
  const int blocks = eps_grad_blocks(a.batch);
  hipLaunchKernelGGL(k_eps_grad, dim3(blocks), dim3(kGradThreads), 0, s, a);
  hipLaunchKernelGGL(k_eps_reduce, dim3((kParams + kWave) / kWave), dim3(kReduceWaves * kWave), 0,
                     s, a.partials, blocks, a.inv_batch, grad, loss);
  return hipGetLastError();
}

hipError_t launch_eps_adam(float* theta, float* m, float* v, const float* grad, float lr,
                           float beta1, float beta2, float eps, float c1, float c2,
                           hipStream_t s) {
  hipLaunchKernelGGL(k_eps_adam, dim3((kParams + 255) / 256), dim3(256), 0, s, theta, m, v, grad,
                     lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_residuals(const PairDev* pairs, const int64_t* qstart, int num_pairs,
                            int64_t n1, const float* kp1, const float* kp2, const int32_t* best,
                            float* residual, int64_t* feat_index, hipStream_t s) {
  if (n1 == 0) return hipSuccess;
  const int64_t blocks = (n1 + 255) / 256;
  hipLaunchKernelGGL(k_residuals, dim3((unsigned)blocks), dim3(256), 0, s, pairs, qstart,
                     num_pairs, n1, kp1, kp2, best, residual, feat_index);
  return hipGetLastError();
}

}  // namespace epm
