// Device helpers shared by the libepm kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "epm_internal.h"

namespace epm {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }
__device__ __forceinline__ int wave_id() { return (int)(threadIdx.x >> 6); }

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  This maps dispatch order to a logical tile order in which groups of
// kXcdGroup consecutive logical tiles -- neighbouring angle ranges that share
// candidates -- run on one XCD, while successive groups rotate over the XCDs
// so uneven work stays balanced.  A bijection of [0, n): the tail that does
// not fill a whole round of groups keeps the identity order.
constexpr int kNumXcd = 8;
constexpr int kXcdGroup = 16;
__device__ __forceinline__ int xcd_tile(int block, int n) {
  constexpr int round = kNumXcd * kXcdGroup;
  const int full = (n / round) * round;
  if (block >= full) return block;
  const int x = block % kNumXcd, k = block / kNumXcd;
  const int g = k / kXcdGroup, o = k % kXcdGroup;
  return (g * kNumXcd + x) * kXcdGroup + o;
}

// XCD that xcd_tile gives tile t: the inverse of the mapping above, mod 8.
__device__ __forceinline__ int xcd_of_tile(int t, int n) {
  constexpr int round = kNumXcd * kXcdGroup;
  const int full = (n / round) * round;
  return t >= full ? t % kNumXcd : (t / kXcdGroup) % kNumXcd;
}

// Cost bucket of the longest-first orders: 0 for no work, else two buckets
// per power of two (the bit below the leading one splits an octave).
__device__ __forceinline__ int cost_bucket(uint32_t c) {
  if (c == 0) return 0;
  const int msb = 31 - __clz(c);
  const int half = msb > 0 ? (int)((c >> (msb - 1)) & 1u) : 0;
  return 1 + 2 * msb + half;
}

// Number of set bits of `mask` below this lane.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                   __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

// Last pair p with starts[p] <= idx (pairs own contiguous, ordered slices).
__device__ __forceinline__ int find_pair(const int64_t* __restrict__ starts, int num_pairs,
                                         int64_t idx) {
  int lo = 0, hi = num_pairs - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (starts[mid] <= idx) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Eq. 2: the epipolar line of (x, y), every product and sum rounded once,
// left to right -- the same operations as the definition of the candidate set.
__device__ __forceinline__ void epipolar_line(const double* __restrict__ F, float xf, float yf,
                                              double& a, double& b, double& c) {
  const double x = (double)xf, y = (double)yf;
  a = __dadd_rn(__dadd_rn(__dmul_rn(F[0], x), __dmul_rn(F[1], y)), F[2]);
  b = __dadd_rn(__dadd_rn(__dmul_rn(F[3], x), __dmul_rn(F[4], y)), F[5]);
  c = __dadd_rn(__dadd_rn(__dmul_rn(F[6], x), __dmul_rn(F[7], y)), F[8]);
}

// sqrt(a^2 + b^2) of a line, correctly rounded (the denominator of Eq. 3).
__device__ __forceinline__ double line_norm(double a, double b) {
  return __dsqrt_rn(__dadd_rn(__dmul_rn(a, a), __dmul_rn(b, b)));
}

// Eq. 3-4 multiplied through by sqrt(a^2 + b^2): the only FP64 step of the
// per-candidate path.  Closed boundary.  nrm = line_norm(a, b), computed once
// per query; the decision is the same bit for bit as with the norm inline.
__device__ __forceinline__ bool within_tolerance_d(double a, double b, double c, double nrm,
                                                   double x, double y, double e) {
  const double num = fabs(__dadd_rn(__dadd_rn(__dmul_rn(a, x), __dmul_rn(b, y)), c));
  return num <= __dmul_rn(e, nrm);
}

// (x, y, eps) are FP32 inputs widened exactly.
__device__ __forceinline__ bool within_tolerance_n(double a, double b, double c, double nrm,
                                                   float xf, float yf, float ef) {
  return within_tolerance_d(a, b, c, nrm, (double)xf, (double)yf, (double)ef);
}

__device__ __forceinline__ bool within_tolerance(double a, double b, double c, float xf,
                                                 float yf, float ef) {
  return within_tolerance_n(a, b, c, line_norm(a, b), xf, yf, ef);
}

// Circular distance between two angle keys (mod 2^32 == mod pi).
__device__ __forceinline__ uint32_t key_distance(uint32_t p, uint32_t c) {
  const uint32_t d = p - c;
  const uint32_t e = c - p;
  return d < e ? d : e;
}

__device__ __forceinline__ int width_class(uint32_t half) {
  const int c = 32 - __clz(half);
  return c > kWideClass ? kWideClass : c;
}

// First index in [lo, hi) whose key is >= target (keys ascending); the whole
// wavefront cooperates, every lane gets the result.
__device__ __forceinline__ int64_t wave_lower_bound(const uint32_t* __restrict__ keys,
                                                    int64_t lo, int64_t hi, uint32_t target) {
  const int lane = lane_id();
  while (hi - lo > kWave) {
    const int64_t len = hi - lo;
    // 64 probes splitting [lo, hi) into 65 parts
    const int64_t pos = lo + (len * (lane + 1)) / (kWave + 1);
    const bool below = keys[pos] < target;
    const uint64_t m = ballot(below);
    const int cnt = __popcll(m);  // probes are ascending: a prefix is below
    const int64_t nlo = cnt == 0 ? lo : lo + (len * cnt) / (kWave + 1) + 1;
    const int64_t nhi = cnt == kWave ? hi : lo + (len * (cnt + 1)) / (kWave + 1) + 1;
    lo = nlo;
    hi = nhi < hi ? nhi : hi;
  }
  const int64_t pos = lo + lane;
  const bool below = pos < hi && keys[pos] < target;
  return lo + __popcll(ballot(below));
}

// Data of another lane by DPP: one vector instruction, where a shuffle through
// LDS takes a hundred cycles.  Lanes that have no neighbour in a step get `none`.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t none, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)v, CTRL, ROWS, 0xF, false);
}

// Value of lane l ^ J: DPP within a row of 16 lanes, swaps of rows (halves) of
// two copies beyond.
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  if constexpr (J == 1) return dpp<0xB1, 0xF>(v, v);
  else if constexpr (J == 2) return dpp<0x4E, 0xF>(v, v);
  else if constexpr (J == 4) return dpp<0x1B, 0xF>(v, dpp<0x141, 0xF>(v, v));  // ^ 7, then ^ 3
  else if constexpr (J == 8) return dpp<0x128, 0xF>(v, v);                     // rotate by 8
  else if constexpr (J == 16) {
    // odd rows of the first with even rows of the second: rows 0 0 2 2 | 1 1 3 3
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (lane_id() & 16) ? r[0] : r[1];
  } else {
    static_assert(J == 32, "one lane bit");
    // upper half of the first with the lower half of the second
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (lane_id() & 32) ? r[0] : r[1];
  }
}
template <int J>
__device__ __forceinline__ int32_t lane_xor(int32_t v) {
  return (int32_t)lane_xor<J>((uint32_t)v);
}
template <int J>
__device__ __forceinline__ float lane_xor(float v) {
  return __uint_as_float(lane_xor<J>(__float_as_uint(v)));
}
template <int J>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v) {
  return ((uint64_t)lane_xor<J>((uint32_t)(v >> 32)) << 32) | lane_xor<J>((uint32_t)v);
}

// Row g of 16 lanes in every row.
template <int G>
__device__ __forceinline__ uint32_t row_bcast(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const uint32_t w = r[G & 1];  // rows G & 1 and 2 + (G & 1), twice each
  const auto h = __builtin_amdgcn_permlane32_swap(w, w, false, false);
  return h[G >> 1];
}

// Reductions over the wavefront (uniform results), over each row of 16 lanes
// and inclusive sums, by DPP.
template <class OP>
__device__ __forceinline__ uint32_t row_reduce(uint32_t v, uint32_t none, OP op) {
  v = op(v, dpp<0xB1, 0xF>(none, v));   // quad [1,0,3,2]
  v = op(v, dpp<0x4E, 0xF>(none, v));   // quad [2,3,0,1]
  v = op(v, dpp<0x141, 0xF>(none, v));  // half-row mirror
  v = op(v, dpp<0x140, 0xF>(none, v));  // row mirror
  return v;
}

template <class OP>
__device__ __forceinline__ uint32_t wave_reduce(uint32_t v, uint32_t none, OP op) {
  v = row_reduce(v, none, op);
  // rows 1 and 3 take lane 15 of the row below, rows 2 and 3 lane 31; lane 63
  // ends with all rows
  v = op(v, dpp<0x142, 0xA>(none, v));
  v = op(v, dpp<0x143, 0xC>(none, v));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, kWave - 1);
}

struct OpSum {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; }
};
struct OpMin {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a < b ? a : b; }
};
struct OpMax {
  __device__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; }
};

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) { return wave_reduce(v, 0u, OpSum()); }
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  return wave_reduce(v, 0xFFFFFFFFu, OpMin());
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) { return wave_reduce(v, 0u, OpMax()); }

__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
  v += dpp<0x111, 0xF>(0u, v);  // one, two, four and eight lanes below, in the row
  v += dpp<0x112, 0xF>(0u, v);
  v += dpp<0x114, 0xF>(0u, v);
  v += dpp<0x118, 0xF>(0u, v);
  v += dpp<0x142, 0xA>(0u, v);
  v += dpp<0x143, 0xC>(0u, v);
  return v;
}

}  // namespace epm
