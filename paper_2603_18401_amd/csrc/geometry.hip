// Angular intervals of the image-2 tolerance circles and the angle keys of
// the image-1 epipolar lines.
//
// Sec. 4.1-4.2 (Eq. 5-6): seen from the epipole, the circle of radius eps_j
// around p_j subtends the interval of line directions between its two
// tangents.  The kernels express line directions in a pencil basis (u, v) of
// the lines through the epipole e (u, v, e orthonormal in normalised line
// space), which covers a finite epipole inside or outside the image and an
// epipole at infinity with one formula: the pencil line at angle phi is
// l(phi) = cos(phi) u + sin(phi) v, and p_j lies within eps of it iff
//     (w_j . c)^2 <= eps^2 c^T G c,   c = (cos phi, sin phi),
// with w_j = (u . p~_j, v . p~_j) and G the Gram matrix of (u_12, v_12).
// The solution set is the arc around the eigenvector of the negative
// eigenvalue of M_j = w_j w_j^T - eps^2 G, half-width atan(sqrt(-l-/l+));
// with an orthonormal basis of a finite epipole this is theta_j +- delta_j of
// Eq. 5-6.  A circle containing the epipole gives a negative semidefinite
// M_j: the full interval (Sec. 4.4).  Angles are stored mod pi as u32 keys,
// which makes the 0/pi wrap-around implicit.
#include "device_common.h"
#include "launch.h"

namespace epm {

namespace {

// Conservative interval of one keypoint: centre key and half-width key.
__device__ void circle_interval(const PairDev& pd, float xf, float yf, float ef, uint32_t& C,
                                uint32_t& H) {
  if (pd.kappa < 0.0) {  // no pencil: the pair's queries scan every record
    C = 0;
    H = kFullHalf;
    return;
  }
  const double px = pd.s * ((double)xf - pd.cx);
  const double py = pd.s * ((double)yf - pd.cy);
  const double w1 = pd.u[0] * px + pd.u[1] * py + pd.u[2];
  const double w2 = pd.v[0] * px + pd.v[1] * py + pd.v[2];
  const double ep = fabs(pd.e[0] * px + pd.e[1] * py + pd.e[2]);
  // tolerance in normalised units, inflated by the rounding slack and by the
  // largest line-to-epipole miss a query may have before it scans the pair
  double epsn = pd.s * ((double)ef * (1.0 + kEpsRelSlack) + kEpsAbsSlackPx);
  epsn += pd.kappa * (epsn * pd.e12 + ep);
  const double e2 = epsn * epsn;
  const double A = w1 * w1 - e2 * pd.G11;
  const double B = w1 * w2 - e2 * pd.G12;
  const double D = w2 * w2 - e2 * pd.G22;
  const double detG = pd.G11 * pd.G22 - pd.G12 * pd.G12;
  const double wadj = pd.G22 * w1 * w1 - 2.0 * pd.G12 * w1 * w2 + pd.G11 * w2 * w2;
  const double det = e2 * (e2 * detG - wadj);  // det M without cancellation
  if (!(det < 0.0)) {
    // both eigenvalues <= 0: the circle holds the epipole, every line hits it
    // (a positive definite M cannot occur; it is also treated as full)
    C = 0;
    H = kFullHalf;
    return;
  }
  const double half = 0.5 * (A - D);
  const double disc = sqrt(half * half + B * B);
  const double lp = 0.5 * (A + D) + disc;  // > 0
  const double lm = det / lp;              // < 0
  double vx, vy;                           // eigenvector of lp
  if (A >= D) {
    vx = half + disc;
    vy = B;
  } else {
    vx = B;
    vy = disc - half;
  }
  // interval centre: the eigenvector of lm, (-vy, vx)
  const double psi = atan2(vx, -vy);
  const double h = atan(sqrt(-lm / lp));
  const double hk = ceil(h * kKeyPerRad) + (double)kGuard;
  if (!(hk < (double)(kFullHalf - 2 * kGuard))) {
    C = 0;
    H = kFullHalf;
    return;
  }
  C = angle_key(psi) - pd.arc.cut;
  H = (uint32_t)hk;
}

}  // namespace

// ------------------------------------------------------------ pair setup
// Algorithm 1, preprocessing, on the device: the image-2 epipole e2 = null(F^T)
// in normalised line coordinates and an orthonormal basis (u, v) of the
// pencil of lines through it, from F in device memory (one thread per pair).
// The normalisation (s, cx, cy from the image size) and the slices are kept
// from the pair record.  A pair without a pencil (F non-finite, zero, or of
// rank <= 1) gets kappa = -1: its queries are then tested against every
// keypoint of the pair, which keeps the result exact.
__device__ __forceinline__ void dcross(const double* a, const double* b, double* r) {
  r[0] = a[1] * b[2] - a[2] * b[1];
  r[1] = a[2] * b[0] - a[0] * b[2];
  r[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ double dnorm3(const double* a) {
  return sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
}

__device__ bool pencil_of(PairDev& pd) {
  const double* F = pd.F;
  double fn = 0.0;
  for (int k = 0; k < 9; ++k) {
    if (!isfinite(F[k])) return false;
    fn += F[k] * F[k];
  }
  if (!(fn > 0.0) || !isfinite(fn)) return false;
  // M = N F T^-1 (lines in normalised image-2 coordinates as functions of
  // normalised image-1 coordinates), scaled to a largest entry of 1
  double M[3][3];
  const double is = 1.0 / pd.s;
  double mx = 0.0;
  for (int r = 0; r < 3; ++r) {
    double NF[3];
    for (int k = 0; k < 3; ++k)
      NF[k] = r == 0 ? F[k] : r == 1 ? F[3 + k] : pd.s * (F[k] * pd.cx + F[3 + k] * pd.cy + F[6 + k]);
    // T^-1 = [[1/s, 0, cx], [0, 1/s, cy], [0, 0, 1]]
    M[r][0] = NF[0] * is;
    M[r][1] = NF[1] * is;
    M[r][2] = NF[0] * pd.cx + NF[1] * pd.cy + NF[2];
    for (int k = 0; k < 3; ++k) mx = fmax(mx, fabs(M[r][k]));
  }
  if (!(mx > 0.0) || !isfinite(mx)) return false;
  double col[3][3];
  for (int k = 0; k < 3; ++k)
    for (int d = 0; d < 3; ++d) col[k][d] = M[d][k] / mx;
  // the left null vector is orthogonal to every column: the largest cross
  // product of two columns
  double best[3] = {0.0, 0.0, 0.0}, bn = 0.0;
  const int pa[3] = {0, 0, 1}, pb[3] = {1, 2, 2};
  for (int t = 0; t < 3; ++t) {
    double cr[3];
    dcross(col[pa[t]], col[pb[t]], cr);
    const double cn = dnorm3(cr);
    if (cn > bn) {
      bn = cn;
      for (int d = 0; d < 3; ++d) best[d] = cr[d];
    }
  }
  if (!(bn > 1e-12)) return false;
  for (int d = 0; d < 3; ++d) pd.e[d] = best[d] / bn;
  int ax = 0;
  for (int d = 1; d < 3; ++d)
    if (fabs(pd.e[d]) < fabs(pd.e[ax])) ax = d;
  double axis[3] = {0.0, 0.0, 0.0};
  axis[ax] = 1.0;
  dcross(pd.e, axis, pd.u);
  const double un = dnorm3(pd.u);
  for (int d = 0; d < 3; ++d) pd.u[d] /= un;
  dcross(pd.e, pd.u, pd.v);
  const double vn = dnorm3(pd.v);
  for (int d = 0; d < 3; ++d) pd.v[d] /= vn;
  pd.G11 = pd.u[0] * pd.u[0] + pd.u[1] * pd.u[1];
  pd.G12 = pd.u[0] * pd.v[0] + pd.u[1] * pd.v[1];
  pd.G22 = pd.v[0] * pd.v[0] + pd.v[1] * pd.v[1];
  pd.e12 = sqrt(pd.e[0] * pd.e[0] + pd.e[1] * pd.e[1]);
  pd.kappa = kKappaBuild;
  return true;
}

__global__ __launch_bounds__(64) void k_pair_setup(PairDev* __restrict__ pairs,
                                                   const double* __restrict__ F, int num_pairs) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= num_pairs) return;
  PairDev pd = pairs[p];
  for (int k = 0; k < 9; ++k) pd.F[k] = F[9 * (int64_t)p + k];
  if (!pencil_of(pd)) {
    // no pencil: every query scans its pair, every record is a full interval
    for (int d = 0; d < 3; ++d) pd.u[d] = pd.v[d] = pd.e[d] = 0.0;
    pd.G11 = pd.G12 = pd.G22 = pd.e12 = 0.0;
    pd.kappa = -1.0;
  }
  set_key_arc(pd);
  pairs[p] = pd;
}

// The digit counts of the first radix pass of the keys this workgroup wrote
// (its tile, in LDS), as the sort reads them.  A segment of one tile counts
// for itself.
__device__ __forceinline__ void first_pass_counts(const uint32_t* h, const SortSeg& sg,
                                                  uint32_t* __restrict__ hist) {
  if (sg.tile_count < 2) return;  // uniform
  __syncthreads();
  const int tid = threadIdx.x;
  hist[(int64_t)(sg.hist_begin + (int)blockIdx.x - sg.tile_begin) * kHistWords + tid] =
      h[2 * tid] | (h[2 * tid + 1] << 16);
}

// One workgroup per record sort tile.
__global__ __launch_bounds__(kSortThreads) void k_intervals(
    const PairDev* __restrict__ pairs, const SortTile* __restrict__ tiles,
    const SortSeg* __restrict__ segs, const float* __restrict__ kp2,
    const float* __restrict__ eps2, float eps_scalar, uint32_t* __restrict__ sort_key,
    uint32_t* __restrict__ recC, uint32_t* __restrict__ recH, uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kRadix];
  h[2 * threadIdx.x] = h[2 * threadIdx.x + 1] = 0u;
  __syncthreads();
  const SortTile t = tiles[blockIdx.x];
  const PairDev& pd = pairs[t.seg];
  const KeyArc arc = pd.arc;  // (loaded before the geometry)
  for (int k = threadIdx.x; k < t.count; k += kSortThreads) {
    const int64_t r = t.begin + k;
    const float xf = kp2[2 * r], yf = kp2[2 * r + 1];
    const float ef = eps2 ? eps2[r] : eps_scalar;
    uint32_t C = 0, H = kFullHalf;
    // keypoints the interval formula cannot describe are always scanned and
    // left to the exact test
    if (ef > 0.0f && isfinite(ef) && isfinite(xf) && isfinite(yf))
      circle_interval(pd, xf, yf, ef, C, H);
    const uint32_t cls = (uint32_t)width_class(H);
    const uint32_t key = (cls << kCentreBits) | position_code(arc, C);
    sort_key[r] = key;
    recC[r] = C;
    recH[r] = H;
    atomicAdd(&h[key & (kRadix - 1)], 1u);
  }
  first_pass_counts(h, segs[t.seg], hist);
}

// Eq. 2 and Eq. 7: the angle of each query's epipolar line in the pencil,
// reduced mod pi (an undirected line).
// One workgroup per query sort tile.  shift: that of the sort's first pass.
__global__ __launch_bounds__(kSortThreads) void k_query_keys(
    const PairDev* __restrict__ pairs, const SortTile* __restrict__ tiles,
    const SortSeg* __restrict__ segs, const float* __restrict__ kp1, uint32_t* __restrict__ qkey,
    uint32_t* __restrict__ qflag, uint32_t* __restrict__ sort_key, double4* __restrict__ qline,
    int shift, uint32_t* __restrict__ hist, unsigned long long* __restrict__ stats,
    uint32_t* __restrict__ sched, unsigned long long* __restrict__ match_stats) {
  __shared__ uint32_t h[kRadix];
  h[2 * threadIdx.x] = h[2 * threadIdx.x + 1] = 0u;
  if (blockIdx.x == 0) {  // the query's counters start from zero
    if (stats && threadIdx.x < kNumStats) stats[threadIdx.x] = 0ull;
    if (match_stats && threadIdx.x < kMatchStatWords) match_stats[threadIdx.x] = 0ull;
    if (sched)
      for (int k = (int)threadIdx.x; k < kSchedWords; k += (int)blockDim.x) sched[k] = 0u;
  }
  __syncthreads();
  const SortTile t = tiles[blockIdx.x];
  const PairDev& pd = pairs[t.seg];
  const KeyArc arc = pd.arc;  // (loaded before the geometry)
  for (int kk = threadIdx.x; kk < t.count; kk += kSortThreads) {
    const int64_t i = t.begin + kk;
    double a, b, c;
    epipolar_line(pd.F, kp1[2 * i], kp1[2 * i + 1], a, b, c);
    uint32_t flag = kQueryNormal, key = 0;
    if (a == 0.0 && b == 0.0) {
      flag = kQueryEmpty;
    } else if (!isfinite(a) || !isfinite(b) || !isfinite(c)) {
      flag = kQueryBrute;
    } else {
      // the same line in normalised image-2 coordinates (scaled by 1/s)
      const double l3 = pd.s * (a * pd.cx + b * pd.cy + c);
      const double lam = pd.u[0] * a + pd.u[1] * b + pd.u[2] * l3;
      const double mu = pd.v[0] * a + pd.v[1] * b + pd.v[2] * l3;
      const double nu = pd.e[0] * a + pd.e[1] * b + pd.e[2] * l3;
      const double n1c = lam * pd.u[0] + mu * pd.v[0];
      const double n2c = lam * pd.u[1] + mu * pd.v[1];
      const double nrm = sqrt(n1c * n1c + n2c * n2c);
      if (pd.kappa < 0.0 || !(fabs(nu) <= pd.kappa * nrm)) {
        flag = kQueryBrute;  // the line misses the epipole by more than absorbed
      } else {
        key = angle_key(atan2(mu, lam)) - arc.cut;
      }
    }
    qkey[i] = key;
    qflag[i] = flag;
    const uint32_t sk = position_code(arc, key) << kClassBits;
    sort_key[i] = sk;
    // the line and its norm for the tile passes (the denominator of Eq. 3)
    qline[i] = flag == kQueryEmpty ? make_double4(0.0, 0.0, 0.0, 0.0)
                                   : make_double4(a, b, c, line_norm(a, b));
    atomicAdd(&h[(sk >> shift) & (kRadix - 1)], 1u);
  }
  first_pass_counts(h, segs[t.seg], hist);
}

// Start of every width class inside each pair's sorted segment.
__global__ __launch_bounds__(64) void k_class_bounds(const int64_t* __restrict__ kstart,
                                                     const uint32_t* __restrict__ skey,
                                                     int64_t* __restrict__ class_begin) {
  const int p = blockIdx.x;
  const int64_t lo = kstart[p], hi = kstart[p + 1];
  const int c = lane_id();
  // every lane runs the same cooperative search for its own class in turn
  for (int cc = 0; cc < kClassSlots; ++cc) {
    const int64_t b = cc == kNumClasses ? hi : wave_lower_bound(skey, lo, hi, (uint32_t)cc << kCentreBits);
    if (c == 0) class_begin[(int64_t)p * kClassSlots + cc] = b;
  }
}

hipError_t launch_pair_setup(PairDev* pairs, const double* F, int num_pairs, hipStream_t s) {
  if (num_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_pair_setup, dim3((unsigned)((num_pairs + 63) / 64)), dim3(64), 0, s, pairs,
                     F, num_pairs);
  return hipGetLastError();
}

hipError_t launch_intervals(const PairDev* pairs, const SortCall& c, const float* kp2,
                            const float* eps2, float eps_scalar, uint32_t* recC, uint32_t* recH,
                            hipStream_t s) {
  if (c.num_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_intervals, dim3((unsigned)c.num_tiles), dim3(kSortThreads), 0, s, pairs,
                     c.tiles, c.segs, kp2, eps2, eps_scalar, c.k0, recC, recH, c.hist0);
  return hipGetLastError();
}

hipError_t launch_query_keys(const PairDev* pairs, const SortCall& c, bool two_passes,
                             const float* kp1, uint32_t* qkey, uint32_t* qflag, double4* qline,
                             unsigned long long* stats, uint32_t* sched,
                             unsigned long long* match_stats, hipStream_t s) {
  if (c.num_tiles == 0) return launch_clear_stats(stats, s, sched, match_stats);
  hipLaunchKernelGGL(k_query_keys, dim3((unsigned)c.num_tiles), dim3(kSortThreads), 0, s, pairs,
                     c.tiles, c.segs, kp1, qkey, qflag, c.k0, qline, two_passes ? 0 : kRadixBits,
                     c.hist0, stats, sched, match_stats);
  return hipGetLastError();
}

hipError_t launch_class_bounds(const int64_t* kstart, int num_pairs, const uint32_t* skey,
                               int64_t* class_begin, hipStream_t s) {
  if (num_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_class_bounds, dim3(num_pairs), dim3(64), 0, s, kstart, skey, class_begin);
  return hipGetLastError();
}

}  // namespace epm
