// Stabbing query (Sec. 4.2, Algorithm 1 match loop): every query's angle key
// is tested against the angle-sorted intervals of its pair; each angular hit
// is confirmed by the FP64 point-line test (Eq. 3), so the rows are exactly
// the candidate sets of Eq. 4.
//
// Queries are taken in tiles of kTileQ angle-sorted queries of one pair.  For
// width class c the only centres that can hold a key lie within 2^c - 1 key
// units of it, so the window pass finds each tile's record window in every
// class; the tile pass tests every (query, record) pair of the window, writes
// the row lengths and parks short rows.  After the scan of the lengths the
// parked rows are copied and the long rows of brute-force queries rebuilt one
// wavefront per query (scan, LDS sort by j); long rows of normal queries are
// written tile by tile by the wide-row pass.  The tile pass can
// also select every short row's match (Sec. 4.3) while its hits are on chip:
// FP32 chains, or MFMA bounds over BF16 or FP8 rows with an exact FP32
// re-rank.
#include "device_common.h"
#include "launch.h"
#include "match_common.h"
#include "mfma_bounds.h"

namespace epm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;
constexpr int kFinishRows = 256;  // queries per workgroup of k_finish_rows

// Bitonic sort of one value per lane, ascending over the wavefront (21
// exchanges, 18 of them by DPP).
template <int K, int J, typename T>
__device__ __forceinline__ void sort_step(T& v, int lane) {
  const T o = lane_xor<J>(v);
  const bool low = ((lane & K) == 0) == ((lane & J) == 0);
  v = (o < v) == low ? o : v;
  if constexpr (J > 1) sort_step<K, J / 2>(v, lane);
  else if constexpr (K < kWave) sort_step<2 * K, K>(v, lane);
}
template <typename T>
__device__ __forceinline__ T wave_sort64(T v) {
  sort_step<2, 1>(v, lane_id());
  return v;
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bitonic sort of buf[0..len) (len a power of two, 128..kRowSortMax) by one
// wavefront.
__device__ void wave_sort_lds(int32_t* buf, int len) {
  const int lane = lane_id();
  for (int k = 2; k <= len; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int t = lane; t < len / 2; t += kWave) {
        // comparator t: element pair (lo, lo + j)
        const int lo = ((t / j) * 2 * j) + (t % j);
        const int hi = lo + j;
        const bool up = (lo & k) == 0;
        const int32_t a = buf[lo], b = buf[hi];
        if ((a > b) == up) {
          buf[lo] = b;
          buf[hi] = a;
        }
      }
      wave_sync_lds();
    }
  }
}

// Position of the k-th set bit (k from 0) of w, which has more than k bits set.
__device__ __forceinline__ int nth_bit(uint64_t w, uint32_t k) {
  const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
  const uint32_t below = (uint32_t)__popc(lo);
  const bool up = k >= below;
  uint32_t x = up ? hi : lo;
  k = up ? k - below : k;
  int pos = up ? 32 : 0;
  #pragma unroll
  for (int half = 16; half > 0; half >>= 1) {
    const uint32_t c = (uint32_t)__popc(x & ((1u << half) - 1u));
    const bool u = k >= c;
    k = u ? k - c : k;
    x = u ? x >> half : x;
    pos += u ? half : 0;
  }
  return pos;
}

struct QueryCtx {
  double a, b, c;
  uint32_t key;
  bool brute;
};

// First index in [lo, hi) whose key is >= target (keys ascending), by one
// lane: seven probes in flight per step cut the range to an eighth.
__device__ __forceinline__ int64_t lower_bound_scalar(const uint32_t* __restrict__ keys,
                                                      int64_t lo, int64_t hi, uint32_t target) {
  // the answer lies in [lo, hi]
  while (hi - lo > 8) {
    const int64_t step = (hi - lo) / 8;
    uint32_t k[7];
    #pragma unroll
    for (int m = 0; m < 7; ++m) k[m] = keys[lo + (m + 1) * step];
    int c = 0;  // the probes below the target are a prefix
    #pragma unroll
    for (int m = 0; m < 7; ++m) c += k[m] < target ? 1 : 0;
    const int64_t nlo = c == 0 ? lo : lo + c * step + 1;
    const int64_t nhi = c == 7 ? hi : lo + (c + 1) * step;
    lo = nlo;
    hi = nhi;
  }
  int c = 0;
  #pragma unroll
  for (int m = 0; m < 8; ++m) c += lo + m < hi && keys[lo + m] < target ? 1 : 0;
  return lo + c;
}

// The record ranges of the pair that can meet the keys [kmin, kmax]: every
// width class's centres within [kmin - 2^c + 1, kmax + 2^c - 1], as slots.  Slot
// s = lane is part s % 2 of class s / 2 (the second part only where the range
// runs through the pair's cut); returns this lane's slot, its begin in `begin`
// and its length as the result.  Lane c < 32 searches the start of class c's
// range, lane c + 32 its end: all searches run side by side.
__device__ __forceinline__ uint32_t class_ranges(const StabArgs& A, const PairDev& pd, int pair,
                                                 uint32_t kmin, uint32_t kmax, bool any,
                                                 uint32_t& begin) {
  const int lane = lane_id();
  const int c = lane & (kNumClasses - 1);
  static_assert(2 * kNumClasses == kWave, "two lanes per width class");
  int64_t beg = 0, end = 0, r = 0;
  bool full = false, wrap = false;
  if (any) {
    const int64_t* cb = A.class_begin + (int64_t)pair * kClassSlots;
    beg = cb[c];
    end = cb[c + 1];
    if (beg < end) {
      const uint32_t span = c == kWideClass ? 0u : (1u << c) - 1u;
      const uint64_t width = (uint64_t)(kmax - kmin) + 2ull * span;
      full = c == kWideClass || width >= 0xFFFFE000ull;
      if (!full) {
        const uint32_t lo = kmin - span, hi = kmax + span;
        const uint32_t cls = (uint32_t)c << kCentreBits;
        const uint32_t blo = cls | position_code(pd.arc, lo), bhi = cls | position_code(pd.arc, hi);
        // bhi + 1 > blo without a wrap; through the cut the two ranges may
        // meet in one code (and then take the whole class once)
        wrap = lo > hi;
        r = lower_bound_scalar(A.skey, beg, end, lane < kNumClasses ? blo : bhi + 1u);
      }
    }
  }
  // record positions fit 32 bits (the windows store them so)
  const uint32_t rb = (uint32_t)r, re = (uint32_t)__shfl((int)rb, c + kNumClasses);
  const uint32_t ub = (uint32_t)beg, ue = (uint32_t)end;
  uint32_t b0 = 0, l0 = 0, b1 = 0, l1 = 0;
  if (any && ub < ue) {
    b0 = full ? ub : rb;
    l0 = full || wrap ? ue - b0 : re - rb;
    b1 = ub;
    l1 = !full && wrap ? (re < rb ? re : rb) - ub : 0u;
  }
  const int src = lane >> 1;
  const uint32_t be = (uint32_t)__shfl((int)b0, src), bo = (uint32_t)__shfl((int)b1, src);
  const uint32_t le = (uint32_t)__shfl((int)l0, src), lo_ = (uint32_t)__shfl((int)l1, src);
  begin = (lane & 1) ? bo : be;
  return (lane & 1) ? lo_ : le;
}

// The row of query q: the image-2 indices of its hits in buf (the first
// kRowSortMax, in any order); returns their number.  The record ranges are
// found for all classes at once and scanned as one sequence.  What bounds it:
// the latency of a row's dependent loads.  (Class after class, each with two
// searches of its own: 22.4 us for the rows of 48 pairs of 500 to 10000
// keypoints whose windows are too long for the tile pass, 9.2 this way; 37 and
// 18.9 at 512 pairs.)
__device__ uint32_t stab_query(const StabArgs& A, const PairDev& pd, int pair, const QueryCtx& q,
                               int32_t* buf) {
  const int lane = lane_id();
  uint32_t begin = (uint32_t)pd.k_begin, len = lane == 0 ? (uint32_t)pd.n : 0u;
  if (!q.brute) len = class_ranges(A, pd, pair, q.key, q.key, true, begin);
  const uint32_t incl = wave_scan_u32(len);
  const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  const uint32_t off = begin - (incl - len);  // position of entry v: off + v
  uint32_t total = 0;
  for (uint32_t base = 0; base < all; base += kWave) {
    const uint32_t v = base + (uint32_t)lane;
    int s = 0;  // the slot that holds entry v: slots before it end at or below v
    #pragma unroll
    for (int step = 32; step > 0; step >>= 1) {
      const uint32_t e = (uint32_t)__shfl((int)incl, s + step - 1);
      if (e <= v) s += step;
    }
    const uint32_t pos = (uint32_t)__shfl((int)off, s) + v;
    bool hit = false;
    int32_t j = 0;
    if (v < all) {
      j = A.rj[pos];
      const float2 xy = A.rxy[pos];
      hit = (q.brute || key_distance(q.key, A.rC[pos]) <= A.rH[pos]) &&
            within_tolerance(q.a, q.b, q.c, xy.x, xy.y, A.reps[pos]);
    }
    const uint64_t m = ballot(hit);
    const uint32_t slot = total + lanes_below(m);
    if (hit && slot < (uint32_t)kRowSortMax) buf[slot] = j;
    total += (uint32_t)__popcll(m);
  }
  return total;
}

// Writes query i's CSR row in ascending j (rows of any length).
__device__ void fill_row(const StabArgs& A, int64_t i, int32_t* buf) {
  const int lane = lane_id();
  const int pair = find_pair(A.qstart, A.num_pairs, i);
  const PairDev& pd = A.pairs[pair];
  const uint32_t flag = A.qflag[i];
  const int64_t o0 = A.row_offsets[i];
  const int64_t len = A.row_offsets[i + 1] - o0;
  if (len == 0 || flag == kQueryEmpty) return;
  QueryCtx q;
  epipolar_line(pd.F, A.kp1[2 * i], A.kp1[2 * i + 1], q.a, q.b, q.c);
  q.key = A.qkey[i];
  q.brute = flag == kQueryBrute;

  if (len > kRowSortMax) {
    // long row: rebuild it in ascending j directly from the definition
    const int64_t kb = pd.k_begin;
    uint32_t total = 0;
    constexpr int kU = 4;  // blocks of 64 j whose gathers are in flight together
    for (int64_t j0 = 0; j0 < pd.n; j0 += kU * kWave) {
      uint32_t pos[kU];
      #pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t j = j0 + u * kWave + lane;
        pos[u] = j < pd.n ? A.rinv[kb + j] : 0u;
      }
      float2 xy[kU];
      float ee[kU];
      #pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t j = j0 + u * kWave + lane;
        xy[u] = j < pd.n ? A.rxy[pos[u]] : make_float2(0.0f, 0.0f);
        ee[u] = j < pd.n ? A.reps[pos[u]] : 0.0f;
      }
      #pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int64_t j = j0 + u * kWave + lane;
        const bool hit = j < pd.n && within_tolerance(q.a, q.b, q.c, xy[u].x, xy[u].y, ee[u]);
        const uint64_t m = ballot(hit);
        const int64_t dst = o0 + total + lanes_below(m);
        if (hit && dst < A.capacity) A.cols[dst] = (int32_t)j;
        total += (uint32_t)__popcll(m);
      }
    }
    return;
  }

  const uint32_t total = stab_query(A, pd, pair, q, buf);
  wave_sync_lds();
  const int n = (int)(total < (uint32_t)len ? total : (uint32_t)len);
  if (n <= kWave) {
    const int32_t v = wave_sort64(lane < n ? buf[lane] : INT32_MAX);
    if (lane < n && o0 + lane < A.capacity) A.cols[o0 + lane] = v;
  } else {
    int p2 = 128;
    while (p2 < n) p2 <<= 1;
    for (int t = n + lane; t < p2; t += kWave) buf[t] = INT32_MAX;
    wave_sync_lds();
    wave_sort_lds(buf, p2);
    for (int t = lane; t < n; t += kWave)
      if (o0 + t < A.capacity) A.cols[o0 + t] = buf[t];
  }
  wave_sync_lds();
}

// The fused pass's record of a query: its row length and its match (as
// write_match_to would store it), or kMatchDeferred for a match that a later
// pass writes.
__device__ __forceinline__ uint4 query_record(uint32_t count, float ratio, const Top2& t,
                                              bool matched) {
  int32_t idx = t.bj == INT32_MAX ? -1 : t.bj;
  if (idx >= 0 && ratio > 0.0f && !(t.bd < ratio * ratio * t.sd)) idx = -1;
  if (!matched) idx = kMatchDeferred;
  return make_uint4(count, (uint32_t)idx, __float_as_uint(t.bd), __float_as_uint(t.sd));
}

// ------------------------------------------------------------- tiled pass
constexpr int kQPerWave = kTileQ / kWaves;
static_assert(kQPerWave == 16, "the pair test packs four records of 16 queries per wavefront");
static_assert(kTileQ == 64, "pair indexing uses a 6-bit query field");

// Queries per tile of the pairs with many records per query: a workgroup per
// pair, which looks at kSplitSamples places and takes as many queries as the
// cheapest of 64, 32, 16 and 8 for the windows that they would have there.  With
// w records that the middle of 64 queries can meet and v more between the
// first and the last, T of them have about w + v T / 64 records in their
// window; a tile's time is taken as that and kTileCost, times the tiles that run
// one after another, and kLongCost times that for rows that a fused pass leaves
// because of the window's length.  (Rows of more than kStage candidates go to
// the wide-row pass, whose time is the windows' too: there small tiles only
// multiply it.)
// What bounds it: a binary search per place and the atomic of a pair's base,
// 10 us for a pair, 14 for 512.  What it gives, counted / matched in BF16
// in one call: 48 pairs of 1000 queries and 40000 records take 198 / 455 us at
// 22 candidates per query and 518 / 929 at 1083 with 64 queries in all tiles,
// 236 / 375 and 1106 / 2021 with tile_queries' numbers, 213 / 379 and 509 / 882
// with this; one pair of 2000 and 100000 at 21: 188 / 174, 76 / 124, 87 / 127;
// 512 uneven pairs in BF16: 3327 us, 2960, 2990 (with kLongWindow 600: 3262;
// with kTileCost 64: 3014).
constexpr int kSplitSamples = 8;
constexpr int kSplitThreads = 2 * kWave * kSplitSamples;  // two wavefronts per place
constexpr float kTileCost = 256.0f, kLongCost = 4.0f, kLongWindow = 900.0f;
__global__ __launch_bounds__(kSplitThreads) void k_tile_split(StabArgs A, float fill) {
  __shared__ float s_cost[kSplitSamples][4], s_one[kSplitSamples];
  __shared__ uint32_t s_base;
  const int lane = lane_id(), place = wave_id() >> 1, pair = (int)blockIdx.x;
  const bool middle = (wave_id() & 1) != 0;  // this wavefront searches for the middle query
  const PairDev& pd = A.pairs[pair];
  const int least = tile_queries(pd.m, pd.n);
  if (least == kTileQ || pd.m == 0) return;  // uniform
  // 64 queries around the middle of the place's part of the pair
  const int64_t mid = pd.m * (2 * place + 1) / (2 * kSplitSamples);
  const int64_t from = mid < kTileQ / 2 ? 0 : mid - kTileQ / 2;
  const int64_t first = pd.m < kTileQ ? 0 : from + kTileQ <= pd.m ? from : pd.m - kTileQ;
  const int64_t at = first + lane;
  const uint32_t qi = at < pd.m ? A.qperm[pd.q_begin + at] : 0u;
  const bool normal = at < pd.m && A.qflag[qi] == kQueryNormal;
  const uint32_t key = normal ? A.qkey[qi] : 0u;
  const uint32_t kmin = wave_min_u32(normal ? key : 0xFFFFFFFFu);
  const uint32_t kmax = wave_max_u32(key);
  const uint64_t have = ballot(normal);
  const uint32_t kmid = (uint32_t)__builtin_amdgcn_readlane(
      (int)key, have != 0ull ? nth_bit(have, (uint32_t)__popcll(have) / 2u) : 0);
  uint32_t begin;
  const float found = (float)wave_sum_u32(class_ranges(
      A, pd, pair, middle ? kmid : kmin, middle ? kmid : kmax, have != 0ull, begin));
  if (middle && lane == 0) s_one[place] = found;
  __syncthreads();
  const float one = s_one[place], between = fmaxf(found - one, 0.0f);
  const bool kept_rows = A.qrec != nullptr && one <= 2.0f * kStage;  // rows that a fused pass keeps
  if (!middle && lane < 4) {
    const float part = 1.0f / (float)(1 << lane);  // of kTileQ queries
    const float window = one + between * part;
    float cost = fmaxf(1.0f, fill / part) * (window + kTileCost);
    if (kept_rows && window > kLongWindow) cost *= kLongCost;
    s_cost[place][lane] = cost;
  }
  __syncthreads();
  int best = kTileQ;
  float best_cost = __builtin_inff();
  for (int k = 0; k < 4 && kTileQ >> k >= least; ++k) {
    float cost = 0.0f;
    #pragma unroll
    for (int w = 0; w < kSplitSamples; ++w) cost += s_cost[w][k];
    if (cost < best_cost) {
      best_cost = cost;
      best = kTileQ >> k;
    }
  }
  // the pair's tiles, behind those of the pairs that were faster
  const int64_t tiles = (pd.m + best - 1) / best;
  if (threadIdx.x == 0) s_base = atomicAdd(A.split_tiles, (uint32_t)tiles);
  __syncthreads();
  StabTile* to = A.tiles + A.even_tiles + s_base;
  for (int64_t t = threadIdx.x; t < tiles; t += kSplitThreads) {
    StabTile T;
    T.begin = pd.q_begin + t * best;
    T.count = (int32_t)(pd.m - t * best < best ? pd.m - t * best : best);
    T.pair = pair;
    to[t] = T;
  }
}

// Window pass: for tile t, the record ranges of every width class whose
// centres lie within [min key - 2^c + 1, max key + 2^c - 1] of the tile's
// queries (class_ranges), one wavefront per tile, so every tile's searches are
// in flight at once.
constexpr int kWindowTiles = 4;  // tiles (one wavefront each) per workgroup
constexpr int kWindowThreads = kWave * kWindowTiles;
constexpr int kWindowQ = kTileQ * kWindowTiles;
static_assert(kWindowQ == kWindowThreads, "a thread per query slot");

// A large group of the query sort in the order of its keys, by every workgroup
// that holds a part of it for itself: the group's keys are counted in
// kRefineBins bins over their span, and the queries of the bins that this
// workgroup's places fall into are collected and ranked.  A bin of more than
// kRefineBin queries (nearly equal keys) leaves the group as the sort wrote it,
// in all of its workgroups.  What bounds it: three walks over the group by a
// workgroup, a few loads per thread for groups of a thousand.  (Without it
// 60000 queries and 240000 records in 8 of the 2048 groups took 1665 us to
// count, 167 with it.)
constexpr int kRefineBins = 1024, kRefineBin = 384;
constexpr int kRefineMax = kWindowQ + 2 * kRefineBin;
struct Refine {
  uint64_t v[kRefineMax];  // key and place in the group, by bin
  uint32_t start[kRefineBins + 1], cursor[kRefineBins];
  uint32_t wsum[kWindowTiles], wmax[kWindowTiles], lo, hi, base, end;
};

// Group: places [gs, ge) of the segment that starts at query seg; the workgroup
// holds places [pa, pb) of it in its tiles w0 to w1 - 1 (place, count: of its
// tiles).  Called by the whole workgroup.
__device__ void refine_group(const StabArgs& A, int64_t seg, uint32_t gs, uint32_t ge, uint32_t pa,
                             uint32_t pb, int w0, int w1, const uint32_t* place,
                             const int32_t* count, uint32_t* s_i, uint32_t* s_k, Refine& S) {
  static_assert(kRefineBins == 4 * kWindowThreads, "four bins per thread");
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const uint32_t n = ge - gs;  // at most 2^17 (one-pass segments)
  const uint32_t* perm = A.qperm + seg + gs;
  #pragma unroll
  for (int u = 0; u < 4; ++u) S.start[4 * tid + u] = S.cursor[4 * tid + u] = 0u;
  if (tid == 0) {
    S.lo = 0xFFFFFFFFu;
    S.hi = 0u;
  }
  __syncthreads();
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  #pragma unroll 4
  for (uint32_t e = tid; e < n; e += kWindowThreads) {
    const uint32_t k = A.qkey[perm[e]];
    lo = min(lo, k);
    hi = max(hi, k);
  }
  lo = wave_min_u32(lo);
  hi = wave_max_u32(hi);
  if (lane == 0) {
    atomicMin(&S.lo, lo);
    atomicMax(&S.hi, hi);
  }
  __syncthreads();
  lo = S.lo;
  const uint32_t span = S.hi - lo;
  const int shift = span < (uint32_t)kRefineBins ? 0 : 22 - (int)__builtin_clz(span);
  static_assert(kRefineBins == 1 << 10, "span >> shift has ten bits");
  #pragma unroll 4
  for (uint32_t e = tid; e < n; e += kWindowThreads)
    atomicAdd(&S.start[(A.qkey[perm[e]] - lo) >> shift], 1u);
  __syncthreads();
  uint32_t c[4];
  #pragma unroll
  for (int u = 0; u < 4; ++u) c[u] = S.start[4 * tid + u];
  const uint32_t own = c[0] + c[1] + c[2] + c[3];
  const uint32_t most = wave_max_u32(max(max(c[0], c[1]), max(c[2], c[3])));
  const uint32_t incl = wave_scan_u32(own);
  if (lane == kWave - 1) S.wsum[wave] = incl;
  if (lane == 0) S.wmax[wave] = most;
  __syncthreads();
  uint32_t at = incl - own, biggest = 0u;
  #pragma unroll
  for (int w = 0; w < kWindowTiles; ++w) {
    at += w < wave ? S.wsum[w] : 0u;
    biggest = max(biggest, S.wmax[w]);
  }
  if (biggest > (uint32_t)kRefineBin) {  // uniform
    __syncthreads();
    return;
  }
  // this workgroup's ranks in the group, and the bins that hold them
  const uint32_t r0 = max(pa, gs) - gs, r1 = min(pb, ge) - gs;
  #pragma unroll
  for (int u = 0; u < 4; ++u) {
    S.start[4 * tid + u] = at;
    if (at <= r0 && r0 < at + c[u]) S.base = at;
    if (at < r1 && r1 <= at + c[u]) S.end = at + c[u];
    at += c[u];
  }
  if (tid == kWindowThreads - 1) S.start[kRefineBins] = at;
  __syncthreads();
  const uint32_t base = S.base, end = S.end;
  #pragma unroll 4
  for (uint32_t e = tid; e < n; e += kWindowThreads) {
    const uint32_t k = A.qkey[perm[e]], bin = (k - lo) >> shift, b = S.start[bin];
    if (b >= base && b < end) S.v[b - base + atomicAdd(&S.cursor[bin], 1u)] = ((uint64_t)k << 17) | e;
  }
  __syncthreads();
  for (uint32_t p = tid; p < end - base; p += kWindowThreads) {
    const uint64_t v = S.v[p];
    const uint32_t k = (uint32_t)(v >> 17), bin = (k - lo) >> shift;
    const uint32_t b = S.start[bin] - base, e = S.start[bin + 1] - base;
    uint32_t r = base + b;
    for (uint32_t u = b; u < e; ++u) r += S.v[u] < v ? 1u : 0u;
    if (r >= r0 && r < r1) {
      const uint32_t x = gs + r;
      for (int w = w0; w < w1; ++w) {
        if (x - place[w] < (uint32_t)count[w]) {
          s_i[w * kTileQ + (int)(x - place[w])] = perm[v & 0x1FFFFull];
          s_k[w * kTileQ + (int)(x - place[w])] = k;
        }
      }
    }
  }
  __syncthreads();
}

// Bitonic sort of a value per thread of the workgroup, ascending (a
// wavefront's in registers, others' through buf, in turn in its two halves).
__device__ __forceinline__ uint64_t window_sort(uint64_t v, uint64_t* buf) {
  const int tid = threadIdx.x;
  // blocks of k are brought into ascending and descending order in turn
  bool down = (tid & kWave) != 0;
  v = wave_sort64(down ? ~v : v);
  v = down ? ~v : v;
  uint64_t* at = buf;
  #pragma unroll 1
  for (int k = 2 * kWave; k <= kWindowThreads; k *= 2) {
    down = (tid & k) != 0;
    v = down ? ~v : v;
    #pragma unroll 1
    for (int j = k / 2; j >= kWave; j /= 2) {
      at[tid] = v;
      __syncthreads();
      const uint64_t o = at[tid ^ j];
      v = (o < v) == ((tid & j) == 0) ? o : v;
      at = at == buf ? buf + kWindowThreads : buf;
    }
    sort_step<kWave, kWave / 2>(v, lane_id());
    v = down ? ~v : v;
  }
  return v;
}

// Eight wavefronts per SIMD: the pass waits for dependent loads.  (512 uneven
// pairs, whole call: 2984 us with the 66 VGPRs of its own choice, seven
// wavefronts, 2976 this way.)
__global__ __launch_bounds__(kWindowThreads, 8) void k_tile_windows(StabArgs A) {
  const int lane = lane_id(), wave = wave_id();
  // each XCD takes one run of consecutive tiles: the queries of a pair are
  // gathered in their sorted order, and a line of them holds several tiles'
  // (12.5 us with the workgroups dealt in turn, 10.8 so, at 1878 tiles)
  const int run = (int)gridDim.x / kNumXcd;
  const int t =
      (((int)blockIdx.x % kNumXcd) * run + (int)blockIdx.x / kNumXcd) * kWindowTiles + wave;
  // the look-back words of the pass over the rows (one per 256 queries, a
  // tile holds at most 64) start from zero
  for (int64_t k = (int64_t)blockIdx.x * kWindowThreads + threadIdx.x;
       k < (A.n1 + kFinishRows - 1) / kFinishRows; k += (int64_t)gridDim.x * kWindowThreads)
    A.row_sums[k] = 0ull;
  // The sort grouped the queries by the upper bits of their codes.  Sorting
  // the 64 queries around each boundary between two of the workgroup's tiles
  // by their whole keys gives the tiles the queries that a full sort would,
  // as long as a group holds no more than half a tile.  (Without it the
  // windows are longer: the tile pass 90.6 instead of 86.1 us at six pairs of
  // 20000 keypoints, 149 instead of 139 at one of 60000; this costs 2.)
  // Where queries crowd into groups of more than two tiles, those that leave
  // the workgroup are put in order across their workgroups, and the
  // workgroup's queries are sorted by their whole keys; the latter also where
  // a group exceeds a tile, or the tiles hold few of them.  (Groups of one to
  // two tiles, 60000 queries with 60 candidates: match and count 189 us without,
  // 187 with it.)
  __shared__ uint32_t s_i[kWindowQ], s_k[kWindowQ];
  __shared__ int32_t s_pair[kWindowTiles], s_count[kWindowTiles];
  __shared__ uint32_t s_place[kWindowTiles];  // the tile's first place in its segment
  __shared__ Refine refine;
  const bool live = t < A.num_tiles;
  const bool used = live && (t < A.even_tiles || t < A.even_tiles + (int)*A.split_tiles);
  StabTile T;
  T.begin = 0;
  T.count = 0;
  T.pair = -1;
  if (used) T = A.tiles[t];
  const int slot = (int)threadIdx.x;
  uint32_t qi = 0u, key = 0xFFFFFFFFu;  // behind every query, by its place
  if (lane < T.count) {
    qi = A.qperm[T.begin + lane];
    key = A.qkey[qi];
  }
  const bool sorts = used && A.groups && A.groups[T.pair] != kGroupsSmall;
  s_i[slot] = qi;
  s_k[slot] = key;
  if (lane == 0) s_pair[wave] = T.pair;
  if (!__syncthreads_or(sorts)) {
    const bool joined = wave + 1 < kWindowTiles && t + 1 < A.num_tiles && T.count == kTileQ &&
                        s_pair[wave + 1] == T.pair;
    uint32_t moved_i = 0u, moved_k = 0u;
    if (joined) {
      const uint64_t v =
          wave_sort64(((uint64_t)s_k[slot + kTileQ / 2] << 6) | (uint64_t)lane);
      moved_i = s_i[slot - lane + kTileQ / 2 + (int)(v & 63ull)];
      moved_k = (uint32_t)(v >> 6);
    }
    __syncthreads();
    if (joined) {
      s_i[slot + kTileQ / 2] = moved_i;
      s_k[slot + kTileQ / 2] = moved_k;
    }
    __syncthreads();
    qi = s_i[slot];
    key = s_k[slot];
  } else {
    if (lane == 0) {
      s_count[wave] = T.count;
      s_place[wave] = used ? (uint32_t)(T.begin - A.qstart[T.pair]) : 0u;
    }
    __syncthreads();
    int first = 0;             // of this wavefront's run of tiles of one pair
    uint32_t first_place = 0;  // the run's first place in the segment
    for (int w0 = 0; w0 < kWindowTiles;) {  // uniform
      const int p = s_pair[w0];
      int w1 = w0, from = w0, last = w0;  // the first and the last tile that holds queries
      for (; w1 < kWindowTiles && s_pair[w1] == p; ++w1) {
        if (s_count[from] == 0) from = w1;
        if (s_count[w1] > 0) last = w1;
      }
      if (w0 <= wave) {
        first = w0;
        first_place = s_place[from];
      }
      if (p >= 0 && s_count[from] > 0 && A.groups[p] == kGroupsLarge) {
        const SortSeg sg = A.qsegs[p];
        const uint32_t pa = s_place[from], pb = s_place[last] + (uint32_t)s_count[last];
        const auto put = [&](uint32_t gs, uint32_t ge) {
          refine_group(A, sg.begin, gs, ge, pa, pb, w0, w1, s_place, s_count, s_i, s_k, refine);
        };
        if (sg.tile_count < 2) {  // a segment of one sort tile: all of it as one group
          put(0u, (uint32_t)sg.count);
        } else {
          const uint32_t* starts = A.group_starts + (int64_t)sg.hist_begin * kHistWords;
          constexpr int kLow = kCentreBits - kRadixBits;
          const KeyArc arc = A.pairs[p].arc;
          const uint32_t d0 = position_code(arc, s_k[from * kTileQ]) >> kLow;
          const uint32_t d1 = position_code(arc, s_k[last * kTileQ + s_count[last] - 1]) >> kLow;
          for (uint32_t d = d0;; d = d1) {
            const uint32_t gs = starts[d] - (uint32_t)sg.begin;
            const uint32_t ge = d + 1 < (uint32_t)kRadix ? starts[d + 1] - (uint32_t)sg.begin
                                                         : (uint32_t)sg.count;
            if (ge - gs > 2u * (uint32_t)sg.tile) put(gs, ge);
            if (d == d1) break;
          }
        }
      }
      w0 = w1;
    }
    // all queries of every run by (key, slot); empty slots follow them
    const bool full = lane < T.count;
    const uint64_t v = window_sort(((uint64_t)first << 41) | ((uint64_t)(full ? 0 : 1) << 40) |
                                       ((uint64_t)s_k[slot] << 8) | (uint64_t)slot,
                                   refine.v);
    __syncthreads();
    refine.v[slot] = v;
    __syncthreads();
    if (full) {  // the run's k-th query goes to its k-th filled slot
      const uint64_t mine = refine.v[first * kTileQ + (int)(s_place[wave] - first_place) + lane];
      qi = s_i[(int)(mine & 255ull)];
      key = (uint32_t)(mine >> 8);
    }
  }
  if (!live) return;  // whole wavefronts
  if (!used) {  // no kernel looks further
    T.pair = 0;
    if (lane == 0) A.tiles[t] = T;
    if (lane == 0) A.tile_wide[t] = 0u;
    if (lane == 0 && A.tile_cost) A.tile_cost[t] = 0u;
    if (lane < kTileCounts && A.tile_counts)
      A.tile_counts[(int64_t)t * kTileCounts + lane] = 0ull;
    return;
  }
  bool normal = false, brute = false;
  TileQuery tq;
  tq.a = tq.b = tq.c = 0.0;
  tq.i = 0;
  tq.flag = kQueryEmpty;
  tq.key = tq.pad = 0;
  if (lane < T.count) {
    const int64_t i = qi;
    A.qperm_out[T.begin + lane] = qi;
    const uint32_t flag = A.qflag[i];
    normal = flag == kQueryNormal;
    brute = flag == kQueryBrute;
    tq.i = (uint32_t)i;
    tq.flag = flag;
    tq.key = key;
    const double4 L = A.qline[i];  // the line of Eq. 2, from the key pass
    tq.a = L.x;
    tq.b = L.y;
    tq.c = L.z;
  }
  A.tile_q[(int64_t)t * kTileQ + lane] = tq;
  if (lane == 0) {
    A.tile_wide[t] = 0u;  // set by the tile pass when a row is wide
    // the pair's flag likewise, cleared by the pair's first tile
    if (A.pair_wide && T.begin == A.qstart[T.pair]) A.pair_wide[T.pair] = 0u;
  }
  const uint32_t kmin = wave_min_u32(normal ? key : 0xFFFFFFFFu);
  const uint32_t kmax = wave_max_u32(normal ? key : 0u);
  const bool any = ballot(normal) != 0;
  uint32_t begin = 0;
  const uint32_t len = class_ranges(A, A.pairs[T.pair], T.pair, kmin, kmax, any, begin);
  const uint32_t incl = wave_scan_u32(len);
  TileWindow* w = A.windows + t;
  w->slot_b[lane] = begin;
  w->slot_pref[lane + 1] = incl;
  if (lane == 0) w->slot_pref[0] = 0u;
  if (A.tile_cost) {
    // work estimate: (query, record) pairs of the window scan, brute-force
    // scans, and one unit per query
    const uint64_t wlen = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    const uint64_t nn = (uint64_t)__popcll(ballot(normal));
    const uint64_t nb = (uint64_t)__popcll(ballot(brute));
    if (lane == 0) {
      const uint64_t c = nn * wlen + nb * (uint64_t)A.pairs[T.pair].n + (uint64_t)T.count;
      const uint32_t c32 = c > 0xFFFFFFFFull ? 0xFFFFFFFFu : (uint32_t)c;
      A.tile_cost[t] = c32;
    }
  }
}

// Counts every row of a tile of kTileQ angle-sorted queries and parks rows of
// up to kStage candidates in ascending j in the staging buffer.  The window
// records of the tile are staged in LDS; wavefront w owns queries 16w..16w+15
// (lane & 15), whose lines stay in registers, and tests them against four
// records per step (lane >> 4, LDS broadcasts): angle test and FP64 test.  A
// hit sets a bit of its query's bitmap by window position; in kStabF32 it goes
// to the query's list, in ascending window position, its slot from a ballot
// over the query's four lanes.  Windows longer than kKeepJ have no bitmaps
// (kStabCount lists the hits' j for those).
//
// FUSE: the same pass also selects every query's match (Sec. 4.3) from its
// hits while they are still in LDS (window positions; their j from the
// window's j, kept in LDS for windows of up to kKeepJ records).  kStabF32: the
// window's descriptor rows are copied to LDS kFuseRows at a time (over the
// record chunk buffers and the window's order, dead by then), and four
// lanes per query evaluate canonical FP32 distances of that query's hits in
// the chunk, each lane resuming where the last chunk left it, and keep a
// top-2, merged across the four lanes at the end.  Rows longer than kStage are
// matched by the wide-row pass; the rows this pass does not keep (brute-force
// queries, windows longer than kKeepJ) are marked and their queries listed:
// k_finish_listed rebuilds the rows and matches them; empty rows get their
// (-1, inf, inf) here.  The LDS and
// register budget allows three workgroups per CU.  Outside the order of the
// window every wavefront works on its own 16 queries, so the tile needs only
// the barriers of the record and row chunks and of the order; its counters
// gather in LDS and go to global memory once per tile (per-wavefront global
// atomics on the same counters cost more than a barrier).
constexpr int kFuseRows = 48;
constexpr int kFuseStride = 132;  // floats per staged row: 16-byte reads of rows hit distinct banks
// LDS bytes of a round of CH window records (C, H, x y, eps, j).
constexpr int rec_bytes(int CH) { return CH * (4 + 4 + 8 + 4 + 4); }
// The staged rows are copied straight from global memory to LDS (lane l of a
// wavefront copy writes 16-byte chunk l of it): kFuseCopies wavefront copies
// cover the rows with their padding, and the tail of the last one is slack.
constexpr int kFuseChunks = kFuseRows * (kFuseStride / 4);
constexpr int kFuseCopies = (kFuseChunks + kWave - 1) / kWave;
constexpr int kFuseBytes = kFuseCopies * kWave * 16;
// First entry of a parked row that was not parked: k_finish_listed rebuilds it.
constexpr int32_t kRowNotParked = -1;
// Flag of a listed query (a.rest) whose row has to be rebuilt first; there are
// fewer than 2^31 queries (their parked rows alone would fill 1 TB).
constexpr uint32_t kRestRebuild = 0x80000000u;

// FUSE: the j of the first kKeepJ window positions stay in LDS; the hits
// are kept as 16-bit window positions, and tiles with longer windows are not
// fused (their rows are rebuilt and matched from the list)
constexpr int kKeepJ = 1024;
constexpr int64_t kFuseMaxWindow = kKeepJ;

// Starts the copy of rows [c0, c0 + nr) of the window (0 < nr <= kFuseRows)
// to LDS at a stride of kFuseStride floats.  Chunk p of the image is column
// p % 33 of row p / 33; the padding column and the rows past nr repeat real
// data.  The copies complete asynchronously: wait for them (vmcnt) before the
// barrier that publishes the rows.
__device__ __forceinline__ void fuse_stage(const StabArgs& A, int c0, int nr, int64_t kb,
                                           const int32_t* sJ, float4* rows4, int wave, int lane) {
  constexpr int kRowChunks = kFuseStride / 4;
  for (int g = wave; g < kFuseCopies; g += kWaves) {
    const int p = g * kWave + lane;
    int r = p / kRowChunks;
    int c = p - r * kRowChunks;
    r = r < nr ? r : nr - 1;
    c = c < 32 ? c : 31;
    const float4* src = reinterpret_cast<const float4*>(A.desc2) + (kb + sJ[c0 + r]) * 32 + c;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(rows4 + g * kWave),
                                     16, 0, 0);
  }
}

// s_waitcnt vmcnt(0): this wavefront's copies to LDS have landed.
__device__ __forceinline__ void wait_lds_copies() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// ------------------------------------------------ BF16 fused selection
// MODE kStabBF16: the caller's descriptors are BF16 codes with FP32 masters,
// and the final matches must be the canonical FP32 selection on the masters.
// The window's BF16 rows are staged kBfRows at a time; wavefront w scores its
// 16 queries against them on MFMA (A = the window rows, B = the queries, so
// lane l holds query l & 15 against rows 16 cb + 4 i + (l >> 4)).  Every hit
// gets certified bounds D_lo <= D <= D_hi on its exact canonical distance D:
//   |q^ - w^|^2 is within em = 3e-5 (|q^| + |w^|)^2 of |q^|^2 + |w^|^2 - 2 q^.w^
//   (FP32 accumulation), |q - w| is within eps_q + eps_w of |q^ - w^| (eps_q
//   the measured norm of the query's rounding error, exact in FP32 from its
//   master; eps_w the BF16 bound u |w^| / (1 - u), u = 2^-8, of a row rounded
//   to nearest even), and D is within 2e-5 (relative) of |q - w|^2 (130
//   roundings of 2^-24).
// Let U2 be the second smallest D_hi over any set of the row's candidates.
// Two candidates have D <= U2, so a candidate with D_lo > U2 is strictly
// worse than both and is neither best nor second: the candidates with
// D_lo <= U2 are evaluated exactly (canonical chains on the masters) and
// their top-2 is the row's.  Each lane keeps only the kBfKeep smallest
// approximate distances A of its hits, with their rows' bound norms; after
// the last chunk it works out D_lo and D_hi of those (U2 is taken over the
// row's kept candidates) and, since D_lo grows with A and shrinks with the
// row norm, a lower bound on D_lo of every pushed-out hit from the smallest
// pushed-out A and the largest row norm.  A row whose pushed-out bound is not
// above U2 is left to the listed-query match, exact either way.
constexpr int kBfRows = 32;  // window rows per chunk: with 256-record rounds, four workgroups per CU
constexpr int kBfBlocks = kBfRows / 16;     // 16-row MFMA blocks per chunk
constexpr int kBfStride = 256 + 16;         // LDS bytes per row: 16 rows' reads hit distinct banks
constexpr int kBfPieces = kBfStride / 16;   // 16-byte pieces per row (the last repeats one)
constexpr int kBfCopies = (kBfRows * kBfPieces + kWave - 1) / kWave;
constexpr int kBfRowBytes = kBfCopies * kWave * 16;
constexpr int kBfKeep = 3;
// MODE kStabFP8: the image-2 rows are 128 one-byte E4M3 codes c with a scale
// s per row (w^ = s c), staged at a stride of 144 bytes (the padding
// staggers the rows over the LDS banks) and decoded to BF16 for the MFMA,
// exactly; the queries are rounded to BF16 on chip from their masters (eps_q
// measured as above).  The score of the codes times s is q^.w^ within the
// same accumulation bound, |w^|^2 = s^2 |c|^2, and eps_w is the caller's
// bound on |w - w^| for the row, carried per kept candidate rounded up to
// FP16 (the accumulation term takes the lane's largest row norm).  These
// errors are an order of magnitude above BF16's, so more candidates per row
// fall within the row's second upper bound: each lane keeps six.
constexpr int kF8Stride = 128 + 16;
constexpr int kF8Pieces = kF8Stride / 16;
constexpr int kF8Copies = (kBfRows * kF8Pieces + kWave - 1) / kWave;
constexpr int kF8RowBytes = kF8Copies * kWave * 16;
constexpr int kF8Keep = 6;
// After the pair test the record chunk holds the chunk's row terms (a float4
// per row) and the per-query task lists (four lanes of `keep` entries).
constexpr int red_scratch(int keep) { return kBfRows * 16 + kTileQ * 4 * keep * 2; }

// Starts the copy of BF16 rows [c0, c0 + nr) of the window to LDS (stride
// kBfStride, 0 < nr <= kBfRows); rows past nr and the padding piece repeat
// real data.  The copies complete asynchronously (wait_lds_copies).
__device__ __forceinline__ void bf16_stage(const StabArgs& A, int c0, int nr, int64_t kb,
                                           const int32_t* sJ, uint8_t* rows, int wave, int lane) {
  for (int g = wave; g < kBfCopies; g += kWaves) {
    const int p = g * kWave + lane;
    int r = p / kBfPieces;
    int c = p - r * kBfPieces;
    r = r < nr ? r : nr - 1;
    c = c < 16 ? c : 15;
    const uint4* src = reinterpret_cast<const uint4*>(A.codes2) + (kb + sJ[c0 + r]) * 16 + c;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(rows + g * kWave * 16),
                                     16, 0, 0);
  }
}

// Starts the copy of FP8 rows [c0, c0 + nr) of the window to LDS (stride
// kF8Stride, 0 < nr <= kBfRows), as bf16_stage.
__device__ __forceinline__ void f8_stage(const StabArgs& A, int c0, int nr, int64_t kb,
                                         const int32_t* sJ, uint8_t* rows, int wave, int lane) {
  for (int g = wave; g < kF8Copies; g += kWaves) {
    const int p = g * kWave + lane;
    int r = p / kF8Pieces;
    int c = p - r * kF8Pieces;
    r = r < nr ? r : nr - 1;
    c = c < 8 ? c : 7;
    const uint4* src = reinterpret_cast<const uint4*>(A.f8codes2) + (kb + sJ[c0 + r]) * 8 + c;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(rows + g * kWave * 16),
                                     16, 0, 0);
  }
}

// Eight OCP E4M3FN codes (byte e is element e) as BF16 values.  Every E4M3
// value has at most four significant bits and an exponent inside BF16's
// range, so the upper half of the hardware's FP32 decode is the value itself.
__device__ __forceinline__ bf16x8 e4m3x8_bf16(uint2 v) {
  const uint32_t src[2] = {v.x, v.y};
  uint32_t w[4];
  #pragma unroll
  for (int h = 0; h < 2; ++h) {
    const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)src[h], false);  // bytes 0, 1
    const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)src[h], true);   // bytes 2, 3
    w[2 * h] = (__float_as_uint(lo[0]) >> 16) | (__float_as_uint(lo[1]) & 0xFFFF0000u);
    w[2 * h + 1] = (__float_as_uint(hi[0]) >> 16) | (__float_as_uint(hi[1]) & 0xFFFF0000u);
  }
  return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
}

// Sum of the squares of sixteen E4M3 codes (decoded exactly; each square is
// exact in FP32).
__device__ __forceinline__ float e4m3x16_sumsq(uint4 v, float acc) {
  const uint32_t src[4] = {v.x, v.y, v.z, v.w};
  #pragma unroll
  for (int h = 0; h < 4; ++h) {
    const auto lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)src[h], false);
    const auto hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)src[h], true);
    acc = __builtin_fmaf(lo[0], lo[0], acc);
    acc = __builtin_fmaf(lo[1], lo[1], acc);
    acc = __builtin_fmaf(hi[0], hi[0], acc);
    acc = __builtin_fmaf(hi[1], hi[1], acc);
  }
  return acc;
}

// Per-lane state of one query's selection with deferred bounds (lane group g
// of its four lanes): the K smallest approximate distances
// A = |q^|^2 + |w^|^2 - 2 q^.w^ seen (FP32, as the bounds take them), with
// their window positions and a row bound term rounded up to FP16 (BF16 rows:
// the bound norm |w^|; FP8 rows: the norm of the row's rounding error), the
// smallest A pushed out of that list, the largest row bound norm and (FP8)
// the largest rounding-error term seen.  The certified bounds D_lo <= D <=
// D_hi of the kept candidates, and a lower bound on D_lo of every pushed-out
// one (D_lo grows with A and shrinks with the row's norm and error), are
// worked out once after the last chunk.
constexpr uint32_t kNoPick = 0xFFFFFFFFu;
template <int K>
struct BfKeep {
  float a[K];      // ascending
  uint32_t pk[K];  // window position | FP16 row term << 16, kNoPick: empty
  float a_drop = __builtin_inff();
  float nb_max = 0.0f;
  uint32_t ew_max = 0u;  // FP16 bits: positive halves order as their bit patterns
  bool bad = false;

  __device__ __forceinline__ BfKeep() {
    #pragma unroll
    for (int t = 0; t < K; ++t) {
      a[t] = __builtin_inff();
      pk[t] = kNoPick;
    }
  }

  // sorted insertion: entry t moves down one place when A goes before entry
  // t - 1, takes A when A goes between them, and the last entry drops out
  __device__ __forceinline__ void add(float at, uint32_t p, float nb, uint32_t ew) {
    // an infinite A (norms whose squares overflow) may stand for any distance:
    // it is not kept below, and +inf would read as "nothing pushed out"
    bad |= !(fabsf(at) < __builtin_inff());
    nb_max = fmaxf(nb_max, nb);
    ew_max = ew_max > ew ? ew_max : ew;
    if constexpr (K == 3) {  // written out: the compiler keeps it free of branches
      const bool c0 = at < a[0], c1 = at < a[1], c2 = at < a[2];  // c0 => c1 => c2
      const float out = c2 ? a[2] : at;
      const bool out_real = c2 ? pk[2] != kNoPick : true;
      a[2] = c1 ? a[1] : (c2 ? at : a[2]);
      pk[2] = c1 ? pk[1] : (c2 ? p : pk[2]);
      a[1] = c0 ? a[0] : (c1 ? at : a[1]);
      pk[1] = c0 ? pk[0] : (c1 ? p : pk[1]);
      a[0] = c0 ? at : a[0];
      pk[0] = c0 ? p : pk[0];
      a_drop = out_real ? fminf(a_drop, out) : a_drop;
    } else {
      // new entry t: the old one, A, or the old entry t - 1, from the two
      // comparisons around it (selects only)
      float na[K];
      uint32_t np[K];
      bool prev = false;  // A goes before entry t - 1
      #pragma unroll
      for (int t = 0; t < K; ++t) {
        const bool ct = at < a[t];
        na[t] = prev ? a[t - (t > 0)] : (ct ? at : a[t]);
        np[t] = prev ? pk[t - (t > 0)] : (ct ? p : pk[t]);
        prev = ct;
      }
      const float out = prev ? a[K - 1] : at;
      const bool out_real = prev ? pk[K - 1] != kNoPick : true;
      a_drop = out_real ? fminf(a_drop, out) : a_drop;
      #pragma unroll
      for (int t = 0; t < K; ++t) {
        a[t] = na[t];
        pk[t] = np[t];
      }
    }
  }
};

// Certified bounds on the exact canonical distance of a candidate whose
// approximate distance is `at` and whose row bound norm is at most nb (query
// terms q_nb, q_db; see the comment above kBfRows).
// ew: a bound on |q - q^| + |w - w^|.
__device__ __forceinline__ void bounds_from(float at, float nb, float q_nb, float ew, float& dlo,
                                            float& dhi) {
  const float sum = q_nb + nb;
  const float em = 3e-5f * sum * sum;
  // sqrt(at +- em) from the hardware reciprocal square root (within a few
  // ulps): the 1e-6 factors cover it; arguments under 2^-100 take the
  // trivially valid bounds 0 and 2^-50
  // (a row term past FP16's range is +inf: the upper bound is +inf then, and
  // not the NaN that inf * rsqrt(inf) would make of it)
  const float th = fminf(fmaxf(at, 0.0f) + em, 0x1.fffffep127f);
  const float tl = at - em;
  const float r_hi = th > 0x1p-100f ? th * __builtin_amdgcn_rsqf(th) * (1.0f + 1e-6f) : 0x1p-50f;
  const float r_lo = tl > 0x1p-100f ? tl * __builtin_amdgcn_rsqf(tl) * (1.0f - 1e-6f) : 0.0f;
  // the 1e-6 r_lo term covers the rounding of the two subtractions
  const float e_lo = fmaxf(r_lo - ew - 1e-6f * r_lo, 0.0f);
  const float e_hi = r_hi + ew;
  dlo = e_lo * e_lo * (1.0f - 3e-5f);
  dhi = e_hi * e_hi * (1.0f + 3e-5f);
}

// BF16 rows: |w - w^| <= u |w^| / (1 - u) for a row rounded to nearest even.
__device__ __forceinline__ void bf_bounds(float at, float nb, float q_nb, float q_db, float& dlo,
                                          float& dhi) {
  bounds_from(at, nb, q_nb,
              q_db + nb * (float)(Fmt<0>::kUnit / (1.0 - Fmt<0>::kUnit) * (1.0 + 1e-6)) + 1e-30f,
              dlo, dhi);
}

// f(value of lane S of each row of 16 lanes) for S = 0 .. n - 1 (n <= 16).
template <int S, class F>
__device__ __forceinline__ void for_steps(int v, int n, const F& f) {
  if constexpr (S < 16) {
    if (S >= n) return;
    f(__builtin_amdgcn_update_dpp(0, v, 0x150 + S, 0xF, 0xF, false));  // row_newbcast:S
    for_steps<S + 1>(v, n, f);
  }
}

// The order by j of a tile's window of W <= kKeepJ records with distinct j:
// rank[v] for every window position and the j in ascending order.  The window's
// j are dealt to kOrderBuckets buckets over their span (the map is monotone),
// the buckets are laid out one after the other, and a record's rank is its
// bucket's start plus the smaller j in the bucket: about one compare each for
// scattered j, and never more than the window.  scratch: the j by bucket
// [kKeepJ], then counts, cursors and starts of the buckets; counts and cursors
// are zero at the start.  A barrier goes between two of the three passes.
constexpr int kOrderBuckets = 256;
constexpr int kOrderBytes = kKeepJ * 6;      // rank and sorted j
constexpr int kBruteBytes = kWaves * kStage * 4;  // kStabCount: a row per wavefront
constexpr int kRankWords = kKeepJ / 32 + 1;  // bitmap row: + 1 puts rows in different banks
constexpr int kRankBytes = kTileQ * kRankWords * 4;
constexpr int kWordsPer = kKeepJ / 32 / 4;   // bitmap words of each of a row's four threads
static_assert((kKeepJ + 3 * kOrderBuckets + 1) * 4 <= kRankBytes, "scratch of the order");
static_assert(kOrderBuckets == 4 * kWave, "four buckets per lane");

struct BucketMap {
  int32_t lo;
  float scale;
  __device__ __forceinline__ explicit BucketMap(const uint32_t* span) {
    lo = (int32_t)~span[0];
    scale = (float)kOrderBuckets / ((float)((int32_t)span[1] - lo) + 1.0f);
  }
  __device__ __forceinline__ int operator()(int32_t j) const {
    const int b = (int)((float)(j - lo) * scale);
    return b < kOrderBuckets ? b : kOrderBuckets - 1;
  }
};

__device__ __forceinline__ void order_count(const int32_t* sJ, int W, const uint32_t* span,
                                            uint32_t* scratch, int tid) {
  const BucketMap bucket(span);
  for (int v = tid; v < W; v += kThreads) atomicAdd(&scratch[kKeepJ + bucket(sJ[v])], 1u);
}

__device__ __forceinline__ void order_place(const int32_t* sJ, int W, const uint32_t* span,
                                            uint32_t* scratch, int tid) {
  const BucketMap bucket(span);
  const int lane = lane_id();
  uint32_t* cursor = scratch + kKeepJ + kOrderBuckets;
  uint32_t* start = cursor + kOrderBuckets;
  // every wavefront scans the counts and writes the same starts, so that it
  // can go on without a barrier
  uint32_t c[4];
  #pragma unroll
  for (int u = 0; u < 4; ++u) c[u] = scratch[kKeepJ + 4 * lane + u];
  const uint32_t own = c[0] + c[1] + c[2] + c[3];
  uint32_t b = wave_scan_u32(own) - own;
  #pragma unroll
  for (int u = 0; u < 4; ++u) {
    start[4 * lane + u] = b;
    b += c[u];
  }
  if (lane == kWave - 1) start[kOrderBuckets] = b;
  wave_sync_lds();
  for (int v = tid; v < W; v += kThreads) {
    const int32_t j = sJ[v];
    const int k = bucket(j);
    scratch[start[k] + atomicAdd(&cursor[k], 1u)] = (uint32_t)j;
  }
}

__device__ __forceinline__ void order_rank(const int32_t* sJ, int W, const uint32_t* span,
                                           const uint32_t* scratch, uint16_t* rank,
                                           int32_t* sorted, int tid) {
  const BucketMap bucket(span);
  const uint32_t* start = scratch + kKeepJ + 2 * kOrderBuckets;
  for (int v = tid; v < W; v += kThreads) {
    const int32_t j = sJ[v];
    const int k = bucket(j);
    const uint32_t s = start[k], e = start[k + 1];
    uint32_t r = s;
    for (uint32_t u = s; u < e; ++u) r += (int32_t)scratch[u] < j ? 1u : 0u;
    rank[v] = (uint16_t)r;
    sorted[r] = j;
  }
}

// MODE: kStabCount (count and park rows), kStabF32 (FP32 selection fused),
// kStabBF16 / kStabFP8 (BF16 or FP8 image-2 rows: MFMA bounds with an exact
// FP32 re-rank, fused), or kCsrBF16: the BF16 selection over a caller's CSR.
// Fused: three workgroups per CU (LDS and registers are sized for it; four
// for kStabBF16 and kCsrBF16)
// CH: window records staged in LDS per round of the pair test.
//
// kCsrBF16 (epm_match on the tiles of the last query): instead of the pair
// test, the CSR's rows say which window positions are hits.  Every entry is
// mapped to its position (inverse permutation, window slots) and sets a bit of
// its query's bitmap; a row whose bits are fewer than its entries (candidates
// outside the window, repeated ones) and rows longer than kStage are listed
// for the exact match, as are tiles with windows over kKeepJ.  What bounds it
// then is what bounds the fused selection.  The window kernel it replaces here
// (a dense entry list in LDS, FP64 bounds per entry, one thread per query for
// the selection) took 205 us for 60000 queries with 60 candidates each, this
// one 57.
//
// Parked rows: a row's hits are known by window position and have to leave in
// ascending j.  The window's order by j is worked out once per tile
// (order_count, order_place, order_rank below: a bucket sort over the span of
// the window's j, O(window)); a row's hits then set bits by rank in a bitmap,
// and its four threads write the words in turn, from the places that the bits
// before them give.  (Ranking every row's hits against each other took 12400
// cycles of a tile's 59000 at 31 hits per row and 41900 of 161000 at 90; the
// order takes 3400 whatever the rows, the bitmaps 5000 and 20000.  The tile pass
// went from 87 to 81 us at six pairs of 20000 keypoints, from 137 to 113 at one
// of 60000 with FP8 rows, and the counting pass from 54 to 44.6 there.)
template <bool PERSIST, int MODE, int CH>
__global__ __launch_bounds__(kThreads, MODE == kStabBF16 || MODE == kCsrBF16 ? 4 : MODE != kStabCount ? 3 : 2) void k_stab_tile(StabArgs A) {
  constexpr bool FUSE = MODE != kStabCount;
  constexpr bool CSR = MODE == kCsrBF16;
  constexpr bool BF = MODE == kStabBF16 || CSR;  // BF16 rows of both images
  // BF16 / FP8: MFMA bounds and an exact re-rank on the masters
  constexpr bool RED = BF || MODE == kStabFP8;
  // hits by window position in bitmaps (kStabF32 lists them)
  constexpr bool BITS = RED || !FUSE;
  // record chunk (sC, sH, sXY, sE; sJ too unless FUSE keeps the window's j
  // in sJ_keep), reused for descriptor rows in the match phase
  constexpr int kRecRaw = FUSE ? rec_bytes(CH) - CH * 4 : rec_bytes(CH);
  constexpr int kMatchRaw = MODE == kStabF32    ? kFuseBytes
                           : BF                ? red_scratch(kBfKeep)
                           : MODE == kStabFP8  ? red_scratch(kF8Keep)
                                               : 0;
  // the window's order by j is kept there after the pair test; in kStabF32 its
  // scratch (then the bitmaps by rank) lies behind the record chunk, elsewhere
  // it is an array of its own
  constexpr bool kScratchInRaw = MODE == kStabF32;
  constexpr int kOrderRaw =
      CSR     ? 0
      : !FUSE ? kOrderBytes + kBruteBytes
      : kScratchInRaw ? (kRecRaw > kOrderBytes ? kRecRaw : kOrderBytes) + kRankBytes
                      : kOrderBytes;
  constexpr int kPairRaw = CSR ? 0 : kRecRaw > kOrderRaw ? kRecRaw : kOrderRaw;
  constexpr int kRaw = kMatchRaw > kPairRaw ? kMatchRaw : kPairRaw;
  __shared__ __attribute__((aligned(16))) unsigned char raw[kRaw];
  // BF16 / FP8: the window's reduced rows, kBfRows at a time (the first
  // chunk is copied in while the pair test runs)
  __shared__ __attribute__((aligned(16)))
  uint8_t bfrows[BF ? kBfRowBytes : MODE == kStabFP8 ? kF8RowBytes : 16];
  __shared__ int32_t sJ_store[FUSE ? kKeepJ : 1];
  uint32_t* sC = reinterpret_cast<uint32_t*>(raw);
  uint32_t* sH = sC + CH;
  float2* sXY = reinterpret_cast<float2*>(sH + CH);
  float* sE = reinterpret_cast<float*>(sXY + CH);
  int32_t* sJ = reinterpret_cast<int32_t*>(sE + CH);  // not FUSE
  // kStabF32: the hits of every query as 16-bit window positions
  __shared__ uint16_t hits_v[MODE == kStabF32 ? kTileQ : 1][MODE == kStabF32 ? kStage + 2 : 1];
  // the others: the hits of every query by window position
  __shared__ uint32_t bits_store[RED ? kTileQ * kRankWords : 1];
  __shared__ uint32_t rank_store[RED && !CSR ? kTileQ * kRankWords : 1];
  // kStabCount: the hits' image-2 indices where the window is longer than
  // kKeepJ (+ 1: rows in different banks), else the window's j and the bitmaps
  constexpr int kHitRow = kStage + 1;
  constexpr int kCountWords = kTileQ * kHitRow;
  static_assert(kCountWords >= 2 * kTileQ * kRankWords + kKeepJ, "bitmaps and the window's j");
  __shared__ uint32_t count_store[FUSE ? 1 : kCountWords];
  int32_t* hits = reinterpret_cast<int32_t*>(count_store);
  uint32_t* bit_rows = FUSE ? bits_store : count_store;
  const auto hit_bits = [&](int q) { return bit_rows + q * kRankWords; };
  uint32_t* scratch = kScratchInRaw ? reinterpret_cast<uint32_t*>(raw + kRaw - kRankBytes)
                      : FUSE        ? rank_store
                                    : count_store + kTileQ * kRankWords;
  int32_t* sJ_keep = FUSE ? sJ_store
                          : reinterpret_cast<int32_t*>(count_store + 2 * kTileQ * kRankWords);
  uint16_t* j_rank = reinterpret_cast<uint16_t*>(raw);          // by window position
  int32_t* j_sorted = reinterpret_cast<int32_t*>(raw + kKeepJ * 2);  // by rank
  __shared__ uint32_t j_span[2];  // the window's largest ~j and largest j
  constexpr int kLines = CSR ? 1 : kTileQ;
  __shared__ double qa[kLines], qb[kLines], qc[kLines], qn[kLines];
  __shared__ uint32_t qk[kTileQ], qmode[kTileQ], cnt[kTileQ];
  __shared__ int64_t qidx[kTileQ];
  __shared__ uint32_t slot_b[kSlots], slot_pref[kSlots + 1];
  // scanned, angle hits, brute-force and empty queries; BF16 fused: rows
  // ranked on bounds, rows left uncertified, exact distances evaluated
  __shared__ uint32_t tile_stats[kTileCounts];
  __shared__ unsigned long long tile_nnz;  // whole_rows: the tile's candidates
  __shared__ int next_tile;

  // a caller's CSR that did not fit its buffer is incomplete: nothing is written
  if (CSR && A.row_offsets[A.n1] > A.capacity) return;
  // one tile per workgroup, or (persistent) tiles from the queue until it is
  // exhausted; every workgroup leaves the loop once the counter passes the
  // last tile
  for (int iter = 0;; ++iter) {
    int tile;
    if (PERSIST) {
      if (threadIdx.x == 0) next_tile = (int)atomicAdd(A.queue, 1u);
      __syncthreads();
      const int t = next_tile;
      if (t >= A.num_tiles) break;
      tile = A.order ? (int)A.order[t] : t;
    } else {
      if (iter > 0) break;
      tile = A.block_tile ? (int)A.block_tile[blockIdx.x] : xcd_tile(blockIdx.x, A.num_tiles);
    }
    if (CSR && A.tile_wide[tile] != 0u) {  // matched by the wide-row pass
      if (!PERSIST) return;                // (a loop here would cost registers)
      __syncthreads();                     // next_tile is read before it is rewritten
      continue;
    }
    const StabTile T = A.tiles[tile];
    if (T.count == 0) {
      if (!PERSIST) return;
      __syncthreads();
      continue;
    }
    const PairDev& pd = A.pairs[T.pair];
    const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();

    if (wave == 0) {
      // the tile's queries with their lines, from the window pass
      const TileQuery tq = A.tile_q[(int64_t)tile * kTileQ + lane];
      if constexpr (!CSR) {
        qa[lane] = tq.a;
        qb[lane] = tq.b;
        qc[lane] = tq.c;
        qn[lane] = line_norm(tq.a, tq.b);  // as the key pass rounds it
      }
      qk[lane] = tq.key;
      qmode[lane] = tq.flag;
      qidx[lane] = tq.i;
      cnt[lane] = 0;
      if (lane < kTileCounts) tile_stats[lane] = 0u;
      if (lane < 2) j_span[lane] = 0u;
      if (lane == 0) tile_nnz = 0ull;
    }
    if constexpr (!CSR) {
      for (int k = tid; k < 2 * kOrderBuckets; k += kThreads) scratch[kKeepJ + k] = 0u;
      if constexpr (BITS)
        for (int k = tid; k < kTileQ * kRankWords; k += kThreads) bit_rows[k] = 0u;
    }
    {
      const TileWindow* w = A.windows + tile;
      if (tid < kSlots) slot_b[tid] = w->slot_b[tid];
      if (tid <= kSlots) slot_pref[tid] = w->slot_pref[tid];
    }
    __syncthreads();

    const int64_t total_len = slot_pref[kSlots];
    const bool fusable = total_len <= kFuseMaxWindow;
    uint32_t scanned = 0, angle_w = 0;  // angle_w: the wavefront's angle hits (uniform)
    // this lane's query of the pair test: its line stays in registers
    const int lq = wave * kQPerWave + (lane & (kQPerWave - 1));
    const bool line_live = qmode[lq] == kQueryNormal;
    const uint64_t live_mask = ballot(line_live);
    const bool any_live = ballot(line_live) != 0;
    const uint32_t lkey = qk[lq];
    double la = 0.0, lb = 0.0, lc = 0.0, ln = 0.0;
    if constexpr (!CSR) {
      la = qa[lq];
      lb = qb[lq];
      lc = qc[lq];
      ln = qn[lq];
    }
    const uint64_t same_query = 0x0001000100010001ull << (lane & (kQPerWave - 1));
    // the wavefront's key span [kmn, kmx] over its live queries: a record
    // whose interval misses every key of the span (circular distance from the
    // span's middle beyond its half-width plus the span's half-length, by the
    // triangle inequality on the circle of keys) cannot meet any of them and
    // is skipped without the per-query test
    uint32_t kmn = line_live ? lkey : 0xFFFFFFFFu, kmx = line_live ? lkey : 0u;
    kmn = row_reduce(kmn, 0xFFFFFFFFu, OpMin());
    kmx = row_reduce(kmx, 0u, OpMax());
    const uint32_t kmid = kmn + ((kmx - kmn) >> 1);
    const uint64_t khalf = ((uint64_t)(kmx - kmn) + 1u) >> 1;
    uint32_t lcnt = 0;
    // kCsrBF16: the row's length (0 past the tile), and whether its bits say it all
    int64_t csr_len = 0;
    bool csr_ok = false;
    if constexpr (CSR) {
      const int g = lane >> 4;
      const int64_t kb = pd.k_begin;
      int64_t o0 = 0;
      if (lq < T.count) {
        o0 = A.row_offsets[qidx[lq]];
        csr_len = A.row_offsets[qidx[lq] + 1] - o0;
      }
      const bool here = line_live && fusable && csr_len <= kStage;
      if (fusable) {
        for (int v = tid; v < (int)total_len; v += kThreads) {
          int s = 0;  // last slot with slot_pref[s] <= v
          #pragma unroll
          for (int step = 32; step > 0; step >>= 1)
            if (s + step <= kSlots && slot_pref[s + step] <= (uint32_t)v) s += step;
          sJ_keep[v] = A.rj[slot_b[s] + ((uint32_t)v - slot_pref[s])];
        }
      }
      #pragma unroll
      for (int k = g; k < kRankWords; k += 4) hit_bits(lq)[k] = 0u;
      // the slots that hold records, for every lane's entries
      uint64_t filled = ballot(slot_pref[lane + 1] > slot_pref[lane]);
      constexpr int kFly = 4;  // entries of a lane whose gathers are in flight together
      const int n = here ? (int)csr_len : 0;
      const int nmax = (int)wave_max_u32((uint32_t)n);
      for (int e0 = g; e0 < nmax; e0 += 4 * kFly) {
        uint32_t pos[kFly];
        #pragma unroll
        for (int u = 0; u < kFly; ++u)
          pos[u] = e0 + 4 * u < n ? A.rinv[kb + A.cols[o0 + e0 + 4 * u]] : 0u;
        int v[kFly];
        #pragma unroll
        for (int u = 0; u < kFly; ++u) v[u] = -1;
        for (uint64_t m = filled; m != 0ull; m &= m - 1ull) {
          const int s = (int)__builtin_ctzll(m);
          const uint32_t b = slot_b[s], p = slot_pref[s], len = slot_pref[s + 1] - p;
          #pragma unroll
          for (int u = 0; u < kFly; ++u)
            if (pos[u] - b < len) v[u] = (int)(p + (pos[u] - b));
        }
        #pragma unroll
        for (int u = 0; u < kFly; ++u)
          if (e0 + 4 * u < n && v[u] >= 0) atomicOr(&hit_bits(lq)[v[u] >> 5], 1u << (v[u] & 31));
      }
      wave_sync_lds();
      int set = 0;
      for (int k = g; k < kKeepJ / 32; k += 4) set += __popc(hit_bits(lq)[k]);
      set += lane_xor<16>(set);
      set += lane_xor<32>(set);
      csr_ok = here && set == n;
      __syncthreads();  // the window's j are complete
      if (fusable && total_len > 0)
        bf16_stage(A, 0, total_len < kBfRows ? (int)total_len : kBfRows, kb, sJ_keep, bfrows, wave,
                   lane);
    }
    // BF16: the query rows are loaded before the pair test so that their
    // latency hides behind it.  Lane l of wavefront w holds query
    // 16 w + (l & 15): as MFMA B operands its BF16 values at dimensions
    // 32 kk + 8 g .. + 7 (g = l >> 4), and its quarter, dimensions
    // 32 g .. 32 g + 31, as BF16 codes and as the FP32 master (the exact
    // chains pass their sum from quarter to quarter)
    bf16x8 bq[4];
    uint4 qcode[4];
    float4 qx[8];
    // FP8: the master's values at the B operand's dimensions, rounded to
    // BF16 after the pair test (the quarter for the exact chains is loaded
    // then, behind the first chunk)
    float4 qraw[8];
    if constexpr (MODE == kStabFP8) {
      const int g = lane >> 4;
      const bool ld = line_live && lq < T.count && fusable;
      const float4* m = reinterpret_cast<const float4*>(A.desc1) + qidx[lq] * 32;
      #pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        qraw[2 * kk] = ld ? m[kk * 8 + g * 2] : make_float4(0.f, 0.f, 0.f, 0.f);
        qraw[2 * kk + 1] = ld ? m[kk * 8 + g * 2 + 1] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
    if constexpr (BF) {
      const int g = lane >> 4;
      const bool ld = line_live && lq < T.count && fusable;
      const int64_t qi = qidx[lq];
      #pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const uint4 c = ld ? reinterpret_cast<const uint4*>(A.codes1)[qi * 16 + kk * 4 + g]
                           : make_uint4(0u, 0u, 0u, 0u);
        bq[kk] = __builtin_bit_cast(bf16x8, c);
        qcode[kk] = ld ? reinterpret_cast<const uint4*>(A.codes1)[qi * 16 + g * 4 + kk]
                    : make_uint4(0u, 0u, 0u, 0u);
      }
      #pragma unroll
      for (int u = 0; u < 8; ++u)
        qx[u] = ld ? reinterpret_cast<const float4*>(A.desc1)[qi * 32 + g * 8 + u]
                   : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int64_t base = 0; !CSR && base < total_len; base += CH) {
      const int clen = (int)(total_len - base < CH ? total_len - base : CH);
      uint32_t jn = 0u, jx = 0u;  // largest ~j and j of this thread's records
      for (int v = tid; v < clen; v += kThreads) {
        const int64_t virt = base + v;
        int s = 0;  // last slot with slot_pref[s] <= virt
        #pragma unroll
        for (int step = 32; step > 0; step >>= 1)
          if (s + step <= kSlots && slot_pref[s + step] <= virt) s += step;
        const int64_t pos = slot_b[s] + (virt - slot_pref[s]);
        sC[v] = A.rC[pos];
        sH[v] = A.rH[pos];
        sXY[v] = A.rxy[pos];
        sE[v] = A.reps[pos];
        if (FUSE ? virt < kKeepJ : fusable) {
          const int32_t j = A.rj[pos];
          sJ_keep[virt] = j;
          jn = max(jn, ~(uint32_t)j);
          jx = max(jx, (uint32_t)j);
        } else if (!FUSE) {
          sJ[v] = A.rj[pos];
        }
      }
      if (fusable && wave * kWave < clen) {
        jn = wave_max_u32(jn);
        jx = wave_max_u32(jx);
        if (lane == 0) {
          atomicMax(&j_span[0], jn);
          atomicMax(&j_span[1], jx);
        }
      }
      __syncthreads();
      if constexpr (RED) {
        // the first reduced rows of the window go to LDS behind the pair test
        if (base == 0 && fusable && total_len > 0) {
          const int nr0 = total_len < kBfRows ? (int)total_len : kBfRows;
          if constexpr (MODE == kStabFP8)
            f8_stage(A, 0, nr0, pd.k_begin, sJ_keep, bfrows, wave, lane);
          else
            bf16_stage(A, 0, nr0, pd.k_begin, sJ_keep, bfrows, wave, lane);
        }
      }
      if (fusable && base + CH >= total_len)
        order_count(sJ_keep, (int)total_len, j_span, scratch, tid);
      if (any_live) {
        // this wave's 16 queries (lane & 15) against four records per step
        // (lane >> 4), over the records of each group of 64 that can meet
        // the wave's key span; a hit's slot is the query's count plus its
        // rank among the query's lanes of the step, so every row lists its
        // hits in ascending window position
        const int g4 = lane >> 4;
        for (int g0 = 0; g0 < clen; g0 += kWave) {
          bool rel = false;
          if (g0 + lane < clen)
            rel = (uint64_t)key_distance(kmid, sC[g0 + lane]) <= (uint64_t)sH[g0 + lane] + khalf;
          uint64_t m = ballot(rel);
          if (line_live && lane < kQPerWave) scanned += (uint32_t)__popcll(m);
          // lane 16 g + t holds the record of group g in step t: the
          // (4 t + g)-th of them, in ascending position; a step takes its four
          // by one DPP move (picking them off the mask step by step, a chain of
          // scalar instructions, the pass took 650 us instead of 533 at six
          // pairs of 50000 keypoints and eps 50, 44.7 instead of 42.2 for 60000
          // queries counted at eps 2)
          const int cnt_m = __popcll(m);
          const int kth = 4 * (lane & 15) + g4;
          int mine_at = kth;
          if (m != ~0ull) mine_at = kth < cnt_m ? nth_bit(m, (uint32_t)kth) : kWave;
          const auto test = [&](int pick) {
            const int r = g0 + pick;
            // branch-free: nearly every step has lanes that pass the angle
            // test, and the SIMD runs the FP64 test for all of its lanes
            // anyway; each test is balloted on its own (a ballot of one
            // comparison is its lane mask as it stands)
            const int rr = pick < kWave ? r : g0;  // an index inside the chunk
            const uint32_t C = sC[rr], H = sH[rr];
            const float2 xy = sXY[rr];
            const bool key_ok = key_distance(lkey, C) <= H;
            const bool fp_ok = within_tolerance_n(la, lb, lc, ln, xy.x, xy.y, sE[rr]);
            const uint64_t vm = live_mask & ballot(pick < kWave);
            const uint64_t am = vm & ballot(key_ok);
            angle_w += (uint32_t)__popcll(am);
            const uint64_t all_hits = am & ballot(fp_ok);
            const bool hit = line_live & (pick < kWave) & key_ok & fp_ok;  // this lane's bit
            const uint64_t hm = all_hits & same_query;
            if (BITS && fusable) {
              if (hit) {
                const uint32_t v = (uint32_t)base + (uint32_t)r;
                atomicOr(&hit_bits(lq)[v >> 5], 1u << (v & 31u));
              }
            } else if (!RED && hit) {
              const uint32_t slot = lcnt + lanes_below(hm);
              if (slot < (uint32_t)kStage) {
                if (FUSE)
                  hits_v[lq][slot] = (uint16_t)(base + r);
                else
                  hits[lq * kHitRow + slot] = sJ[r];
              }
            }
            lcnt += (uint32_t)__popcll(hm);
          };
          for_steps<0>(mine_at, (cnt_m + 3) >> 2, test);
        }
      }
      __syncthreads();
    }
    if constexpr (!CSR) {
    if (line_live && lane < kQPerWave) cnt[lq] = lcnt;

    // queries whose line misses the epipole too far: exact scan of the pair
    uint32_t brute = 0;
    int32_t* brute_row = reinterpret_cast<int32_t*>(raw + kOrderBytes) + wave * kStage;  // not FUSE
    for (uint64_t bm = ballot(lane < kQPerWave && qmode[lq] == kQueryBrute); bm != 0ull;
         bm &= bm - 1ull) {
      const int q = wave * kQPerWave + (int)__builtin_ctzll(bm);
      const double a = qa[q], b = qb[q], c = qc[q], nrm = qn[q];
      uint32_t c0 = 0;
      brute += 1;
      for (int64_t base = pd.k_begin; base < pd.k_begin + pd.n; base += kWave) {
        const int64_t pos = base + lane;
        bool hit = false;
        if (pos < pd.k_begin + pd.n) {
          const float2 xy = A.rxy[pos];
          hit = within_tolerance_n(a, b, c, nrm, xy.x, xy.y, A.reps[pos]);
        }
        const uint64_t m = ballot(hit);
        if (!FUSE && hit) {  // FUSE: counted only, the row is rebuilt from the list
          const uint32_t slot = c0 + lanes_below(m);
          if (slot < (uint32_t)kStage) brute_row[slot] = A.rj[pos];
        }
        c0 += (uint32_t)__popcll(m);
      }
      if (lane == 0) cnt[q] = c0;
      if (!FUSE && c0 <= (uint32_t)kStage) {  // a short row is sorted and parked here
        for (int t = (int)c0 + lane; t < kStage; t += kWave) brute_row[t] = INT32_MAX;
        wave_sync_lds();
        wave_sort_lds(brute_row, kStage);
        for (int t = lane; t < (int)c0; t += kWave) A.staging[qidx[q] * kStage + t] = brute_row[t];
        wave_sync_lds();
      }
    }
    // The hits and counts of a wavefront's 16 queries were written by it, so
    // they are read without a barrier.
    {
      // the tile's counters gather in LDS; one thread adds them to the
      // query's counters once every wavefront has passed a later barrier
      const bool own = lane < kQPerWave && lq < T.count;
      const uint32_t nbrute = (uint32_t)__popcll(ballot(own && qmode[lq] == kQueryBrute));
      const uint32_t empty = (uint32_t)__popcll(ballot(own && qmode[lq] == kQueryEmpty));
      scanned = wave_sum_u32(scanned);
      const uint32_t angle_hits = angle_w;
      // rows longer than kStage of normal queries are written (and, fused,
      // matched) by the wide-row pass over the tile; the window pass cleared
      // the flag
      const uint64_t wm = ballot(own && qmode[lq] == kQueryNormal && cnt[lq] > (uint32_t)kStage);
      if (lane == 0) {
        atomicAdd(&tile_stats[0], scanned);
        atomicAdd(&tile_stats[1], angle_hits);
        atomicAdd(&tile_stats[2], nbrute);
        atomicAdd(&tile_stats[3], empty);
        if (wm != 0ull) {
          A.tile_wide[tile] = 1u;
          A.stats[kStatWide] = 1ull;
          if (A.pair_wide) atomicAdd(&A.pair_wide[T.pair], 1u);
        }
      }
      if (A.whole_rows) {  // (the halves' sums over a wavefront fit 32 bits)
        const uint32_t len = own && qmode[lq] != kQueryEmpty ? cnt[lq] : 0u;
        const uint64_t sum =
            wave_sum_u32(len & 0xFFFFu) + ((uint64_t)wave_sum_u32(len >> 16) << 16);
        if (lane == 0) atomicAdd(&tile_nnz, (unsigned long long)sum);
      }
    }
    (void)brute;
    }

    // FUSE: four threads per query select its match
    const int q = tid >> 2, part = tid & 3;
    const bool mine = q < T.count && qmode[q] == kQueryNormal &&
                      cnt[q] <= (uint32_t)kStage && fusable;

    // row lengths, and short rows parked in ascending j
    // (the fused modes write the row length with the match, in one record)
    if constexpr (!CSR) {
      if (!FUSE && part == 0 && q < T.count)
        A.counts[qidx[q]] = qmode[q] == kQueryEmpty ? 0u : cnt[q];
      const uint32_t n = q < T.count && qmode[q] != kQueryEmpty ? cnt[q] : 0u;
      int32_t* dst = A.staging + qidx[q] * kStage;
      if (fusable && total_len > 0) {
        order_place(sJ_keep, (int)total_len, j_span, scratch, tid);
        __syncthreads();
        order_rank(sJ_keep, (int)total_len, j_span, scratch, j_rank, j_sorted, tid);
        __syncthreads();
        const int words = ((int)total_len + 31) >> 5;
        uint32_t* bits = scratch + q * kRankWords;
        for (int k = part; k < words; k += 4) bits[k] = 0u;
        wave_sync_lds();
        if (mine) {
          if constexpr (BITS) {
            uint32_t w[kWordsPer];
            #pragma unroll
            for (int i = 0; i < kWordsPer; ++i) w[i] = hit_bits(q)[4 * i + part];
            #pragma unroll
            for (int i = 0; i < kWordsPer; ++i) {
              if (4 * i >= words) break;
              const uint16_t* of = j_rank + (4 * i + part) * 32;
              while (w[i] != 0u) {  // four hits at a time, their ranks read together
                uint32_t r[4];
                bool has[4];
                #pragma unroll
                for (int m = 0; m < 4; ++m) {
                  has[m] = w[i] != 0u;
                  r[m] = of[__builtin_ctz(w[i] | 0x80000000u)];
                  w[i] &= w[i] - 1u;
                }
                #pragma unroll
                for (int m = 0; m < 4; ++m)
                  if (has[m]) atomicOr(&bits[r[m] >> 5], 1u << (r[m] & 31u));
              }
            }
          } else {
            #pragma unroll 4
            for (uint32_t u = part; u < n; u += 4) {
              const uint32_t r = j_rank[hits_v[q][u]];
              atomicOr(&bits[r >> 5], 1u << (r & 31u));
            }
          }
        }
        wave_sync_lds();
        // words k = part (mod 4) are the thread's, so that the row's four
        // threads write to neighbouring places
        uint32_t w[kWordsPer];
        #pragma unroll
        for (int i = 0; i < kWordsPer; ++i)
          w[i] = mine && 4 * i + part < words ? bits[4 * i + part] : 0u;
        uint32_t row = 0u;  // the row's entries in words [0, 4 i)
        #pragma unroll
        for (int i = 0; i < kWordsPer; ++i) {
          if (4 * i >= words) break;
          const uint32_t own = (uint32_t)__popc(w[i]);
          uint32_t sum = own;  // over the row's threads up to this one
          const uint32_t t1 = dpp<0x111, 0xF>(0u, sum);
          sum += part >= 1 ? t1 : 0u;
          const uint32_t t2 = dpp<0x112, 0xF>(0u, sum);
          sum += part >= 2 ? t2 : 0u;
          int32_t* to = dst + row + (sum - own);
          row += dpp<0xFF, 0xF>(0u, sum);  // the sum of the last of the four
          const int32_t* of = j_sorted + (4 * i + part) * 32;
          while (w[i] != 0u) {  // four hits at a time
            int32_t j[4];
            bool has[4];
            #pragma unroll
            for (int m = 0; m < 4; ++m) {
              has[m] = w[i] != 0u;
              j[m] = of[__builtin_ctz(w[i] | 0x80000000u)];
              w[i] &= w[i] - 1u;
            }
            #pragma unroll
            for (int m = 0; m < 4; ++m) {
              if (has[m]) to[m] = j[m];
            }
            to += 4;
          }
        }
      }
      if constexpr (!FUSE) {
        // longer windows: four threads per row, each placing a quarter of its
        // hits by rank (the j of a row are distinct, so a hit's place is the
        // number of smaller hits); a thread ranks up to four of its hits in one
        // pass over the row
        if (!fusable && n <= (uint32_t)kStage && qmode[q] == kQueryNormal) {
          const int32_t* row = hits + q * kHitRow;
          for (uint32_t t0 = part; t0 < n; t0 += 16) {
            int32_t v[4];
            uint32_t r[4];
            #pragma unroll
            for (int m = 0; m < 4; ++m) {
              v[m] = t0 + 4 * m < n ? row[t0 + 4 * m] : INT32_MIN;
              r[m] = 0;
            }
            #pragma unroll 4
            for (uint32_t u = 0; u < n; ++u) {
              const int32_t h = row[u];
              #pragma unroll
              for (int m = 0; m < 4; ++m) r[m] += h < v[m] ? 1u : 0u;
            }
            #pragma unroll
            for (int m = 0; m < 4; ++m)
              if (t0 + 4 * m < n) dst[r[m]] = v[m];
          }
        }
      } else if (n > 0 && n <= (uint32_t)kStage && !mine && part == 0) {
        // rows that are not kept (brute-force queries, windows that are not
        // fused) are marked and rebuilt from the list
        dst[0] = kRowNotParked;
      }

      if (FUSE && part == 0 && q < T.count) {
        const uint32_t mode = qmode[q];
        if (mode != kQueryEmpty &&
            (mode != kQueryNormal || (cnt[q] <= (uint32_t)kStage && !fusable))) {
          const unsigned long long at = atomicAdd(&A.stats[kStatRest], 1ull);
          A.rest[at] = (uint32_t)qidx[q] | kRestRebuild;
        }
      }
    }
    if constexpr (MODE == kStabF32) {
      const int nq = mine ? (int)cnt[q] : 0;
      const int64_t kb = pd.k_begin;
      float4* rows4 = reinterpret_cast<float4*>(raw);
      // the query row stays in registers for all its hits
      float4 qreg[32];
      {
        const float4* qrow = reinterpret_cast<const float4*>(A.desc1) + qidx[q] * 32;
        #pragma unroll
        for (int k = 0; k < 32; ++k) qreg[k] = mine ? qrow[k] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      Top2 best;
      int cur = part;
      if (fusable && total_len > 0) {
        const int wlen = (int)total_len;
        for (int c0 = 0; c0 < wlen; c0 += kFuseRows) {
          const int nr = wlen - c0 < kFuseRows ? wlen - c0 : kFuseRows;
          // the window's order (first) or the previous rows are no longer read
          __syncthreads();
          fuse_stage(A, c0, nr, kb, sJ_keep, rows4, wave, lane);
          wait_lds_copies();
          __syncthreads();
          // the row's hits are in ascending window position: this lane's
          // hits in the chunk continue from where the previous chunk stopped
          for (; cur < nq; cur += 4) {
            const int v = hits_v[q][cur];
            if (v >= c0 + nr) break;
            const float4* wr = rows4 + (v - c0) * (kFuseStride / 4);
            float acc = 0.0f;
            #pragma unroll
            for (int k = 0; k < 32; ++k) acc = canonical_step4(acc, qreg[k], wr[k]);
            best.insert(acc, sJ_keep[v]);
          }
        }
      }
      // the four parts of a query are adjacent lanes and hold distinct hits
      best = merge_top2(best, lane_xor_top2<1>(best));
      best = merge_top2(best, lane_xor_top2<2>(best));
      if (part == 0 && q < T.count) {
        const bool empty = qmode[q] == kQueryEmpty;
        A.qrec[qidx[q]] = query_record(empty ? 0u : cnt[q], A.ratio, best, mine || empty);
      }
    } else if constexpr (RED) {
      constexpr bool F8 = MODE == kStabFP8;
      constexpr int kKeep = F8 ? kF8Keep : kBfKeep;
      constexpr int kQTasks = 4 * kKeep;  // exact distances a query can list
      // lane l of wavefront w: query 16 w + (l & 15), lane group g = l >> 4
      const int q2 = wave * kQPerWave + (lane & (kQPerWave - 1));
      const int g = lane >> 4;
      const bool mine2 = CSR ? csr_ok
                             : q2 < T.count && qmode[q2] == kQueryNormal &&
                                   cnt[q2] <= (uint32_t)kStage && fusable;
      const int64_t kb = pd.k_begin;
      const int64_t qi2 = qidx[q2];
      // per chunk row: (|w^|^2, bound norm, rounding bound) -- the record
      // chunk is dead -- then the per-query task lists
      float4* w_terms = reinterpret_cast<float4*>(raw);
      uint16_t* qtask = reinterpret_cast<uint16_t*>(w_terms + kBfRows);  // [kTileQ][kQTasks]
      // the query's BF16 norm and the measured norm of its rounding error
      // (x - x^, exact in FP32), summed over its four quarters (FP8: the
      // query rounded to BF16 here, to nearest even, into the B operand)
      float qn_part = 0.0f, qe_part = 0.0f;
      #pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const float4 xa = F8 ? qraw[2 * kk] : qx[2 * kk];
        const float4 xb = F8 ? qraw[2 * kk + 1] : qx[2 * kk + 1];
        const float x[8] = {xa.x, xa.y, xa.z, xa.w, xb.x, xb.y, xb.z, xb.w};
        uint32_t w[4];
        if constexpr (F8) {
          #pragma unroll
          for (int h = 0; h < 4; ++h) {
            const uint32_t u0 = __float_as_uint(x[2 * h]), u1 = __float_as_uint(x[2 * h + 1]);
            w[h] = ((u0 + 0x7FFFu + ((u0 >> 16) & 1u)) >> 16) |
                   ((u1 + 0x7FFFu + ((u1 >> 16) & 1u)) & 0xFFFF0000u);
          }
          bq[kk] = __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
        } else {
          w[0] = qcode[kk].x;
          w[1] = qcode[kk].y;
          w[2] = qcode[kk].z;
          w[3] = qcode[kk].w;
        }
        #pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float y = __uint_as_float(e & 1 ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16));
          qn_part = __builtin_fmaf(y, y, qn_part);
          const float d = x[e] - y;
          qe_part = __builtin_fmaf(d, d, qe_part);
        }
      }
      if constexpr (F8) {
        const bool ld = mine2;
        const float4* m = reinterpret_cast<const float4*>(A.desc1) + qi2 * 32 + g * 8;
        #pragma unroll
        for (int u = 0; u < 8; ++u) qx[u] = ld ? m[u] : make_float4(0.f, 0.f, 0.f, 0.f);
      }
      qn_part += lane_xor<16>(qn_part);
      qe_part += lane_xor<16>(qe_part);
      qn_part += lane_xor<32>(qn_part);
      qe_part += lane_xor<32>(qe_part);
      // per-query bound terms, inflated for the FP32 sums (2^-24 per term)
      const float q_nb = sqrtf(qn_part) * (1.0f + 2e-5f);
      const float q_db = sqrtf(qe_part) * (1.0f + 2e-5f) + 1e-30f;
      BfKeep<kKeep> st;
      Top2 best;
      uint32_t evals = 0;
      bool cert = mine2;  // a tile without window records has only empty rows
      if (fusable && total_len > 0) {
        const int wlen = (int)total_len;
        for (int c0 = 0; c0 < wlen; c0 += kBfRows) {
          const int nr = wlen - c0 < kBfRows ? wlen - c0 : kBfRows;
          if (c0 > 0) {
            __syncthreads();  // the previous rows are no longer read
            if constexpr (F8)
              f8_stage(A, c0, nr, kb, sJ_keep, bfrows, wave, lane);
            else
              bf16_stage(A, c0, nr, kb, sJ_keep, bfrows, wave, lane);
          }  // the first rows were started during the pair test
          // this query's hits in the chunk
          static_assert(kBfRows == 32, "a chunk's hits are one word of the bitmap");
          const uint32_t hmask = mine2 ? hit_bits(q2)[c0 / 32] : 0u;
          // FP8: the scale and the rounding-error bound of the row whose
          // terms this thread works out below, read beside the copies
          float f8s = 1.0f, f8e = 0.0f;
          if constexpr (F8) {
            const int r = tid / (kThreads / kBfRows);
            if (tid % (kThreads / kBfRows) == 0) {
              const int64_t j = kb + sJ_keep[c0 + (r < nr ? r : nr - 1)];
              f8s = A.f8scale2[j];
              f8e = A.f8err2[j];
            }
          }
          wait_lds_copies();
          __syncthreads();
          {
            // norms of the chunk's rows: kTpr threads per row
            constexpr int kTpr = kThreads / kBfRows;
            const int r = tid / kTpr, part4 = tid % kTpr;
            float sn = 0.0f;
            if constexpr (F8) {
              static_assert(kTpr * 16 == 128, "sixteen codes per thread");
              sn = e4m3x16_sumsq(
                  *reinterpret_cast<const uint4*>(bfrows + r * kF8Stride + part4 * 16), 0.0f);
            } else {
              const uint4* rp =
                  reinterpret_cast<const uint4*>(bfrows + r * kBfStride + part4 * (256 / kTpr));
              #pragma unroll
              for (int t = 0; t < 16 / kTpr; ++t) {
                const uint4 c = rp[t];
                const uint32_t w[4] = {c.x, c.y, c.z, c.w};
                #pragma unroll
                for (int e = 0; e < 8; ++e) {
                  const float y =
                      __uint_as_float(e & 1 ? (w[e >> 1] & 0xFFFF0000u) : (w[e >> 1] << 16));
                  sn = __builtin_fmaf(y, y, sn);
                }
              }
            }
            static_assert(kTpr == 8, "eight threads per row");
            sn += lane_xor<1>(sn);
            sn += lane_xor<2>(sn);
            sn += lane_xor<4>(sn);
            if (part4 == 0) {
              if constexpr (F8) {
                // w^ = s c: |w^|^2 = s^2 |c|^2, and the MFMA scores of the
                // codes are scaled by s; the last term is the row's
                // rounding-error bound rounded up to FP16
                const float wn = sn * (f8s * f8s);
                const float nb = sqrtf(wn) * (1.0f + 2e-5f);
                w_terms[r] = make_float4(wn, nb, f8s, __uint_as_float(half_up(f8e)));
              } else {
                const float nb = sqrtf(sn) * (1.0f + 2e-5f);
                // |w - w^| <= u |w^| / (1 - u) for a row rounded to nearest even
                const float db =
                    nb * (float)(Fmt<0>::kUnit / (1.0 - Fmt<0>::kUnit) * (1.0 + 1e-6)) + 1e-30f;
                w_terms[r] = make_float4(sn, nb, db, __uint_as_float(half_up(nb)));
              }
            }
          }
          __syncthreads();
          if (ballot(hmask != 0u) != 0ull) {
            // S^T = W^ Q^T on MFMA, for the row blocks where one of the
            // wave's queries has a hit (the others are never read).  Block
            // position m of block cb holds window row 16 cb + 4 (m & 3) +
            // (m >> 2), so that the scores of consecutive rows -- a query's
            // hits come in runs of neighbouring window positions -- land in
            // its four lane groups in turn and the lanes share the work
            f32x4 acc[kBfBlocks];
            const int arow = ((lane & 3) << 2) | ((lane >> 2) & 3);
            #pragma unroll
            for (int cb = 0; cb < kBfBlocks; ++cb) {
              acc[cb] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
              if (ballot(((hmask >> (16 * cb)) & 0xFFFFu) != 0u) == 0ull) continue;
              #pragma unroll
              for (int kk = 0; kk < 4; ++kk) {
                bf16x8 a;
                if constexpr (F8)
                  a = e4m3x8_bf16(*reinterpret_cast<const uint2*>(
                      bfrows + (cb * 16 + arow) * kF8Stride + kk * 32 + g * 8));
                else
                  a = *reinterpret_cast<const bf16x8*>(bfrows + (cb * 16 + arow) * kBfStride +
                                                       (kk * 32 + g * 8) * 2);
                acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, bq[kk], acc[cb], 0, 0, 0);
              }
            }
            // this lane's hits among its scores: slot 4 cb + i (element i of
            // acc[cb]) is window row 16 cb + 4 i + g; only set slots are
            // visited
            uint32_t slots = 0u;
            #pragma unroll
            for (int cb = 0; cb < kBfBlocks; ++cb)
              #pragma unroll
              for (int i = 0; i < 4; ++i)
                slots |= ((hmask >> (16 * cb + 4 * i + g)) & 1u) << (4 * cb + i);
            // the slots in a fixed order, a block's four row terms read
            // together; a slot without a hit leaves the state unchanged
            #pragma unroll
            for (int cb = 0; cb < kBfBlocks; ++cb) {
              if (((slots >> (4 * cb)) & 0xFu) == 0u) continue;
              float4 wt[4];
              #pragma unroll
              for (int i = 0; i < 4; ++i) wt[i] = w_terms[16 * cb + 4 * i + g];
              #pragma unroll
              for (int i = 0; i < 4; ++i) {
                if (!((slots >> (4 * cb + i)) & 1u)) continue;
                const float sc = F8 ? wt[i].z * acc[cb][i] : acc[cb][i];
                const float at = (qn_part + wt[i].x) - 2.0f * sc;
                const uint32_t term = __float_as_uint(wt[i].w);
                st.add(at, (uint32_t)(c0 + 16 * cb + 4 * i + g) | (term << 16), wt[i].y,
                       F8 ? term : 0u);
              }
            }
          }
        }
        // this lane's bounds: the kept candidates' D_lo and D_hi (two
        // smallest D_hi), and a lower bound on D_lo of the pushed-out ones
        float klo[kKeep];
        float u1 = __builtin_inff(), u2 = __builtin_inff();
        #pragma unroll
        for (int t = 0; t < kKeep; ++t) {
          float dlo = __builtin_inff(), dhi = __builtin_inff();
          if (st.pk[t] != kNoPick) {
            if constexpr (F8)  // the lane's largest row norm for the MFMA term
              bounds_from(st.a[t], st.nb_max, q_nb, q_db + half_value(st.pk[t] >> 16), dlo, dhi);
            else
              bf_bounds(st.a[t], half_value(st.pk[t] >> 16), q_nb, q_db, dlo, dhi);
          }
          klo[t] = dlo;
          u2 = fminf(u2, fmaxf(u1, dhi));
          u1 = fminf(u1, dhi);
        }
        float dmin = __builtin_inff();
        if (st.a_drop != __builtin_inff()) {
          float dhi_unused;
          if constexpr (F8)
            bounds_from(st.a_drop, st.nb_max, q_nb, q_db + half_value(st.ew_max), dmin,
                        dhi_unused);
          else
            bf_bounds(st.a_drop, st.nb_max, q_nb, q_db, dmin, dhi_unused);
        }
        bool bad = st.bad || !(u1 == u1) || !(u2 == u2) || !(dmin == dmin);
        // the row's U2 and smallest dropped bound over its four lanes
        const auto join = [&](float o1, float o2, float od, uint32_t ob) {
          u2 = fminf(fmaxf(u1, o1), fminf(u2, o2));
          u1 = fminf(u1, o1);
          dmin = fminf(dmin, od);
          bad |= ob != 0u;
        };
        join(lane_xor<16>(u1), lane_xor<16>(u2), lane_xor<16>(dmin), lane_xor<16>((uint32_t)bad));
        join(lane_xor<32>(u1), lane_xor<32>(u2), lane_xor<32>(dmin), lane_xor<32>((uint32_t)bad));
        // nothing dropped (dmin = +inf): every candidate that can be best or
        // second is kept, including rows of fewer than two candidates (U2 = +inf)
        cert = mine2 && !bad && (dmin == __builtin_inff() || dmin > u2);
        // the row's exact distances (kept candidates within U2) are listed
        // per query and dealt to its four lanes
        uint32_t tmask = 0u;
        #pragma unroll
        for (int t = 0; t < kKeep; ++t)
          if (cert && st.pk[t] != kNoPick && klo[t] <= u2) tmask |= 1u << t;
        const uint32_t myn = (uint32_t)__popc(tmask);
        const uint32_t n0 = row_bcast<0>(myn), n1 = row_bcast<1>(myn), n2 = row_bcast<2>(myn),
                       n3 = row_bcast<3>(myn);
        const uint32_t before = (g > 0 ? n0 : 0u) + (g > 1 ? n1 : 0u) + (g > 2 ? n2 : 0u);
        const uint32_t qtotal = n0 + n1 + n2 + n3;
        uint16_t* mylist = qtask + q2 * kQTasks;
        {
          uint32_t k = before;
          #pragma unroll
          for (int t = 0; t < kKeep; ++t)
            if ((tmask >> t) & 1u) mylist[k++] = (uint16_t)(st.pk[t] & 0xFFFFu);
        }
        wave_sync_lds();
        // one task of each query per round: the query's four lanes load their
        // quarters of the candidate's FP32 row (the next round's while this
        // one is summed) and pass the canonical sum on from quarter to
        // quarter, so it runs over dimensions 0 .. 127 in order
        const uint32_t rounds = wave_max_u32(qtotal);
        const float4* w2 = reinterpret_cast<const float4*>(A.desc2);
        auto wslice = [&](uint32_t k, float4* dst) {
          const bool has = k < qtotal;
          const int32_t j = has ? sJ_keep[mylist[k]] : 0;
          const float4* wr = w2 + (kb + j) * 32 + g * 8;
          #pragma unroll
          for (int u = 0; u < 8; ++u) dst[u] = has ? wr[u] : make_float4(0.f, 0.f, 0.f, 0.f);
        };
        float4 wcur[8], wnext[8];
        if (rounds > 0) wslice(0, wcur);
        for (uint32_t rd = 0; rd < rounds; ++rd) {
          if (rd + 1 < rounds) wslice(rd + 1, wnext);
          const auto quarter = [&](float acc) {
            #pragma unroll
            for (int u = 0; u < 8; ++u) acc = canonical_step4(acc, qx[u], wcur[u]);
            return __float_as_uint(acc);
          };
          // quarter by quarter, each one's result from its own lane group
          float sum = __uint_as_float(row_bcast<0>(quarter(0.0f)));
          sum = __uint_as_float(row_bcast<1>(quarter(sum)));
          sum = __uint_as_float(row_bcast<2>(quarter(sum)));
          sum = __uint_as_float(row_bcast<3>(quarter(sum)));
          if (rd < qtotal && g == 0) {
            best.insert(sum, sJ_keep[mylist[rd]]);
            ++evals;
          }
          #pragma unroll
          for (int u = 0; u < 8; ++u) wcur[u] = wnext[u];
        }
      }
      if constexpr (CSR) {
        if (g == 0 && q2 < T.count) {
          if (csr_len == 0 || (mine2 && cert)) {
            write_match_to(A.ratio, A.best_idx, A.best_dist, A.second_dist, qi2, best, false);
          } else {
            const unsigned long long at = atomicAdd(A.rest_count, 1ull);
            A.rest[at] = (uint32_t)qi2;
          }
        }
        // rows listed for what they are, not for their bounds
        const uint32_t n_long =
            (uint32_t)__popcll(ballot(g == 0 && q2 < T.count && csr_len > 0 && !mine2));
        if (lane == 0) atomicAdd(&tile_stats[7], n_long);
      } else if (g == 0 && q2 < T.count) {  // lane group 0 holds the query's selection
        const bool empty = qmode[q2] == kQueryEmpty;
        A.qrec[qi2] = query_record(empty ? 0u : cnt[q2], A.ratio, best, (mine2 && cert) || empty);
        if (mine2 && !cert) {
          const unsigned long long at = atomicAdd(&A.stats[kStatRest], 1ull);
          A.rest[at] = (uint32_t)qi2;
        }
      }
      const uint32_t n_rank = (uint32_t)__popcll(ballot(mine2 && g == 0 && (!CSR || csr_len > 0)));
      const uint32_t n_unc = (uint32_t)__popcll(ballot(mine2 && g == 0 && !cert));
      const uint32_t n_ev = wave_sum_u32(evals);
      if (lane == 0) {
        atomicAdd(&tile_stats[4], n_rank);
        atomicAdd(&tile_stats[5], n_unc);
        atomicAdd(&tile_stats[6], n_ev);
      }
    }
    // the tile's counters: complete once every wavefront has passed a barrier
    // after adding its share (the match phase has one unless it was skipped);
    // written per tile, summed on the host when they are asked for
    // (the BF16 phase adds its counters after its last barrier: one more)
    if (!FUSE || RED || !(fusable && total_len > 0)) __syncthreads();
    if (CSR) {
      if (A.match_stats && tid < 4) {
        // rows ranked, uncertified, listed otherwise, exact distances
        const uint32_t c = tile_stats[tid == 0 ? 4 : tid == 1 ? 5 : tid == 2 ? 7 : 6];
        if (c) atomicAdd(&A.match_stats[tid], (unsigned long long)c);
      }
    } else if (A.whole_rows && tid == kWave) {
      atomicAdd(&A.stats[kStatNnz], tile_nnz);
    } else if (A.tile_counts && tid == 0) {
      const uint64_t nb = tile_stats[2];
      unsigned long long* tc = A.tile_counts + (int64_t)tile * kTileCounts;
      tc[0] = (unsigned long long)tile_stats[0] + nb * (uint64_t)pd.n;
      tc[1] = (unsigned long long)tile_stats[1] + nb * (uint64_t)pd.n;
      tc[2] = nb;
      tc[3] = tile_stats[3];
      tc[4] = tile_stats[4];
      tc[5] = tile_stats[5];
      tc[6] = tile_stats[6];
      tc[7] = 0ull;
    }
    if (PERSIST) __syncthreads();  // the tile's LDS is dead before the next one starts
  }
}

// The pass after the tiles, in one launch: row offsets, matches and parked
// rows.  A workgroup owns kFinishRows consecutive queries: it scans their row
// lengths, publishes their sum, finds the sum of all earlier workgroups by
// looking back over what those have published, and then writes its offsets,
// the fused pass's matches (unless a later pass writes them) and the parked
// (already sorted) short rows.  After a counting pass the long rows of
// brute-force queries are queued for k_fill_long (a fused pass has listed what
// it leaves); long rows of normal queries belong to the wide-row pass.
//
// A word of row_sums is a sum with a flag in its top bits: of the workgroup
// alone, or of it and all before it.  Nothing has to be waited for: the row
// lengths are complete when the launch starts, so a workgroup that finds
// nothing published after kFinishPolls looks adds up that workgroup's lengths
// itself.  What bounds it: the latency of its three dependent steps (lengths,
// look-back, stores), so the first 16 entries of every row are on their way
// before the look-back; on large batches the staging reads and the CSR.  The
// separate launches it replaces (partial sums, offsets, matches, rows) took
// 4.7 + 5.7 + 4.7 + 9.0 us for 120000 queries; this takes 13.9.  Beyond what
// the chip holds about twice over, the look-back walks over the workgroups
// that run at the same time in every workgroup, and the separate launches are
// faster again: whole calls of 84000 / 168000 / 336000 / 672000 queries
// 145 / 215 / 352 / 652 us with this one, 155 / 222 / 353 / 635 with those.
constexpr int kCopyLanes = 16;  // lanes per row
constexpr int kFinishThreads = 1024;
constexpr int kFinishWaves = kFinishRows / kWave;  // wavefronts that hold a query per lane
constexpr int kFinishGroups = kFinishThreads / kCopyLanes;
constexpr int kFinishPer = kFinishRows / kFinishGroups;  // rows per group of lanes
constexpr int kFinishPolls = 256;
constexpr int64_t kFinishOneLaunch = 262144;  // queries
constexpr uint64_t kSumOwn = 1ull << 62, kSumAll = 2ull << 62, kSumMask = (1ull << 62) - 1ull;

__device__ __forceinline__ uint32_t row_length(const StabArgs& A, int64_t i) {
  return A.qrec ? A.qrec[i].x : A.counts[i];
}

// The rows do not fit, and the caller is told so instead (uniform).
__device__ __forceinline__ bool rows_dropped(const StabArgs& A) {
  return A.whole_rows && (int64_t)A.stats[kStatNnz] > A.capacity;
}

// Sum of the row lengths before workgroup b, by its first kFinishRows threads
// (the others take part in the barriers); every thread gets it.
__device__ __forceinline__ int64_t look_back(const StabArgs& A, int64_t b, int64_t* s_sum,
                                             int* s_all) {
  const int lane = lane_id(), wave = wave_id();
  int64_t before = 0;
  for (int64_t top = b; top > 0; top -= kFinishRows) {
    if (wave < kFinishWaves) {
      const int64_t p = top - 1 - (int64_t)threadIdx.x;
      uint64_t w = kSumAll;  // before the first workgroup
      if (p >= 0) {
        w = __hip_atomic_load(&A.row_sums[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        for (int k = 0; k < kFinishPolls && (w >> 62) == 0; ++k) {
          __builtin_amdgcn_s_sleep(1);
          w = __hip_atomic_load(&A.row_sums[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if ((w >> 62) == 0) {
          w = kSumOwn;
          for (int k = 0; k < kFinishRows; ++k) w += row_length(A, p * kFinishRows + k);
        }
      }
      // workgroups up to the nearest one with a complete sum
      const uint64_t all = ballot((w >> 62) == 2);
      const int last = all != 0ull ? (int)__builtin_ctzll(all) : kWave - 1;
      int64_t v = lane <= last ? (int64_t)(w & kSumMask) : 0;
      #pragma unroll
      for (int off = 1; off < kWave; off <<= 1) v += __shfl_xor(v, off);
      if (lane == 0) {
        s_sum[wave] = v;
        s_all[wave] = all != 0ull;
      }
    }
    __syncthreads();
    bool done = false;
    #pragma unroll
    for (int k = 0; k < kFinishWaves; ++k) {
      before += done ? 0 : s_sum[k];
      done |= s_all[k] != 0;
    }
    if (done) break;
    __syncthreads();  // the sums are read before they are written again
  }
  return before;
}

__global__ __launch_bounds__(kFinishThreads) void k_finish_rows(StabArgs A,
                                                                int64_t* __restrict__ offsets) {
  __shared__ int64_t s_off[kFinishRows], s_sum[kFinishWaves], s_back[kFinishWaves];
  __shared__ uint32_t s_len[kFinishRows];
  __shared__ int s_all[kFinishWaves];
  static_assert(kCopyLanes <= kStage && kFinishPer <= 32, "first pieces; one bit per row");
  const int tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const int64_t b = blockIdx.x, i0 = b * kFinishRows, i = i0 + tid;
  const bool mine = tid < kFinishRows && i < A.n1;  // this thread's query
  const bool dropped = rows_dropped(A);
  uint4 rec = make_uint4(0u, (uint32_t)kMatchDeferred, 0u, 0u);
  if (mine) {
    if (A.qrec) rec = A.qrec[i];
    else rec.x = A.counts[i];
  }
  // the lengths' exclusive scan
  int64_t incl = rec.x;
  if (wave < kFinishWaves) {
    s_len[tid] = rec.x;
    // (the halves' sums over a wavefront fit 32 bits)
    incl = (int64_t)wave_scan_u32(rec.x & 0xFFFFu) + ((int64_t)wave_scan_u32(rec.x >> 16) << 16);
    if (lane == kWave - 1) s_sum[wave] = incl;
  }
  __syncthreads();
  // the rows' first pieces; its first word tells whether a row was parked
  const int grp = tid / kCopyLanes, sub = tid % kCopyLanes;
  int32_t v[kFinishPer];
  #pragma unroll
  for (int u = 0; u < kFinishPer; ++u) {
    const int row = u * kFinishGroups + grp;
    const uint32_t len = s_len[row];
    v[u] = (uint32_t)sub < len && len <= (uint32_t)kStage ? A.staging[(i0 + row) * kStage + sub] : 0;
  }
  int64_t total = 0;
  #pragma unroll
  for (int k = 0; k < kFinishWaves; ++k) {
    incl += k < wave ? s_sum[k] : 0;
    total += s_sum[k];
  }
  if (tid == 0)
    __hip_atomic_store(&A.row_sums[b], (b == 0 ? kSumAll : kSumOwn) | (uint64_t)total, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  if (wave < kFinishWaves) s_off[tid] = incl - rec.x;
  const int64_t before = look_back(A, b, s_back, s_all);
  if (b == 0) __syncthreads();  // s_off is complete (look_back has a barrier otherwise)
  if (tid == 0 && b > 0)
    __hip_atomic_store(&A.row_sums[b], kSumAll | (uint64_t)(before + total), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  if (mine) offsets[i] = before + s_off[tid];
  if (b == (int64_t)gridDim.x - 1 && tid == 0) {
    offsets[A.n1] = before + total;
  }
  if (dropped) return;
  if (mine && (int32_t)rec.y != kMatchDeferred) {
    A.best_idx[i] = (int32_t)rec.y;
    A.best_dist[i] = __uint_as_float(rec.z);
    A.second_dist[i] = __uint_as_float(rec.w);
  }
  uint32_t parked = 0u;  // bit u: the row's pieces are copied
  uint32_t longest = 0u;
  #pragma unroll
  for (int u = 0; u < kFinishPer; ++u) {
    const int row = u * kFinishGroups + grp;
    const uint32_t len = s_len[row];
    const int32_t first = __shfl(v[u], 0, kCopyLanes);
    if (len == 0) continue;
    if (len <= (uint32_t)kStage && first != kRowNotParked) {
      const int64_t dst = before + s_off[row] + sub;
      if ((uint32_t)sub < len && dst < A.capacity) A.cols[dst] = v[u];
      parked |= 1u << u;
      longest = len > longest ? len : longest;
    } else if (sub == 0 && !A.qrec &&
               (len <= (uint32_t)kStage || A.qflag[i0 + row] != kQueryNormal)) {
      const unsigned long long slot = atomicAdd(&A.stats[kStatLongRows], 1ull);
      A.long_rows[slot] = (uint32_t)(i0 + row);
    }
  }
  for (uint32_t k0 = kCopyLanes; k0 < longest; k0 += kCopyLanes) {
    const uint32_t k = k0 + sub;
    #pragma unroll
    for (int u = 0; u < kFinishPer; ++u) {
      const int row = u * kFinishGroups + grp;
      const bool take = ((parked >> u) & 1u) != 0u && k < s_len[row];
      v[u] = take ? A.staging[(i0 + row) * kStage + k] : 0;
    }
    #pragma unroll
    for (int u = 0; u < kFinishPer; ++u) {
      const int row = u * kFinishGroups + grp;
      const int64_t dst = before + s_off[row] + k;
      if (((parked >> u) & 1u) != 0u && k < s_len[row] && dst < A.capacity) A.cols[dst] = v[u];
    }
  }
}

// The same over several launches, for more than kFinishOneLaunch queries: the
// scan of the row lengths, the matches, and the rows, sixteen lanes per query.
constexpr int kCopyQueries = kThreads / kCopyLanes;
constexpr int kCopyUnroll = 4;  // rows per group
__global__ __launch_bounds__(kThreads) void k_copy_rows(StabArgs A) {
  static_assert(kCopyLanes <= kStage, "the first piece lies inside the staging slot");
  const int sub = (int)(threadIdx.x & (kCopyLanes - 1));
  // kCopyUnroll consecutive rows per group of kCopyLanes, their loads in flight together
  const int64_t i0 =
      ((int64_t)blockIdx.x * kCopyQueries + (threadIdx.x / kCopyLanes)) * kCopyUnroll;
  if (rows_dropped(A)) return;
  if (i0 >= A.n1) return;  // whole groups of kCopyLanes leave together
  // each slot's first piece is read beside the row offsets (before the row's
  // length is known); its first word tells whether the row was parked
  int32_t v[kCopyUnroll];
  int64_t o0[kCopyUnroll], o1[kCopyUnroll];
  #pragma unroll
  for (int u = 0; u < kCopyUnroll; ++u) {
    const int64_t i = i0 + u;
    const bool in = i < A.n1;
    v[u] = in ? A.staging[i * kStage + sub] : 0;
    o0[u] = in ? A.row_offsets[i] : 0;
    o1[u] = in ? A.row_offsets[i + 1] : 0;
  }
  #pragma unroll
  for (int u = 0; u < kCopyUnroll; ++u) {
    const int64_t i = i0 + u;
    if (i >= A.n1) break;  // uniform in the group
    const int64_t len = o1[u] - o0[u];
    const int32_t first = __shfl(v[u], 0, kCopyLanes);
    if (len <= kStage && (len == 0 || first != kRowNotParked)) {
      if (sub < len && o0[u] + sub < A.capacity) A.cols[o0[u] + sub] = v[u];
      const int32_t* src = A.staging + i * kStage;
      for (int k = sub + kCopyLanes; k < (int)len; k += kCopyLanes)
        if (o0[u] + k < A.capacity) A.cols[o0[u] + k] = src[k];
    } else if (sub == 0 && !A.qrec && (len <= kStage || A.qflag[i] != kQueryNormal)) {
      // long rows of normal queries belong to the wide-row pass of their tile
      const unsigned long long slot = atomicAdd(&A.stats[kStatLongRows], 1ull);
      A.long_rows[slot] = (uint32_t)i;
    }
  }
}

// The fused pass's matches, from its per-query records to the caller's
// arrays (thread per query, all accesses coalesced), unless a later pass
// writes the query's match.
__global__ __launch_bounds__(kThreads) void k_write_matches(StabArgs A) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (rows_dropped(A) || i >= A.n1) return;
  const uint4 r = A.qrec[i];
  if ((int32_t)r.y == kMatchDeferred) return;
  A.best_idx[i] = (int32_t)r.y;
  A.best_dist[i] = __uint_as_float(r.z);
  A.second_dist[i] = __uint_as_float(r.w);
}

// Rebuilds the queued rows (grid-stride over the
// queue, whose length only the device knows).
__global__ __launch_bounds__(kThreads) void k_fill_long(StabArgs A) {
  __shared__ int32_t rowbuf[kWaves][kRowSortMax];
  const int wave = wave_id();
  const uint64_t n = A.stats[kStatLongRows];
  for (uint64_t t = (uint64_t)blockIdx.x * kWaves + wave; t < n;
       t += (uint64_t)gridDim.x * kWaves)
    fill_row(A, (int64_t)A.long_rows[t], rowbuf[wave]);
}

// The queries that the fused passes left over, a wavefront each: rows that are
// not in the CSR yet are rebuilt, then the match is taken from the row.  (As
// two launches, the rebuild took 4.4 us of a call even where there was nothing
// to rebuild.)
__global__ __launch_bounds__(kThreads) void k_finish_listed(StabArgs A, MatchArgs M) {
  __shared__ int32_t rowbuf[kWaves][kRowSortMax];
  __shared__ float4 qdesc[kWaves][32];
  const int wave = wave_id();
  const uint64_t n = A.stats[kStatRest];
  if (n == 0) return;
  const bool fits = !csr_overflow(M);  // an incomplete CSR is completed, not matched
  for (uint64_t t = (uint64_t)blockIdx.x * kWaves + wave; t < n;
       t += (uint64_t)gridDim.x * kWaves) {
    const uint32_t w = A.rest[t];
    const int64_t i = (int64_t)(w & ~kRestRebuild);
    if (w & kRestRebuild) {
      fill_row(A, i, rowbuf[wave]);
      // the row is read back by other lanes of the wavefront
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    if (fits) match_row_f32(M, i, qdesc[wave]);
  }
}

// ------------------------------------------------------------------ scan
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanBlock = kScanThreads * kScanItems;
constexpr int64_t kScanDirectBlocks = 4096;  // up to 8 M counts: no top-level scan launch

__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t* sh, int64_t* total) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {
    const int64_t o = tid >= off ? sh[tid - off] : 0;
    __syncthreads();
    sh[tid] += o;
    __syncthreads();
  }
  const int64_t incl = sh[tid];
  *total = sh[kScanThreads - 1];
  __syncthreads();
  return incl - v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_partials(const uint32_t* __restrict__ counts, int stride,
                                                                int64_t n,
                                                                int64_t* __restrict__ partials) {
  __shared__ int64_t sh[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanBlock;
  int64_t s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t idx = base + (int64_t)k * kScanThreads + threadIdx.x;
    if (idx < n) s += counts[idx * stride];
  }
  int64_t tot;
  block_exclusive_scan(s, sh, &tot);
  if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_top(int64_t* __restrict__ partials,
                                                           int64_t nb) {
  __shared__ int64_t sh[kScanThreads];
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
    const int64_t idx = b0 + threadIdx.x;
    const int64_t v = idx < nb ? partials[idx] : 0;
    int64_t tot;
    const int64_t ex = block_exclusive_scan(v, sh, &tot);
    if (idx < nb) partials[idx] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) partials[nb] = carry;
}

// Sum of partials[0 .. nb) by one workgroup (every thread gets it).
__device__ __forceinline__ int64_t block_sum(const int64_t* __restrict__ partials, int64_t nb,
                                             int64_t* sh) {
  int64_t v = 0;
  for (int64_t k = threadIdx.x; k < nb; k += kScanThreads) v += partials[k];
  int64_t tot;
  block_exclusive_scan(v, sh, &tot);
  return tot;
}

// Final pass without the top-level scan (few blocks): block b adds up the
// partial sums of blocks 0 .. b - 1 itself; the last block writes offsets[n].
__global__ __launch_bounds__(kScanThreads) void k_scan_final_direct(
    const uint32_t* __restrict__ counts, int stride, int64_t n, const int64_t* __restrict__ partials,
    int64_t nb, int64_t* __restrict__ offsets) {
  __shared__ int64_t sh[kScanThreads];
  const int64_t before = block_sum(partials, (int64_t)blockIdx.x, sh);
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  int64_t s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? counts[(base + k) * stride] : 0u;
    s += v[k];
  }
  int64_t tot;
  int64_t run = before + block_exclusive_scan(s, sh, &tot);
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) offsets[base + k] = run;
    run += v[k];
  }
  if (blockIdx.x == nb - 1 && threadIdx.x == 0) offsets[n] = before + tot;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_final(const uint32_t* __restrict__ counts, int stride,
                                                             int64_t n,
                                                             const int64_t* __restrict__ partials,
                                                             int64_t nb,
                                                             int64_t* __restrict__ offsets) {
  __shared__ int64_t sh[kScanThreads];
  // thread t owns items [base + t*kScanItems, +kScanItems): blocked order
  const int64_t base = (int64_t)blockIdx.x * kScanBlock + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  int64_t s = 0;
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? counts[(base + k) * stride] : 0u;
    s += v[k];
  }
  int64_t tot;
  int64_t run = partials[blockIdx.x] + block_exclusive_scan(s, sh, &tot);
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) offsets[base + k] = run;
    run += v[k];
  }
  if (blockIdx.x == nb - 1 && threadIdx.x == 0) offsets[n] = partials[nb];
}

}  // namespace

__global__ __launch_bounds__(256) void k_clear_stats(unsigned long long* stats, uint32_t* sched,
                                                     unsigned long long* match_stats) {
  if (stats && threadIdx.x < kNumStats) stats[threadIdx.x] = 0ull;
  if (match_stats && threadIdx.x < kMatchStatWords) match_stats[threadIdx.x] = 0ull;
  if (sched)
    for (int k = (int)threadIdx.x; k < kSchedWords; k += 256) sched[k] = 0u;
}

hipError_t launch_clear_stats(unsigned long long* stats, hipStream_t s, uint32_t* sched,
                              unsigned long long* match_stats) {
  hipLaunchKernelGGL(k_clear_stats, dim3(1), dim3(256), 0, s, stats, sched, match_stats);
  return hipGetLastError();
}

hipError_t launch_tile_split(const StabArgs& a, float fill, hipStream_t s) {
  if (a.num_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_split, dim3((unsigned)a.num_pairs), dim3(kSplitThreads), 0, s, a, fill);
  return hipGetLastError();
}

hipError_t launch_tile_windows(const StabArgs& a, hipStream_t s) {
  if (a.num_tiles == 0) return hipSuccess;
  const int blocks = (a.num_tiles + kWindowTiles - 1) / kWindowTiles;
  hipLaunchKernelGGL(k_tile_windows, dim3((blocks + kNumXcd - 1) / kNumXcd * kNumXcd),
                     dim3(kWindowThreads), 0, s, a);
  return hipGetLastError();
}

namespace {

template <int MODE, int CH>
void launch_stab_mode(const StabArgs& a, int grid, const dim3& g, hipStream_t s) {
  if (grid > 0)
    hipLaunchKernelGGL((k_stab_tile<true, MODE, CH>), g, dim3(kThreads), 0, s, a);
  else
    hipLaunchKernelGGL((k_stab_tile<false, MODE, CH>), g, dim3(kThreads), 0, s, a);
}

template <int CH>
hipError_t launch_stab_chunk(const StabArgs& a, int grid, int mode, const dim3& g,
                             hipStream_t s) {
  switch (mode) {
    case kStabCount: launch_stab_mode<kStabCount, CH>(a, grid, g, s); break;
    case kStabF32: launch_stab_mode<kStabF32, CH>(a, grid, g, s); break;
    case kStabBF16: launch_stab_mode<kStabBF16, CH>(a, grid, g, s); break;
    case kStabFP8: launch_stab_mode<kStabFP8, CH>(a, grid, g, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_stab_tiles(const StabArgs& a, int grid, int mode, int chunk, hipStream_t s) {
  if (a.num_tiles == 0) return hipSuccess;
  if (grid > 0 && !a.queue) return hipErrorInvalidValue;
  if (mode != kStabCount && (!a.desc1 || !a.desc2 || !a.best_idx || !a.best_dist ||
                             !a.second_dist || !a.rest || (!a.qrec && mode != kCsrBF16)))
    return hipErrorInvalidValue;
  if ((mode == kStabBF16 || mode == kCsrBF16) && (!a.codes1 || !a.codes2))
    return hipErrorInvalidValue;
  if (mode == kCsrBF16) {
    if (!a.rest_count || !a.tile_wide || !a.row_offsets) return hipErrorInvalidValue;
    launch_stab_mode<kCsrBF16, 256>(
        a, grid, dim3(grid > 0 && grid < a.num_tiles ? grid : a.num_tiles), s);
    return hipGetLastError();
  }
  // (FP8: the image-2 pointers are read only through window records, so they
  // may be NULL when image 2 is empty; the entry point checks them otherwise)
  const dim3 g(grid > 0 ? (grid < a.num_tiles ? grid : a.num_tiles) : a.num_tiles);
  // default: 256 records for the BF16 and FP8 passes (their LDS then allows
  // four workgroups per CU), kChunk otherwise
  if (chunk == 0) chunk = mode == kStabBF16 || mode == kStabFP8 ? 256 : kChunk;
  switch (chunk) {
    case 256: return launch_stab_chunk<256>(a, grid, mode, g, s);
    case 512: return launch_stab_chunk<512>(a, grid, mode, g, s);
    case 1024: return launch_stab_chunk<1024>(a, grid, mode, g, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_fill_long(const StabArgs& a, hipStream_t s) {
  if (a.n1 == 0) return hipSuccess;
  const int64_t blocks = (a.n1 + kWaves - 1) / kWaves;
  // long rows are few and each is latency-bound: up to 2048 workgroups
  // (8192 wavefronts) take them from the queue
  const int64_t lblocks = blocks < 2048 ? blocks : 2048;
  hipLaunchKernelGGL(k_fill_long, dim3((unsigned)lblocks), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_finish_listed(const StabArgs& a, const MatchArgs& m, hipStream_t s) {
  if (a.n1 == 0) return hipSuccess;
  // as many workgroups as fit with their row buffers, and no more than queries
  const int64_t blocks = (a.n1 + kWaves - 1) / kWaves;
  hipLaunchKernelGGL(k_finish_listed, dim3((unsigned)(blocks < 1024 ? blocks : 1024)),
                     dim3(kThreads), 0, s, a, m);
  return hipGetLastError();
}

int64_t scan_partials_count(int64_t n) { return (n + kScanBlock - 1) / kScanBlock + 1; }

hipError_t launch_scan_counts(const uint32_t* counts, int stride, int64_t n, int64_t* offsets,
                              int64_t* partials, hipStream_t s) {
  if (n == 0) {
    // offsets[0] = 0 is written by the caller
    return hipSuccess;
  }
  const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
  hipLaunchKernelGGL(k_scan_partials, dim3((unsigned)nb), dim3(kScanThreads), 0, s, counts, stride,
                     n, partials);
  if (nb <= kScanDirectBlocks) {  // every block sums the partials before it
    hipLaunchKernelGGL(k_scan_final_direct, dim3((unsigned)nb), dim3(kScanThreads), 0, s, counts,
                       stride, n, partials, nb, offsets);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kScanThreads), 0, s, partials, nb);
  hipLaunchKernelGGL(k_scan_final, dim3((unsigned)nb), dim3(kScanThreads), 0, s, counts, stride,
                     n, partials, nb, offsets);
  return hipGetLastError();
}

int64_t finish_state_words(int64_t n1) { return (n1 + kFinishRows - 1) / kFinishRows; }

hipError_t launch_finish_rows(const StabArgs& a, int64_t* partials, int64_t* offsets,
                              hipStream_t s) {
  if (a.n1 == 0) return hipSuccess;
  if (!a.row_sums || !partials || !offsets || !a.stats || !a.staging || (a.capacity > 0 && !a.cols))
    return hipErrorInvalidValue;
  if (a.n1 <= kFinishOneLaunch) {
    hipLaunchKernelGGL(k_finish_rows, dim3((unsigned)finish_state_words(a.n1)),
                       dim3(kFinishThreads), 0, s, a, offsets);
    return hipGetLastError();
  }
  const hipError_t e =
      a.qrec ? launch_scan_counts(reinterpret_cast<const uint32_t*>(a.qrec), 4, a.n1, offsets,
                                  partials, s)
             : launch_scan_counts(a.counts, 1, a.n1, offsets, partials, s);
  if (e != hipSuccess) return e;
  if (a.qrec)
    hipLaunchKernelGGL(k_write_matches, dim3((unsigned)((a.n1 + kThreads - 1) / kThreads)),
                       dim3(kThreads), 0, s, a);
  const int64_t rows_per_block = (int64_t)kCopyQueries * kCopyUnroll;
  hipLaunchKernelGGL(k_copy_rows, dim3((unsigned)((a.n1 + rows_per_block - 1) / rows_per_block)),
                     dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace epm
