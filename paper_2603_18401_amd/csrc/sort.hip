// Segmented, stable LSD radix sort of (key, index) pairs, 11 bits per pass.
//
// Builds the angle-sorted interval layout that replaces the paper's centred
// segment tree (Sec. 4.4): every pair's records are one segment.  Each
// segment is cut into tiles that never straddle two segments.  The records'
// 22-bit keys take two passes, the second of which writes the records in
// their final order; the queries, which are only grouped by angle, one pass
// over the upper 11 bits (two in very large segments).
//
// A pass is one launch, a workgroup of 1024 threads per tile.  It adds up the
// digit counts of its segment's tiles (rows of 2048 16-bit counts, left by the
// kernel that wrote the keys or by k_sort_hist), scans them over the digits,
// and ranks its own elements with wavefront ballots.  What bounds it is
// latency: the rows, read with kRowsInFlight loads in flight, are a few
// microseconds in segments of 60 tiles, the rest is the launch itself.  Three
// 8-bit passes of 512-element tiles and a gather for the records and two for
// the queries took 52 us for six pairs of 20000 keypoints, 65 us for one of
// 60000 and 322 us for 3.7 M records and 3.6 M queries; the passes here take
// 33, 37 and 222 us.
// Workgroups take their tiles through xcd_tile: groups of consecutive tiles
// run on one XCD, so what neighbouring tiles of a segment write side by side
// in every bucket meets in one L2 before it is written back.
#include "device_common.h"
#include "launch.h"

namespace epm {

namespace {

constexpr int kSortWaves = kSortThreads / kWave;
constexpr int kRowsInFlight = 32;
static_assert(kSortThreads == kHistWords, "two digits per thread");
static_assert(kSortTileMin == kSortThreads, "one element per thread and round");
static_assert(kSortTileMax < 65536, "16-bit counts");

// Digit counts of every tile's keys for the second pass.  (Counted by the
// first pass as it writes, with global atomics, they cost 9 us more there for
// 120000 records: the second pass's digits crowd into few words.  This launch
// costs 3 to 5.)
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const uint32_t* __restrict__ keys,
                                                            const SortTile* __restrict__ tiles,
                                                            const SortSeg* __restrict__ segs,
                                                            int shift,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kRadix];
  const int tid = threadIdx.x;
  const int tb = xcd_tile((int)blockIdx.x, (int)gridDim.x);  // this workgroup's tile
  const SortTile t = tiles[tb];
  const SortSeg sg = segs[t.seg];
  if (sg.tile_count < 2) return;  // uniform
  h[2 * tid] = h[2 * tid + 1] = 0u;
  __syncthreads();
  for (int k = tid; k < t.count; k += kSortThreads)
    atomicAdd(&h[(keys[t.begin + k] >> shift) & (kRadix - 1)], 1u);
  __syncthreads();
  hist[(int64_t)(sg.hist_begin + tb - sg.tile_begin) * kHistWords + tid] =
      h[2 * tid] | (h[2 * tid + 1] << 16);
}

// The tile lists of the record sort, the query sort and the stabbing pass,
// filled on the device from the per-pair tables (segments, query slice starts
// and the first stabbing tile of each pair), so that only those go up from
// the host; the host only counts them.  One thread per tile: its segment (or
// pair) is the last one whose first tile is not after it, which skips empty
// ones.  rsize, qsize: elements per sort tile.
__global__ __launch_bounds__(256) void k_expand_tiles(
    const SortSeg* __restrict__ rsegs, const SortSeg* __restrict__ qsegs,
    const int64_t* __restrict__ qstart, const int32_t* __restrict__ stile_begin, int num_pairs,
    SortTile* __restrict__ rtiles, int64_t tr, int rsize, SortTile* __restrict__ qtiles,
    int64_t tq, int qsize, StabTile* __restrict__ stiles, int64_t ts) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g < tr + tq) {
    const bool rec = g < tr;
    const SortSeg* segs = rec ? rsegs : qsegs;
    const int64_t t = rec ? g : g - tr;
    const int size = rec ? rsize : qsize;
    int lo = 0, hi = num_pairs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((int64_t)segs[mid].tile_begin <= t) lo = mid;
      else hi = mid - 1;
    }
    const SortSeg sg = segs[lo];
    const int64_t o = (t - sg.tile_begin) * size;
    SortTile st;
    st.begin = sg.begin + o;
    st.count = (int32_t)(sg.count - o < size ? sg.count - o : size);
    st.seg = lo;
    (rec ? rtiles : qtiles)[t] = st;
  } else if (g < tr + tq + ts) {
    const int64_t t = g - tr - tq;
    int lo = 0, hi = num_pairs - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if ((int64_t)stile_begin[mid] <= t) lo = mid;
      else hi = mid - 1;
    }
    const int64_t m = qstart[lo + 1] - qstart[lo];
    const int64_t o = (t - stile_begin[lo]) * kTileQ;
    StabTile st;
    st.begin = qstart[lo] + o;
    st.count = (int32_t)(m - o < kTileQ ? m - o : kTileQ);
    st.pair = lo;
    stiles[t] = st;
  }
}

// Exclusive scan over the workgroup's threads, one value each; ends with
// wsum free for the next one only after a further barrier.
// (By DPP, the wavefronts' sums too: with shuffles and a loop over the sums the
// three passes of one pair of 1000 keypoints took 15.4 us, so 13.4; 237 and 219
// at 512 pairs.)
__device__ __forceinline__ uint32_t scan_threads(uint32_t v, uint32_t* wsum) {
  const int lane = lane_id(), wave = wave_id();
  const uint32_t incl = wave_scan_u32(v);
  if (lane == kWave - 1) wsum[wave] = incl;
  __syncthreads();
  // every wavefront scans the wavefronts' sums
  const uint32_t sums = lane < kSortWaves ? wsum[lane] : 0u;
  const uint32_t before = wave_scan_u32(sums) - sums;
  return incl - v + (uint32_t)__builtin_amdgcn_readlane((int)before, __builtin_amdgcn_readfirstlane(wave));
}

// What a pass writes: (key, index) pairs for the next pass, the indices alone
// (the queries' order), or the records.
constexpr int kOutPairs = 0, kOutIndex = 1, kOutRecords = 2;

// One pass.  vin NULL: an element's index is its place.  hist: the tiles'
// digit counts of this pass.  The records are brought into the tile's order
// by digit in LDS first, so that the lanes of a wavefront write runs of
// neighbouring places: the second pass's digits are few and its runs long.
template <int OUT>
__global__ __launch_bounds__(kSortThreads) void k_sort_pass(
    const uint32_t* __restrict__ kin, const uint32_t* __restrict__ vin,
    uint32_t* __restrict__ kout, uint32_t* __restrict__ vout, const SortTile* __restrict__ tiles,
    const SortSeg* __restrict__ segs, int num_segs, int shift, const uint32_t* __restrict__ hist,
    RecordSort R, uint32_t* __restrict__ group_starts, uint32_t* __restrict__ groups) {
  constexpr bool REC = OUT == kOutRecords;
  __shared__ uint32_t run[kRadix];  // the digits' next places
  __shared__ uint32_t wsum[kSortWaves], wmost[OUT == kOutIndex ? kSortWaves : 1];
  __shared__ __attribute__((aligned(16))) uint8_t wcnt[kSortWaves][kRadix];
  // the round in the order of its digits: starts of the digits, elements
  __shared__ uint16_t local[REC ? kRadix : 1];
  __shared__ uint32_t s_key[REC ? kSortThreads : 1], s_val[REC ? kSortThreads : 1],
      s_pos[REC ? kSortThreads : 1];
  const int tid = threadIdx.x, wave = wave_id();
  const int tb = xcd_tile((int)blockIdx.x, (int)gridDim.x);
  const SortTile t = tiles[tb];
  const SortSeg sg = segs[t.seg];
  const int mine = tb - sg.tile_begin;
  // the first round's elements, loaded while the places are worked out
  uint32_t key = 0u, val = 0u;
  const auto load = [&](int idx) {
    if (idx >= t.count) return;
    key = kin[t.begin + idx];
    val = vin ? vin[t.begin + idx] : (uint32_t)(t.begin + idx);
  };
  load(tid);
  // digits 2 tid and 2 tid + 1: count in the segment's earlier tiles, and in
  // all of them
  uint32_t before[2] = {0u, 0u}, total[2] = {0u, 0u};
  if (sg.tile_count < 2) {
    run[2 * tid] = run[2 * tid + 1] = 0u;
    __syncthreads();
    for (int idx = tid; idx < t.count; idx += kSortThreads)
      atomicAdd(&run[(kin[t.begin + idx] >> shift) & (kRadix - 1)], 1u);
    __syncthreads();
    total[0] = run[2 * tid];
    total[1] = run[2 * tid + 1];
  } else {
    const uint32_t* rows = hist + (int64_t)sg.hist_begin * kHistWords + tid;
    for (int r0 = 0; r0 < sg.tile_count; r0 += kRowsInFlight) {
      uint32_t c[kRowsInFlight];
      #pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u)
        c[u] = r0 + u < sg.tile_count ? rows[(int64_t)(r0 + u) * kHistWords] : 0u;
      #pragma unroll
      for (int u = 0; u < kRowsInFlight; ++u) {
        const uint32_t lo = c[u] & 0xFFFFu, hi = c[u] >> 16;
        total[0] += lo;
        total[1] += hi;
        before[0] += r0 + u < mine ? lo : 0u;
        before[1] += r0 + u < mine ? hi : 0u;
      }
    }
  }
  const uint32_t start = (uint32_t)sg.begin + scan_threads(total[0] + total[1], wsum);
  run[2 * tid] = start + before[0];
  run[2 * tid + 1] = start + total[0] + before[1];
  if constexpr (OUT == kOutIndex) {
    const uint32_t most = wave_max_u32(max(total[0], total[1]));
    if (lane_id() == 0) wmost[wave] = most;  // read at the end
  }
  if constexpr (REC) {
    // the start of width class c: of digit c << (kRadixBits - kClassBits)
    constexpr int kStep = 1 << (kRadixBits - kClassBits);
    static_assert(kStep % 2 == 0, "a class starts at a thread's first digit");
    int64_t* cb = R.class_begin + (int64_t)t.seg * kClassSlots;
    if (mine == 0 && 2 * tid % kStep == 0) cb[2 * tid / kStep] = start;
    if (mine == 0 && tid == 0) cb[kNumClasses] = sg.begin + sg.count;
    // segments without elements have no tile: the first workgroup writes theirs
    if (blockIdx.x == 0) {
      for (int g = tid; g < num_segs; g += kSortThreads)
        if (segs[g].count == 0)
          for (int c = 0; c < kClassSlots; ++c)
            R.class_begin[(int64_t)g * kClassSlots + c] = segs[g].begin;
    }
  }
  for (int base = 0; base < t.count; base += kSortThreads) {
    if (base > 0) load(base + tid);
    const bool valid = base + tid < t.count;
    const uint32_t d = (key >> shift) & (kRadix - 1);
    uint64_t same = ballot(valid);  // lanes of the wavefront with the same digit
    #pragma unroll
    for (int b = 0; b < kRadixBits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t m = ballot(valid && bit);
      same &= bit ? m : ~m;
    }
    const uint32_t rank = lanes_below(same);
    {
      uint4* z = reinterpret_cast<uint4*>(&wcnt[0][0]);
      #pragma unroll
      for (int k = 0; k < kSortWaves * kRadix / 16 / kSortThreads; ++k)
        z[k * kSortThreads + tid] = make_uint4(0u, 0u, 0u, 0u);
    }
    __syncthreads();
    if (valid && rank == 0) wcnt[wave][d] = (uint8_t)__popcll(same);
    __syncthreads();
    uint32_t ahead = rank;  // of the round's elements with this digit
    if (valid) {
      #pragma unroll 4
      for (int w = 0; w < wave; ++w) ahead += wcnt[w][d];
    }
    uint32_t own[2] = {0u, 0u};  // of digits 2 tid, 2 tid + 1 in the round
    const bool more = base + kSortThreads < t.count;
    if (REC || more) {
      #pragma unroll
      for (int w = 0; w < kSortWaves; ++w) {
        const uint32_t two = *reinterpret_cast<const uint16_t*>(&wcnt[w][2 * tid]);
        own[0] += two & 0xFFu;
        own[1] += two >> 8;
      }
    }
    if constexpr (REC) {
      const uint32_t at = scan_threads(own[0] + own[1], wsum);
      local[2 * tid] = (uint16_t)at;
      local[2 * tid + 1] = (uint16_t)(at + own[0]);
      __syncthreads();
      if (valid) {
        const uint32_t k = local[d] + ahead;
        s_key[k] = key;
        s_val[k] = val;
        s_pos[k] = run[d] + ahead;
      }
      __syncthreads();
      if (valid) {  // as many elements as valid threads, from thread 0 on
        const uint32_t r = s_val[tid], pos = s_pos[tid];
        const uint32_t C = R.recC[r], H = R.recH[r];
        const float2 xy = make_float2(R.kp2[2 * (int64_t)r], R.kp2[2 * (int64_t)r + 1]);
        const float eps = R.eps2 ? R.eps2[r] : R.eps_scalar;
        kout[pos] = s_key[tid];
        R.rC[pos] = C;
        R.rH[pos] = H;
        R.rj[pos] = (int32_t)((int64_t)r - sg.begin);
        R.rxy[pos] = xy;
        R.reps[pos] = eps;
        R.rinv[r] = pos;
      }
    } else if (valid) {
      const uint32_t pos = run[d] + ahead;
      if constexpr (OUT == kOutPairs) kout[pos] = key;
      vout[pos] = val;
    }
    if (more) {
      __syncthreads();
      run[2 * tid] += own[0];
      run[2 * tid + 1] += own[1];
      __syncthreads();
    }
  }
  if constexpr (OUT == kOutIndex) {
    // The first tile's workgroup tells the window pass about large groups.
    // (Here, behind a round's barriers: with reductions of its own before the
    // rounds the pass took 1 us more.)
    if (groups && mine == 0) {
      uint32_t most = 0u;
      #pragma unroll
      for (int w = 0; w < kSortWaves; ++w) most = max(most, wmost[w]);
      const uint32_t tile = (uint32_t)sg.tile;
      const bool large = most > 2u * tile, some = most > tile || tile < (uint32_t)kTileQ;
      if (tid == 0) groups[t.seg] = large ? kGroupsLarge : some ? kGroupsLocal : kGroupsSmall;
      if (large && sg.tile_count >= 2) {
        static_assert(2 * kHistWords == kRadix, "two rows of counts hold the starts");
        uint32_t* g = group_starts + (int64_t)sg.hist_begin * kHistWords;
        g[2 * tid] = start;
        g[2 * tid + 1] = start + total[0];
      }
    }
  }
}

// The first of two passes, and the counts of the second.
void first_pass(const SortCall& c, hipStream_t s) {
  const dim3 g((unsigned)c.num_tiles), b(kSortThreads);
  hipLaunchKernelGGL((k_sort_pass<kOutPairs>), g, b, 0, s, c.k0, (const uint32_t*)nullptr, c.k1,
                     c.v1, c.tiles, c.segs, c.num_segs, 0, c.hist0, RecordSort{}, (uint32_t*)nullptr,
                     (uint32_t*)nullptr);
  if (c.rows > 0)
    hipLaunchKernelGGL(k_sort_hist, g, b, 0, s, c.k1, c.tiles, c.segs, kRadixBits, c.hist1);
}

}  // namespace

int sort_tile_size(int64_t largest_segment) {
  // up to 128 rows of counts per tile, as far as 16-bit counts allow
  int size = kSortTileMin;
  while (size < kSortTileMax && largest_segment > (int64_t)128 * size) size *= 2;
  return size;
}

hipError_t launch_expand_tiles(const SortSeg* rsegs, const SortSeg* qsegs, const int64_t* qstart,
                               const int32_t* stile_begin, int num_pairs, SortTile* rtiles,
                               int64_t tr, int rsize, SortTile* qtiles, int64_t tq, int qsize,
                               StabTile* stiles, int64_t ts, hipStream_t s) {
  const int64_t n = tr + tq + ts;
  if (n == 0 || num_pairs < 1) return hipSuccess;
  hipLaunchKernelGGL(k_expand_tiles, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rsegs,
                     qsegs, qstart, stile_begin, num_pairs, rtiles, tr, rsize, qtiles, tq, qsize,
                     stiles, ts);
  return hipGetLastError();
}

hipError_t sort_records(const SortCall& c, const RecordSort& r, hipStream_t s) {
  if (c.num_tiles == 0) return hipSuccess;
  first_pass(c, s);
  hipLaunchKernelGGL((k_sort_pass<kOutRecords>), dim3((unsigned)c.num_tiles), dim3(kSortThreads),
                     0, s, c.k1, c.v1, c.k0, (uint32_t*)nullptr, c.tiles, c.segs, c.num_segs,
                     kRadixBits, c.hist1, r, (uint32_t*)nullptr, (uint32_t*)nullptr);
  return hipGetLastError();
}

hipError_t sort_queries(const SortCall& c, bool two_passes, uint32_t* perm, uint32_t* groups,
                        hipStream_t s) {
  if (c.num_tiles == 0) return hipSuccess;
  if (two_passes) first_pass(c, s);
  hipLaunchKernelGGL((k_sort_pass<kOutIndex>), dim3((unsigned)c.num_tiles), dim3(kSortThreads), 0,
                     s, two_passes ? c.k1 : c.k0, two_passes ? c.v1 : (uint32_t*)nullptr,
                     (uint32_t*)nullptr, perm, c.tiles, c.segs, c.num_segs, kRadixBits,
                     two_passes ? c.hist1 : c.hist0, RecordSort{},
                     two_passes ? nullptr : c.hist1, two_passes ? nullptr : groups);
  return hipGetLastError();
}

}  // namespace epm
