// Plain descriptor matching over the candidate CSR (Sec. 4.3): one wavefront
// per query, one lane per candidate, the candidate's descriptor gathered from
// global memory.  This is the reference GPU path the tiled kernels are
// measured against.
//
// Float distance: canonical FP32 squared L2, t = a_k - b_k then
// acc = fmaf(t, t, acc) for k = 0..127 in order, so every distance is
// bit-reproducible.  Binary distance: popcount of the XOR over 8 words.
// Selection: smallest (distance, j), then the next one; optional ratio test.
#include "device_common.h"
#include "launch.h"
#include "match_common.h"

namespace epm {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;

__global__ __launch_bounds__(kThreads) void k_match_plain_f32(MatchArgs A) {
  __shared__ float4 qdesc[kWaves][32];
  if (csr_overflow(A)) return;
  const int lane = lane_id(), wave = wave_id();
  const int64_t blk = A.xcd_order ? xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x;
  const int64_t qs = blk * kWaves + wave;
  if (qs >= A.n1) return;
  const int64_t i = A.qperm ? (int64_t)A.qperm[qs] : qs;
  const int pair = find_pair(A.qstart, A.num_pairs, i);
  const int64_t kb = A.kstart[pair];
  const float4* d1 = reinterpret_cast<const float4*>(A.desc1) + i * 32;
  if (lane < 32) qdesc[wave][lane] = d1[lane];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int64_t o0 = A.row_offsets[i], o1 = A.row_offsets[i + 1];
  Top2 t;
  for (int64_t e = o0 + lane; e < o1; e += kWave) {
    const int32_t j = A.cols[e];
    const float4* d2 = reinterpret_cast<const float4*>(A.desc2) + (kb + j) * 32;
    float acc = 0.0f;
    #pragma unroll 8
    for (int k = 0; k < 32; ++k) {
      const float4 a = qdesc[wave][k];
      const float4 b = d2[k];
      acc = canonical_step4(acc, a, b);
    }
    t.insert(acc, j);
  }
  t = wave_merge_top2(t);
  if (lane == 0) write_match(A, i, t, false);
}

__global__ __launch_bounds__(kThreads) void k_match_plain_bin256(MatchArgs A) {
  if (csr_overflow(A)) return;
  const int lane = lane_id(), wave = wave_id();
  const int64_t qs = (int64_t)blockIdx.x * kWaves + wave;
  if (qs >= A.n1) return;
  const int64_t i = A.qperm ? (int64_t)A.qperm[qs] : qs;
  const int pair = find_pair(A.qstart, A.num_pairs, i);
  const int64_t kb = A.kstart[pair];
  const uint4* d1 = reinterpret_cast<const uint4*>(A.desc1) + i * 2;
  const uint4 qa = d1[0], qb = d1[1];
  const int64_t o0 = A.row_offsets[i], o1 = A.row_offsets[i + 1];
  Top2 t;
  for (int64_t e = o0 + lane; e < o1; e += kWave) {
    const int32_t j = A.cols[e];
    const uint4* d2 = reinterpret_cast<const uint4*>(A.desc2) + (kb + j) * 2;
    const uint4 ba = d2[0], bb = d2[1];
    const uint32_t h = __popc(qa.x ^ ba.x) + __popc(qa.y ^ ba.y) + __popc(qa.z ^ ba.z) +
                       __popc(qa.w ^ ba.w) + __popc(qb.x ^ bb.x) + __popc(qb.y ^ bb.y) +
                       __popc(qb.z ^ bb.z) + __popc(qb.w ^ bb.w);
    t.insert((float)h, j);
  }
  t = wave_merge_top2(t);
  if (lane == 0) write_match(A, i, t, true);
}

// The same with 16 lanes per query, for calls whose queries fill the chip: a
// row of a few dozen candidates leaves half of a wavefront's lanes idle, and
// what bounds a wavefront is the latency of its dependent loads and of the
// merge, which here goes by DPP.  Two lanes read a candidate's two halves (one
// line, one address slot; 19.4 us with both read by one lane).  A candidate is
// kept as (distance, j) in one 64-bit key.  60000 queries with 66 candidates
// each: 30.0 us with a wavefront per query, 15.9 this way.
//
// Where the line lies, in us per call with a wavefront per query / 16 lanes,
// for rows of 9, 70, 320, 1070 and 4250 candidates:
//    8192 queries  11.0/11.4  11.3/11.6  14.3/12.8  41.3/33.9  139/114
//   16384          11.1/12.0  11.8/11.5  25.9/16.6  74.0/43.0  330/181
//   24576          11.6/12.1  14.8/11.7  36.7/21.1   108/56.0  544/268
//   32768          13.7/11.1  19.0/11.4  47.5/26.8   143/72.4  726/367
//   65536          27.5/11.3  34.2/17.4  89.9/45.1   365/174  1461/700
// From 32768 on the groups win everywhere; below, rows of a few candidates are
// as fast with a wavefront each (the line could lie lower for longer rows).
constexpr int kBinLanes = 16;
constexpr int kBinQueries = kThreads / kBinLanes;
constexpr int64_t kBinGroupMin = 32768;
__global__ __launch_bounds__(kThreads) void k_match_groups_bin256(MatchArgs A) {
  if (csr_overflow(A)) return;
  const int sub = (int)threadIdx.x & (kBinLanes - 1);
  const int64_t qs = (int64_t)blockIdx.x * kBinQueries + threadIdx.x / kBinLanes;
  const bool live = qs < A.n1;
  int64_t i = 0, kb = 0, o0 = 0, o1 = 0;
  const int half = sub & 1;
  uint4 qa = make_uint4(0u, 0u, 0u, 0u);  // this lane's half of the query's bits
  if (live) {
    i = A.qperm ? (int64_t)A.qperm[qs] : qs;
    o0 = A.row_offsets[i];
    o1 = A.row_offsets[i + 1];
    qa = reinterpret_cast<const uint4*>(A.desc1)[i * 2 + half];
    kb = A.kstart[find_pair(A.qstart, A.num_pairs, i)];
  }
  uint64_t best = ~0ull, second = ~0ull;
  constexpr int kFly = 4;  // candidates of a lane whose gathers are in flight together
  for (int64_t e0 = o0 + (sub >> 1); e0 < o1; e0 += kFly * kBinLanes / 2) {
    int32_t j[kFly];
    #pragma unroll
    for (int u = 0; u < kFly; ++u) {
      const int64_t e = e0 + u * (kBinLanes / 2);
      j[u] = A.cols[e < o1 ? e : e0];
    }
    uint4 b[kFly];
    #pragma unroll
    for (int u = 0; u < kFly; ++u)
      b[u] = reinterpret_cast<const uint4*>(A.desc2)[(kb + j[u]) * 2 + half];
    #pragma unroll
    for (int u = 0; u < kFly; ++u) {
      uint32_t h = __popc(qa.x ^ b[u].x) + __popc(qa.y ^ b[u].y) + __popc(qa.z ^ b[u].z) +
                   __popc(qa.w ^ b[u].w);
      h += lane_xor<1>(h);
      const uint64_t key = ((uint64_t)h << 32) | (uint32_t)j[u];
      if (e0 + u * (kBinLanes / 2) < o1) {
        second = key < best ? best : key < second ? key : second;
        best = key < best ? key : best;
      }
    }
  }
  auto merge = [&](uint64_t ob, uint64_t os) {
    const uint64_t lose = ob < best ? best : ob, wins = ob < best ? os : second;
    best = ob < best ? ob : best;
    second = lose < wins ? lose : wins;
  };
  merge(lane_xor<2>(best), lane_xor<2>(second));
  merge(lane_xor<4>(best), lane_xor<4>(second));
  merge(lane_xor<8>(best), lane_xor<8>(second));
  if (live && sub == 0) {
    Top2 t;
    if (best != ~0ull) {
      t.bd = (float)(uint32_t)(best >> 32);
      t.bj = (int32_t)(uint32_t)best;
    }
    if (second != ~0ull) {
      t.sd = (float)(uint32_t)(second >> 32);
      t.sj = (int32_t)(uint32_t)second;
    }
    write_match(A, i, t, true);
  }
}

// Listed queries (the ones the fused stab + match pass left over): one
// wavefront per listed query, grid-stride over a list whose length only the
// device knows.
__global__ __launch_bounds__(kThreads) void k_match_listed_f32(MatchArgs A,
                                                               const uint32_t* __restrict__ list,
                                                               const unsigned long long* __restrict__ count) {
  __shared__ float4 qdesc[kWaves][32];
  if (csr_overflow(A)) return;
  const int lane = lane_id(), wave = wave_id();
  const uint64_t n = *count;
  for (uint64_t t = (uint64_t)blockIdx.x * kWaves + wave; t < n;
       t += (uint64_t)gridDim.x * kWaves) {
    const int64_t i = (int64_t)list[t];
    match_row_f32(A, i, qdesc[wave]);
  }
}

}  // namespace

hipError_t launch_match_listed_f32(const MatchArgs& a, const uint32_t* list,
                                   const unsigned long long* count, int64_t max_count,
                                   hipStream_t s) {
  if (max_count <= 0) return hipSuccess;
  // the list is usually short and its rows latency-bound: enough
  // workgroups that every listed query has its own wavefront up to 16384
  int64_t blocks = (max_count + kWaves - 1) / kWaves;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_match_listed_f32, dim3((unsigned)blocks), dim3(kThreads), 0, s, a, list,
                     count);
  return hipGetLastError();
}

hipError_t launch_match_plain_f32(const MatchArgs& a, hipStream_t s) {
  if (a.n1 == 0) return hipSuccess;
  const int64_t blocks = (a.n1 + kWaves - 1) / kWaves;
  hipLaunchKernelGGL(k_match_plain_f32, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_match_plain_bin256(const MatchArgs& a, hipStream_t s) {
  if (a.n1 == 0) return hipSuccess;
  // (fewer queries: the longest rows end sooner with a wavefront each)
  if (a.n1 >= kBinGroupMin) {
    hipLaunchKernelGGL(k_match_groups_bin256,
                       dim3((unsigned)((a.n1 + kBinQueries - 1) / kBinQueries)), dim3(kThreads), 0,
                       s, a);
    return hipGetLastError();
  }
  const int64_t blocks = (a.n1 + kWaves - 1) / kWaves;
  hipLaunchKernelGGL(k_match_plain_bin256, dim3((unsigned)blocks), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace epm
