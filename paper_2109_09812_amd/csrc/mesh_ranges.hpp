// Vertex ranges and hash buckets of a batch's meshes.
//
// A batch's offsets are device data that no host code has read. What the
// grouping indexes by them (tiles, buckets, element positions) has to stay in
// range whatever they hold, so they are put in order first: mesh b's range
// begins at the largest of the offsets up to b, cut to [0, n], the first
// mesh's at 0, and the last one's ends at n (vertices behind the last offset
// count with the last mesh). Offsets that keep their rules are unchanged.
#pragma once

#include "device_common.hpp"

namespace mrx {

// Offset b of nmesh + 1, cut to the vertices there are.
__host__ __device__ inline uint32_t cut_offset(const int64_t* off, int64_t b, int32_t nmesh, int64_t n) {
  if (b <= 0) return 0u;
  const int64_t x = b < nmesh ? off[b] : n;
  return uint32_t(x < 0 ? 0 : x < n ? x : n);
}

// Hash buckets of a mesh of nb vertices: for one partition pass, as many as
// bring the vertices per bucket down to `target`; for passes by hash digits
// (mesh_bucket) the smallest power of two that does.
__host__ __device__ inline uint32_t mesh_bucket_count(uint32_t nb, int32_t target, bool digits) {
  if (!digits) return (nb + uint32_t(target) - 1u) / uint32_t(target);  // nb < 2^30
  int k = 0;
  while (k < 30 && int64_t(nb >> k) > target) ++k;
  return 1u << k;
}

// ordered[0, nmesh] and mb[b] = (first bucket, buckets, or for hash digits
// buckets - 1) of every mesh, in mesh order. One workgroup, several meshes a
// thread, so that a batch of thousands takes one round of loads and two scans
// (4,096 meshes a thousand at a time took 5 us longer).
constexpr int kMeshBucketBlock = 1024;
template <bool DIGITS>
__global__ __launch_bounds__(kMeshBucketBlock) void k_mesh_buckets(const int64_t* __restrict__ off, int32_t nmesh,
                                                                   int64_t n, int32_t target,
                                                                   int64_t* __restrict__ ordered,
                                                                   uint2* __restrict__ mb) {
  constexpr int WAVES = kMeshBucketBlock / kWave, PER = 6;
  __shared__ uint32_t s_wave[WAVES];
  const int lane = lane_id(), wave = threadIdx.x / kWave;
  uint32_t buckets = 0, reached = 0;  // of the meshes before this round's
  for (int64_t r0 = 0; r0 < nmesh; r0 += kMeshBucketBlock * PER) {
    const int64_t b0 = r0 + threadIdx.x * PER;
    uint32_t cut[PER + 1], most = 0;
#pragma unroll
    for (int i = 0; i <= PER; ++i) cut[i] = b0 + i <= nmesh ? cut_offset(off, b0 + i, nmesh, n) : 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) most = max(most, cut[i]);
    // the largest offset of the threads before
    uint32_t inc = most;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t t = __shfl_up(inc, o);
      if (lane >= o) inc = max(inc, t);
    }
    if (lane == kWave - 1) s_wave[wave] = inc;
    const uint32_t before = __shfl_up(inc, 1);
    __syncthreads();
    uint32_t at = lane > 0 ? max(reached, before) : reached;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const uint32_t t = s_wave[w];
      if (w < wave) at = max(at, t);
      reached = max(reached, t);
    }
    __syncthreads();  // s_wave is used again
    uint32_t cnt[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      cut[i] = at = max(at, cut[i]);
      cnt[i] = b0 + i < nmesh ? mesh_bucket_count(max(at, cut[i + 1]) - at, target, DIGITS) : 0u;
      sum += cnt[i];
    }
    uint32_t total;
    uint32_t first = buckets + block_exclusive_scan<kMeshBucketBlock>(sum, s_wave, &total);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (b0 + i >= nmesh) break;
      ordered[b0 + i] = cut[i];
      mb[b0 + i] = make_uint2(first, DIGITS ? cnt[i] - 1u : cnt[i]);
      first += cnt[i];
    }
    buckets += total;
  }
  if (threadIdx.x == 0) ordered[nmesh] = n;
}

}  // namespace mrx
