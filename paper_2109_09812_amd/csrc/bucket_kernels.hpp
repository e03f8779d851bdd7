// Hash buckets in one partition pass, grouped whole.
//
// For up to some tens of millions of vertices the records go straight into up
// to kBucketMax hash buckets, each grouped by one workgroup. Compared with two
// or three stable 8-bit passes (k_onesweep) and a grouping that rebuilds the
// bucket borders from overlapping windows (k_group), the elements move once
// instead of two or three times, nothing waits on other tiles, and every
// element is hashed into a table once instead of 1.5 times.
//  * k_bucket_count: elements per (tile, bucket), beside Step 1's marking;
//  * k_bucket_offsets: each tile's place in every bucket (a scan down the
//    tiles) and the elements per bucket;
//  * k_bucket_scatter: elements (record, id | used << 31) to their buckets,
//    put in bucket order in LDS first so that runs are written together;
//  * k_group_bucket: equal records of a bucket by a hash table in LDS;
//  * k_group_over: the same for buckets that k_group leaves (digit path).
// Measured (MI355X), 26.4M 12-byte vertices of a soup: offsets 0.035, scatter
// 0.235 (3.3 TB/s, bound by runs of three elements per tile and bucket) and
// grouping 0.239 ms (3.0 TB/s, phases of memory and LDS work of two workgroups
// a CU), where two stable passes and k_group took 0.21 + 0.24 and 0.27 ms; 15M
// in 256 meshes 0.010 + 0.196 + 0.185 ms, the whole call 1.65 -> 1.23 ms.
// The order inside a bucket is that of atomics, so a group's representative is
// the minimum of its ids. Only a bucket's distinct records take LDS; where they
// do not fit, they take rounds by shares of their hash, and a bucket of many
// copies is grouped in parts by several workgroups.
#pragma once

#include <algorithm>

#include "band_kernels.hpp"
#include "group_kernels.hpp"
#include "scan_kernels.hpp"

namespace mrx {

constexpr int kBucketBlock = 512;
// Buckets: the tables of k_bucket_scatter, 15 or 36 KB of LDS beside the
// stage, leave room for two workgroups on a CU.
constexpr int kBucketMax = 2560;      // one mesh
constexpr int kBucketMaxMesh = 6144;  // batches: at least one per mesh
// Vertices per bucket, beyond which the digit path takes over. Buckets win
// where the records have copies and lose, the more the larger they are (a
// share of a bucket's distinct records is read with all the others), where
// they do not. 12-byte records, ms by buckets and by digits with six, two and
// one copy of each: 26M (10,156 a bucket) 1.40 and 1.64, 2.34 and 2.20, 3.38
// and 2.88; 31M (12,110) 1.65 and 1.90, 2.78 and 2.56, 4.16 and 3.44; 16M
// (6,250) 0.88 and 1.02, 1.18 and 1.26, 1.98 and 1.77. The line lies where the
// loss without copies reaches a sixth, about the gain of six.
constexpr int kBucketMostPer = 10400;
constexpr int kGroupBlock = 1024;     // k_group_bucket
constexpr int kGroupBlockSmall = 256; // where buckets are aimed to be small

template <int K>
struct BucketShape {
  static constexpr int S = K + 1;
  // elements per thread of a large tile (registers) and of a small one
  static constexpr int EPT = K <= 4 ? 16 : K <= 8 ? 8 : 4;
  static constexpr int EPT_SMALL = 4;
  // slots of the LDS stage (24 KB)
  static constexpr int STAGE = 6144 / S / 64 * 64;
  // distinct records a workgroup of k_group_bucket holds (two workgroups per CU)
  static constexpr int DCAP = K == 1 ? 4096 : K <= 4 ? 3072 : K == 5 ? 2560 : K == 6 ? 2048 : K <= 10 ? 1536
                              : 1024;
  static_assert(DCAP % 32 == 0, "bits of the used groups");
  // the same for buckets of a few hundred elements: eight small workgroups
  // on a CU
  static constexpr int DCAP_SMALL = K <= 8 ? 1024 : 512;
  // average bucket: all distinct records of it fit at once
  static constexpr int TARGET = DCAP * 3 / 4;
};

// Buckets and tiles for n vertices in nmesh meshes with m index entries;
// buckets = 0: too many vertices or meshes, or too few entries.
struct BucketPlan {
  int32_t buckets = 0;   // columns (a batch may use fewer)
  int32_t target = 0;    // vertices per bucket aimed at
  int32_t ept = 0;       // elements per thread of a tile
  int64_t tiles = 0;
  int64_t count_words() const { return tiles * ((buckets + 1) / 2); }   // 16-bit counts
  int64_t base_words() const { return tiles * int64_t(buckets); }
};

template <int K>
inline BucketPlan bucket_plan(int64_t n, int64_t m, int32_t nmesh, int64_t words) {
  using SH = BucketShape<K>;
  BucketPlan p;
  const int64_t most = nmesh > 1 ? int64_t(kBucketMaxMesh) - nmesh : int64_t(kBucketMax);
  if (n <= 0 || most < 512) return p;
  // about 1,024 buckets where that leaves them small, then as large as fits
  // one round, then as large as the limit on buckets makes them
  int64_t t = std::max<int64_t>(256, std::min<int64_t>(nmesh > 1 ? n / 2048 : n / 1024, SH::TARGET));
  t = std::max(t, (n + most - 1) / most);
  if (t > kBucketMostPer) return p;
  // Where few entries name few values, the grouping is nearly all there is to
  // do. Were the records distinct, such buckets would take four rounds and
  // more, each over all of a bucket, where the digit path groups in one: 26M
  // distinct 12-byte records 1.95 ms by buckets and 1.54 by digits, six copies
  // of each 1.27 and 1.41. Few used of many is a part cut out of a mesh that is
  // indexed already far more often than one out of a soup.
  if (t > 3 * SH::DCAP && m < n / 8) return p;
  p.target = int32_t(t);
  p.buckets = int32_t((n + t - 1) / t + (nmesh > 1 ? nmesh : 0));
  // small tiles while the large ones would not fill the GPU twice
  for (int ept : {int(SH::EPT_SMALL), int(SH::EPT)}) {
    if (ept != SH::EPT && n > int64_t(kBucketBlock) * SH::EPT * 128) continue;
    p.ept = ept;
    p.tiles = (n + kBucketBlock * ept - 1) / (kBucketBlock * ept);
    if (p.count_words() + p.base_words() <= words) return p;
  }
  return BucketPlan{};
}

struct BucketArgs {
  const uint32_t* vtx;         // [n][K]
  const uint8_t* used;         // [n]
  int64_t n;
  int32_t buckets;
  int64_t tiles;
  int32_t tile;                // elements per tile
  uint16_t* counts;            // [tiles][stride]
  int32_t stride;              // even
  uint32_t* base;              // [tiles][buckets]
  uint32_t* totals;            // [buckets]
  uint32_t* starts;            // [buckets + 1]
  uint32_t* elems;             // [n][K+1]
  uint32_t most;               // a bucket of more elements is large
  uint32_t* large;             // zeroed; set where there is one
  // batches: vertex offsets, their bucket table, and each mesh's (first
  // bucket, buckets)
  const int64_t* mesh_off;
  const int32_t* mesh_tab;
  const uint2* mesh_buckets;
  int32_t nmesh;
};

// Bucket of a record: the hash scaled to the number of buckets (of its mesh).
__device__ __forceinline__ uint32_t scaled_bucket(uint32_t h, uint32_t buckets) { return __umulhi(h, buckets); }

// What is the same for a whole tile [i0, i1): the meshes of its first and last
// vertex and the buckets it can reach, [first, first + count): those of its
// meshes, a few of a batch's thousands, and only these columns of the count
// tables are written and read.
struct TileMesh {
  uint32_t lo, hi;
  uint2 buckets;  // of mesh lo
  int32_t first, count;
};
template <bool MESH>
__device__ __forceinline__ TileMesh tile_mesh(const BucketArgs& a, int64_t i0, int64_t i1) {
  TileMesh t{};
  t.count = a.buckets;
  if constexpr (MESH) {
    t.lo = __builtin_amdgcn_readfirstlane(mesh_of(a.mesh_off, a.nmesh, i0, a.mesh_tab));
    t.hi = __builtin_amdgcn_readfirstlane(mesh_of(a.mesh_off, a.nmesh, i1 - 1, a.mesh_tab));
    t.buckets = a.mesh_buckets[t.lo];
    const uint2 z = a.mesh_buckets[t.hi];
    t.first = int32_t(t.buckets.x);
    t.count = min(int32_t(z.x + z.y), a.buckets) - t.first;
  }
  return t;
}

template <int K, bool MESH>
__device__ __forceinline__ uint32_t bucket_of(const BucketArgs& a, const TileMesh& tm, int64_t i,
                                              const uint32_t (&x)[K]) {
  const uint32_t h = hash_words<K>(x);
  if constexpr (MESH) {
    const uint2 b = tm.lo == tm.hi ? tm.buckets : a.mesh_buckets[mesh_of(a.mesh_off, a.nmesh, i, a.mesh_tab)];
    return b.x + scaled_bucket(h, b.y);
  } else {
    return scaled_bucket(h, uint32_t(a.buckets));
  }
}

// Elements per bucket of one tile; s_cnt holds a.buckets words (a record's
// bucket lies in its mesh's range, so within the tile's).
template <int K, bool MESH, int BLOCK>
__device__ __forceinline__ void bucket_count_tile(const BucketArgs& a, int64_t tile, uint32_t* s_cnt) {
  constexpr int U = K <= 4 ? 8 : K <= 8 ? 4 : 2;
  const int tid = threadIdx.x;
  const int64_t i0 = tile * a.tile, i1 = min(i0 + a.tile, a.n);
  const TileMesh tm = tile_mesh<MESH>(a, i0, i1);
  for (int f = tid; f < tm.count; f += BLOCK) s_cnt[f] = 0;
  __syncthreads();
  for (int64_t j0 = i0; j0 < i1; j0 += BLOCK * U) {
    uint32_t x[U][K];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = min(j0 + r * BLOCK + tid, i1 - 1);
#pragma unroll
      for (int w = 0; w < K; ++w) x[r][w] = a.vtx[i * K + w];
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t i = j0 + r * BLOCK + tid;
      if (i < i1) atomicAdd(&s_cnt[bucket_of<K, MESH>(a, tm, i, x[r]) - tm.first], 1u);
    }
  }
  __syncthreads();
  uint16_t* row = a.counts + tile * int64_t(a.stride) + tm.first;
  for (int f = tid; f < tm.count; f += BLOCK) row[f] = uint16_t(s_cnt[f]);
}

// Step 1's marking and the bucket counts in one launch, their workgroups
// spread evenly over the grid (as in k_mark_histogram): MARK 0 counts alone,
// 1 marks by scattered stores, 2 by vertex bands.
template <int K, bool MESH, int MARK>
__global__ __launch_bounds__(kRandBlock) void k_bucket_count(BucketArgs a, MarkArgs ma, BandArgs ba,
                                                             int64_t mark_blocks) {
  __shared__ uint32_t s_cnt[MESH ? kBucketMaxMesh : kBucketMax];
  const int64_t total = a.tiles + mark_blocks;
  const int64_t b = die_tile(blockIdx.x, total);  // neighbouring bands on one die, see k_band_map
  if (b < 0) return;
  const int64_t c0 = b * a.tiles / total, c1 = (b + 1) * a.tiles / total;
  if (c1 > c0) {
    bucket_count_tile<K, MESH, kRandBlock>(a, c0, s_cnt);
  } else if constexpr (MARK == 1) {
    mark_used_tile<MESH>(ma, b - c0);
  } else if constexpr (MARK == 2) {
    __shared__ BandWalk<kRandBlock> s_walk;
    extern __shared__ uint32_t s_bits[];
    band_mark_body<kRandBlock>(ba, b - c0, s_bits, s_walk);
  }
}

// Scan down the tiles, 32 buckets per workgroup, 32 runs of tiles. (The bucket
// starts are left to the readers of the totals: a last workgroup that scans
// them needs device-wide fences, which took longer than all else here.)
constexpr int kOffsetCols = 32;
constexpr int kOffsetRuns = 32;
template <bool MESH>
__global__ __launch_bounds__(kOffsetCols* kOffsetRuns) void k_bucket_offsets(BucketArgs a) {
  constexpr int U = 16;  // tiles in flight per thread
  __shared__ uint32_t s_sum[kOffsetRuns][kOffsetCols];
  const int tid = threadIdx.x, c = tid % kOffsetCols, run = tid / kOffsetCols;
  const int f = min(int(blockIdx.x) * kOffsetCols + c, a.buckets - 1);
  const bool own = int(blockIdx.x) * kOffsetCols + c < a.buckets;
  const uint16_t* __restrict__ counts = a.counts + f;
  uint32_t* __restrict__ base = a.base + f;
  const int tiles = int(a.tiles), stride = a.stride;
  int first = 0, end = tiles;  // tiles that reach bucket f
  if constexpr (MESH) {
    int lo = 0, hi = a.nmesh - 1;  // last mesh whose buckets start at or before f
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (int(a.mesh_buckets[mid].x) <= f) lo = mid; else hi = mid - 1;
    }
    const uint2 b = a.mesh_buckets[lo];
    const bool in = f < int(b.x + b.y);  // the last columns may belong to no mesh
    first = in ? int(a.mesh_off[lo] / a.tile) : 0;
    end = in ? int((a.mesh_off[lo + 1] + a.tile - 1) / a.tile) : 0;
  }
  const int per = (end - first + kOffsetRuns - 1) / kOffsetRuns;
  const int t0 = min(first + run * per, end), t1 = min(t0 + per, end);
  uint32_t sum = 0;
  for (int t = t0; t < t1; t += U) {
    uint32_t x[U];
#pragma unroll
    for (int j = 0; j < U; ++j) x[j] = counts[int64_t(min(t + j, tiles - 1)) * stride];
#pragma unroll
    for (int j = 0; j < U; ++j) sum += t + j < t1 ? x[j] : 0u;
  }
  s_sum[run][c] = sum;
  __syncthreads();
  uint32_t at = 0;
  for (int r = 0; r < run; ++r) at += s_sum[r][c];
  if (own && run == kOffsetRuns - 1) {
    a.totals[f] = at + sum;
    if (at + sum > a.most) *a.large = 1;
  }
  for (int t = t0; t < t1; t += U) {
    uint32_t x[U];
#pragma unroll
    for (int j = 0; j < U; ++j) x[j] = counts[int64_t(min(t + j, tiles - 1)) * stride];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      if (own && t + j < t1) base[int64_t(t + j) * a.buckets] = at;
      at += x[j];
    }
  }
}

// One tile's elements to their buckets. FMAX bounds the buckets.
template <int K, int EPT, int FMAX, bool MESH>
__global__ __launch_bounds__(kBucketBlock, 4) void k_bucket_scatter(BucketArgs a) {
  using SH = BucketShape<K>;
  constexpr int S = SH::S, BLOCK = kBucketBlock, Q = SH::STAGE, TILE = BLOCK * EPT;
  // a mesh's columns are read with all loads in flight (0.262 -> 0.241 ms for
  // 26.4M vertices); a batch's tile has few of its many columns, and registers
  // for all of them would spill (0.196 -> 0.216 ms for 15M)
  constexpr bool kAllCols = !MESH;
  // by bucket, from the tile's first: elements (two 16-bit counters a word, so
  // that the most buckets leave room for two workgroups on a CU), then the
  // place in the tile
  __shared__ uint32_t s_off[FMAX / 2];
  __shared__ uint32_t s_delta[FMAX];  // place in the bucket order minus place in the tile
  __shared__ alignas(16) uint32_t s_stage[Q * S];
  __shared__ uint16_t s_id[TILE];
  __shared__ uint32_t s_wave[BLOCK / kWave];
  const int tid = threadIdx.x, lane = lane_id();
  // neighbouring tiles write neighbouring runs of every bucket: on one die
  // they leave its L2 as whole lines (0.33 -> 0.26 ms for 26.4M vertices)
  const int64_t tile = die_tile(blockIdx.x, a.tiles);
  if (tile < 0) return;
  const int64_t i0 = tile * TILE, i1 = min(i0 + TILE, a.n);
  const TileMesh tm = tile_mesh<MESH>(a, i0, i1);
  for (int f = tid; f < (tm.count + 1) / 2; f += BLOCK) s_off[f] = 0;
  __syncthreads();
  uint32_t e[EPT][S];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int64_t v = min(i0 + i * BLOCK + tid, i1 - 1);
#pragma unroll
    for (int w = 0; w < K; ++w) e[i][w] = a.vtx[v * K + w];
  }
  // used flags: a wave's 64 bytes of item i are 16 words; lane l loads word
  // l % 16 of item 4 r + l / 16 and the lanes exchange them
  uint32_t flags[EPT / 4];
  static_assert(EPT % 4 == 0, "flags are loaded for four items at once");
#pragma unroll
  for (int r = 0; r < EPT / 4; ++r) {
    const int64_t at = i0 + (4 * r + (lane >> 4)) * BLOCK + (tid - lane) + 4 * (lane & 15);
    flags[r] = 0;
    if (at + 4 <= a.n) {
      flags[r] = *reinterpret_cast<const uint32_t*>(a.used + at);
    } else {
      for (int c = 0; c < 4; ++c)
        if (at + c < a.n) flags[r] |= uint32_t(a.used[at + c]) << (8 * c);
    }
  }
  uint32_t pos[EPT];
  uint32_t fb[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int64_t v = i0 + i * BLOCK + tid;
    const uint32_t word = __shfl(flags[i / 4], ((i & 3) << 4) + (lane >> 2));
    uint32_t x[K];
#pragma unroll
    for (int w = 0; w < K; ++w) x[w] = e[i][w];
    e[i][K] = uint32_t(v) | ((word >> (8 * (lane & 3)) & 1u) << 31);
    fb[i] = 0;
    pos[i] = 0xFFFFFFFFu;
    if (v < i1) {
      fb[i] = bucket_of<K, MESH>(a, tm, v, x) - uint32_t(tm.first);
      const uint32_t sh = 16 * (fb[i] & 1);
      pos[i] = atomicAdd(&s_off[fb[i] >> 1], 1u << sh) >> sh & 0xFFFFu;
    }
  }
  __syncthreads();
  {
    // bucket starts, for an even number of buckets per thread; also left for
    // the grouping, by tile 0 or, in a batch, by every tile for its own
    // buckets (several may write the same)
    uint32_t before = 0;
    if constexpr (MESH) before = uint32_t(a.mesh_off[tm.lo]);  // buckets are in mesh order
    constexpr int PER = (FMAX + 2 * BLOCK - 1) / (2 * BLOCK) * 2;
    const int per = (tm.count + 2 * BLOCK - 1) / (2 * BLOCK) * 2;  // <= PER
    const int f0 = tid * per, f1 = min(f0 + per, tm.count);
    uint32_t sum = 0, own = 0;
    if constexpr (kAllCols) {
      uint32_t t[PER];
#pragma unroll
      for (int i = 0; i < PER; ++i) t[i] = i < per && f0 + i < f1 ? a.totals[tm.first + f0 + i] : 0u;
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int f = f0 + i;
        if (i < per && f < f1) {
          s_delta[f] = t[i];
          own += t[i];
          sum += s_off[f >> 1] >> (16 * (f & 1)) & 0xFFFFu;
        }
      }
    } else {
      for (int f = f0; f < f1; ++f) {
        const uint32_t t = a.totals[tm.first + f];
        s_delta[f] = t;
        own += t;
        sum += s_off[f >> 1] >> (16 * (f & 1)) & 0xFFFFu;
      }
    }
    uint32_t all;
    uint32_t at = block_exclusive_scan<BLOCK>(sum, s_wave, &all);
    uint32_t start = before + block_exclusive_scan<BLOCK>(own, s_wave, &all);
    for (int f = f0; f < f1; f += 2) {
      const uint32_t c = s_off[f >> 1], t0 = s_delta[f], t1 = f + 1 < f1 ? s_delta[f + 1] : 0u;
      const uint32_t at1 = at + (c & 0xFFFFu), start1 = start + t0;
      s_off[f >> 1] = at | at1 << 16;
      s_delta[f] = start - at;
      if (f + 1 < f1) s_delta[f + 1] = start1 - at1;
      if (MESH || tile == 0) {
        a.starts[tm.first + f] = start;
        if (f + 1 < f1) a.starts[tm.first + f + 1] = start1;
      }
      at = at1 + (c >> 16);
      start = start1 + t1;
    }
    // the end of the last bucket, and the columns of a batch that no mesh uses
    if (tile == a.tiles - 1)
      for (int f = tm.first + tm.count + tid; f <= a.buckets; f += BLOCK) a.starts[f] = uint32_t(a.n);
  }
  const uint32_t* base = a.base + tile * int64_t(a.buckets) + tm.first;
  if constexpr (kAllCols) {
    constexpr int BPER = (FMAX + BLOCK - 1) / BLOCK;
    uint32_t bs[BPER];
#pragma unroll
    for (int i = 0; i < BPER; ++i) bs[i] = i * BLOCK + tid < tm.count ? base[i * BLOCK + tid] : 0u;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < BPER; ++i)
      if (i * BLOCK + tid < tm.count) s_delta[i * BLOCK + tid] += bs[i];
  } else {
    __syncthreads();
    for (int f = tid; f < tm.count; f += BLOCK) s_delta[f] += base[f];
  }
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    if (pos[i] == 0xFFFFFFFFu) continue;
    pos[i] += s_off[fb[i] >> 1] >> (16 * (fb[i] & 1)) & 0xFFFFu;
    s_id[pos[i]] = uint16_t(fb[i]);
  }
  const int total = int(i1 - i0);
  for (int q0 = 0; q0 < total; q0 += Q) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const uint32_t q = pos[i] - uint32_t(q0);
      if (q < uint32_t(Q)) store_words<S>(s_stage + q * S, e[i]);
    }
    __syncthreads();
    for (int j = tid; j < min(Q, total - q0); j += BLOCK) {
      uint32_t x[S];
      load_words<S>(s_stage + j * S, x);
      const uint32_t at = s_delta[s_id[q0 + j]] + uint32_t(q0 + j);
      if (int64_t(at) < a.n) store_words<S>(a.elems + int64_t(at) * S, x);
    }
    __syncthreads();
  }
}

// A bucket of more elements than two parts (many copies of some records) is
// grouped by several workgroups: its own takes the elements up to the next
// multiple of `part`, and for every multiple of `part` inside the bucket one
// more the part that begins there. Where there is no large bucket, these
// helpers, the last of the grid, leave after one load.
struct LargeBuckets {
  int32_t part;             // elements
  int32_t helpers;          // multiples of `part` in (0, n)
  const uint32_t* any;      // not 0: some bucket is large
  uint32_t* state;          // [helpers + 1][2] zeroed, by b0 / part: parts done, groups listed

  __device__ __forceinline__ uint32_t* listed(int64_t b0) const {
    return state + 2 * (uint32_t(b0) / uint32_t(part)) + 1;
  }
  // End of the part of a large bucket that begins at q0.
  __device__ __forceinline__ int64_t end(int64_t q0, int64_t b1) const {
    return min(b1, int64_t(uint32_t(q0) / uint32_t(part) + 1) * part);
  }
};
// One workgroup streams about 1,400 elements a microsecond: parts of n / 256
// take less time than the other buckets together, and below 4,096 elements the
// merge costs more than they share out.
constexpr int kLeastPart = 4096;
inline int32_t large_part(int64_t n) { return int32_t(std::max<int64_t>(kLeastPart, (n + 255) / 256)); }
inline int32_t large_helpers(int64_t n) { return int32_t((n + large_part(n) - 1) / large_part(n)) - 1; }

struct GroupBucketArgs {
  GroupArgs g;              // elems, n, pairs, rep, cmap, uelems, chunks, range_sums, ranges, mesh_*
  const uint32_t* starts;   // [buckets + 1]
  int32_t buckets;          // the grid is buckets + helpers
  int32_t target;           // elements per bucket aimed at
  LargeBuckets large;
};

// LDS of a workgroup that groups records: up to DCAP distinct ones at a time.
template <int K, int BLOCK, int DCAP>
struct GroupTable {
  static constexpr int TB = DCAP > 3072 ? 13 : DCAP > 1536 ? 12 : DCAP > 768 ? 11 : 10, TS = 1 << TB;
  static_assert(TS * 3 >= DCAP * 4, "table load");
  uint32_t key[K * DCAP];        // distinct records, word-major
  uint32_t tab[TS];              // place in that list
  uint32_t min[DCAP];            // smallest id
  uint32_t used[DCAP / 32];
  uint32_t wave[BLOCK / kWave];
  uint32_t n, full;
  uint32_t x[4];
};

// Share (hash interval) of a record, by bits that neither its bucket nor its
// slot goes by.
__device__ __forceinline__ uint32_t hash_share(uint32_t h, uint32_t shares) {
  h = (h ^ (h >> 15)) * 0x2C1B3C6Du;
  return __umulhi((h ^ (h >> 13)) * 0x297A2D39u, shares);
}

// Shares for a bucket of cnt elements whose list of dcap distinct records was
// full after e of them: records as many as would leave that many distinct ones
// among e if all were equally frequent, a little less than a list a share. Too
// few shares show as another full list.
__device__ __forceinline__ uint32_t group_shares(uint32_t e, uint32_t cnt, float dcap) {
  float lo = dcap, hi = float(cnt);
  for (int i = 0; i < 12; ++i) {
    const float d = 0.5f * (lo + hi);
    if (d * (1.0f - __expf(-float(e) / d)) < dcap) lo = d; else hi = d;
  }
  return max(2u, uint32_t(ceilf(hi / (0.93f * dcap))));
}
// Most shares a list's worth of elements may be cut into: records of different
// hashes need two at most.
constexpr uint32_t kMostShares = 8;

// Groups the elements [q0, q1) of the bucket [b0, b1), all of it or one part,
// and where this part is the last of its bucket to end, the bucket: true then,
// with the number of used groups, whose elements start at `slot0`.
//
// The records stream past a table in LDS. A thread that finds an empty slot
// writes its record to a free place of the list of distinct records and then
// publishes the place in the slot; if another thread was faster it keeps the
// place for its next new record. A group is named by q0 plus its place (no
// more places are taken than there are elements), so an element's pair is
// written at once. When the list is full, the records are cut into shares by
// their hash and every share takes a round of its own: an element is looked
// up in the round of its share alone, whose list then holds its record. (With
// elements that found the list full left to the next round, which looks all
// of them up again in a full table, 26M distinct 12-byte records of which few
// are used took 3.38 ms a call.)
//
// A part names its groups likewise and lists their elements (record, name) in
// the upper half of the bucket's slots of `uelems`; the last part to end has
// the names of equal records led to one of them (merge_parts), and no pair is
// written again. Where the records' hashes are too much alike for the table,
// or the groups too many for the list, the bucket goes through
// group_big_bucket.
template <int K, bool MESH, int BLOCK, int DCAP, bool PART>
__device__ __forceinline__ bool group_elements(const GroupArgs& a, const LargeBuckets& large,
                                           GroupTable<K, BLOCK, DCAP>& t, int64_t b0, int64_t b1, int64_t q0,
                                           int64_t q1, int64_t slot0, uint32_t* used_out) {
  using T = GroupTable<K, BLOCK, DCAP>;
  constexpr int S = K + 1, TB = T::TB, TS = T::TS;
  constexpr int PER = (DCAP + BLOCK - 1) / BLOCK;
  constexpr uint32_t kEmpty = 0xFFFFFFFFu, kUsedBit = 0x80000000u, kHard = 0x40000000u;
  const int tid = threadIdx.x;
  const uint32_t cnt = uint32_t(q1 - q0), last = cnt - 1u;
  const uint32_t half = uint32_t(b1 - b0) / 2;  // slots of the list
  uint32_t* const list = a.uelems + (b1 - half) * S;
  const uint32_t* const elems = a.elems + q0 * S;
  uint2* const pairs = a.pairs + q0;
  uint32_t names = uint32_t(q0), used_all = 0;
  bool hard = false;
  for (uint32_t share = 0, shares = 1; share < shares;) {
    for (int i = tid; i < TS; i += BLOCK) t.tab[i] = kEmpty;
    for (int i = tid; i < DCAP; i += BLOCK) t.min[i] = kEmpty;
    for (int i = tid; i < DCAP / 32; i += BLOCK) t.used[i] = 0;
    if (tid == 0) t.n = t.full = 0;
    __syncthreads();
    uint32_t mine = kEmpty;  // a place of this thread's own in the list of records
    uint32_t next[S];        // the record after the one in hand is on its way
    load_words<S>(elems + min(uint32_t(tid), last) * S, next);
    for (uint32_t q = tid; q < cnt; q += BLOCK) {
      if (cnt > DCAP && __hip_atomic_load(&t.full, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0) break;
      uint32_t e[S];
#pragma unroll
      for (int w = 0; w < S; ++w) e[w] = next[w];
      load_words<S>(elems + min(q + BLOCK, last) * S, next);
      const uint32_t h = hash_words<K>(e);
      if (shares > 1 && hash_share(h, shares) != share) continue;
      uint32_t sl = (h * 0x9E3779B1u) >> (32 - TB);
      uint32_t at = kEmpty;
      while (true) {
        uint32_t cur = __hip_atomic_load(&t.tab[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == kEmpty) {
          if (mine == kEmpty) mine = atomicAdd(&t.n, 1u);
          if (mine >= uint32_t(DCAP)) break;
#pragma unroll
          for (int w = 0; w < K; ++w) t.key[w * DCAP + mine] = e[w];
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
          cur = atomicCAS(&t.tab[sl], kEmpty, mine);
          if (cur == kEmpty) {
            at = mine;
            mine = kEmpty;
            break;
          }
        }
        bool eq = true;
#pragma unroll
        for (int w = 0; w < K; ++w) eq = eq && t.key[w * DCAP + cur] == e[w];
        if (eq) {
          at = cur;
          break;
        }
        sl = (sl + 1) & (TS - 1);
      }
      if (at == kEmpty) {
        t.full = q + 1;
        break;
      }
      const uint32_t id = e[K] & ~kUsedBit;
      pairs[q] = make_uint2(names + at, id);
      if (id < __hip_atomic_load(&t.min[at], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
        atomicMin(&t.min[at], id);
      if ((e[K] & kUsedBit) && !(__hip_atomic_load(&t.used[at >> 5], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP) >> (at & 31) & 1u))
        atomicOr(&t.used[at >> 5], 1u << (at & 31));
    }
    __syncthreads();
    const uint32_t full = uniform(t.full);
    if (full != 0) {
      const uint32_t more = shares == 1 ? uniform(group_shares(full, cnt, float(DCAP))) : 2;
      shares *= more;
      share *= more;
      hard = shares > kMostShares + kMostShares * (cnt / uint32_t(DCAP));
      __syncthreads();
      if (hard) break;
      continue;
    }
    // slots of the used groups, of all of them for the list; places nobody
    // published are skipped
    uint32_t x[PER], sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int d = tid * PER + j;
      x[j] = d >= DCAP || t.min[d] == kEmpty ? 0u : 1u | (t.used[d >> 5] >> (d & 31) & 1u) << 16;
      sum += x[j];
    }
    uint32_t all;
    uint32_t at = block_exclusive_scan<BLOCK>(sum, t.wave, &all);
    uint32_t listed = 0;  // groups listed before these
    if constexpr (PART) {
      if (tid == 0) t.x[0] = atomicAdd(large.listed(b0), all & 0xFFFFu);
      __syncthreads();
      listed = uniform(t.x[0]);
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int d = tid * PER + j;
      if (x[j] == 0) continue;
      const bool used = x[j] >> 16;
      const uint32_t name = names + uint32_t(d), rank = listed + (at & 0xFFFFu);
      if (PART || used) a.rep[name] = t.min[d];
      if (PART || !used) a.cmap[name] = used ? kUsedMark : -1;
      if (PART ? rank < half : used) {
        uint32_t e[S];
#pragma unroll
        for (int w = 0; w < K; ++w) e[w] = t.key[w * DCAP + d];
        e[K] = name;
        store_words<S>(PART ? list + int64_t(rank) * S : a.uelems + (slot0 + used_all + (at >> 16)) * S, e);
      }
      at += x[j];
    }
    used_all += uniform(all >> 16);
    names += uniform(min(t.n, uint32_t(DCAP)));
    if (++share < shares) __syncthreads();
  }
  if constexpr (PART) {
    // whoever ends last has the groups of all parts in view
    stores_in_l2();
    __syncthreads();
    if (tid == 0) {
      if (hard) atomicOr(large.listed(b0), kHard);
      __threadfence();  // for all of the workgroup's stores
      t.x[0] = atomicAdd(large.listed(b0) - 1, 1u) + 1u;
    }
    __syncthreads();
    const uint32_t parts = uint32_t(b1 - 1) / uint32_t(large.part) - uint32_t(b0) / uint32_t(large.part) + 1;
    if (uniform(t.x[0]) != parts) return false;
    __threadfence();
    const uint32_t listed = uniform(lb_load(large.listed(b0)));
    __syncthreads();  // t.x is used again
    hard = listed > half;
    if (!hard) used_all = merge_parts<K, BLOCK>(a, list, listed, b0, slot0, t.x);
  }
  if (hard) used_all = group_big_bucket<K, MESH, BLOCK>(a, b0, b1, slot0, t.x);
  *used_out = used_all;
  return true;
}

// The whole bucket is kept apart from the parts, whose listing in its loop
// cost the other 3 us of 60 (5.2M 8-byte vertices).
template <int K, bool MESH, int BLOCK, int DCAP>
__device__ __forceinline__ bool group_span(const GroupArgs& a, const LargeBuckets& large,
                                           GroupTable<K, BLOCK, DCAP>& t, int64_t b0, int64_t b1, int64_t q0,
                                           int64_t q1, int64_t slot0, uint32_t* used) {
  if (q1 - q0 < b1 - b0)
    return group_elements<K, MESH, BLOCK, DCAP, true>(a, large, t, b0, b1, q0, q1, slot0, used);
  return group_elements<K, MESH, BLOCK, DCAP, false>(a, large, t, b0, b1, b0, b1, slot0, used);
}

// Groups of one bucket, or of a part of one.
template <int K, bool MESH, int BLOCK, int DCAP>
__global__ __launch_bounds__(BLOCK, K <= 9 ? 8 : 4) void k_group_bucket(GroupBucketArgs b) {
  __shared__ GroupTable<K, BLOCK, DCAP> s_table;
  const GroupArgs& a = b.g;
  const int64_t part = b.large.part;
  int64_t f = blockIdx.x, q0 = 0;
  if (f >= b.buckets) {
    if (*b.large.any == 0) return;
    q0 = (f - b.buckets + 1) * part;
    int lo = 0, hi = b.buckets - 1;  // last bucket that starts at or before q0
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (int64_t(b.starts[mid]) <= q0) lo = mid; else hi = mid - 1;
    }
    f = lo;
  }
  const int64_t b0 = b.starts[f], b1 = b.starts[f + 1];
  const bool large = b1 - b0 > 2 * part;
  if (q0 > 0 && (!large || q0 == b0 || q0 >= b1)) return;  // nothing for a helper
  if (q0 == 0) q0 = b0;
  const int64_t q1 = large ? b.large.end(q0, b1) : b1;
  uint32_t used = 0;
  if (q1 > q0 && !group_span<K, MESH, BLOCK, DCAP>(a, b.large, s_table, b0, b1, q0, q1, b0, &used)) return;
  if (threadIdx.x == 0) {
    a.chunks[f] = make_uint2(uint32_t(b0), used);
    if (used) atomicAdd(&a.range_sums[group_run_of(f, b.buckets, a.ranges)], used);
  }
}

// Buckets that k_group left: two workgroups a CU that take one after the
// other, then the parts of large ones.
constexpr int kOverGrid = 512;
template <int K, bool MESH>
__global__ __launch_bounds__(kGroupBlock, K <= 9 ? 8 : 4) void k_group_over(GroupArgs a, LargeBuckets large,
                                                                            int64_t tiles) {
  constexpr int DCAP = BucketShape<K>::DCAP;
  __shared__ GroupTable<K, kGroupBlock, DCAP> s_table;
  const int64_t part = large.part;
  const uint32_t count = uniform(*a.over_count);
  const bool any = uniform(*a.over_any) != 0;
  uint32_t i = blockIdx.x;
  if (i >= count && !any) return;
  for (bool helper = false; !helper;) {
    uint32_t tile;
    if (i < count) {
      tile = uniform(a.over_list[i]);
      i += gridDim.x;
    } else {
      helper = true;
      if (!any || int(blockIdx.x) >= large.helpers) return;
      tile = uniform(a.over_at[blockIdx.x + 1]);
      if (tile == 0) return;
      --tile;
    }
    const int64_t b0 = uniform(a.over[tile].x), b1 = uniform(a.over[tile].y);
    const int64_t q0 = helper ? int64_t(blockIdx.x + 1) * part : b0;
    const int64_t q1 = b1 - b0 > 2 * part ? large.end(q0, b1) : b1;
    const uint32_t c = uniform(a.chunks[tile].y), slot0 = uniform(a.chunks[tile].x) + c;
    uint32_t used = 0;
    if (group_span<K, MESH, kGroupBlock, DCAP>(a, large, s_table, b0, b1, q0, q1, slot0, &used) &&
        threadIdx.x == 0) {
      a.chunks[tile].y = c + used;
      if (used) atomicAdd(&a.range_sums[group_run_of(tile, tiles, a.ranges)], used);
    }
    __syncthreads();
  }
}

}  // namespace mrx
