// Output order (Section 2, Step 3) of the used groups by sample sort.
//
// The grouping leaves one element (record, group name) per used group, in an
// order that has nothing to do with the records' order (hash order) and with
// no record twice. Their order by record is found in four or five launches
// whatever the record width, where an LSD sort takes one pass per key byte:
//  * k_split_sample: a regular sample of the elements (random in key order),
//    sorted in blocks; with a single block it yields the splitters;
//  * k_split_rank: ranks of the samples over all blocks; every os-th sample
//    becomes a splitter, F - 1 in all (only when there are several blocks);
//  * k_split_count: bucket of every element (a search over the splitters in
//    LDS) and the elements per bucket;
//  * k_split_scatter: the elements bucket by bucket;
//  * k_split_sort: one workgroup per bucket sorts it in LDS and finishes Step
//    3: sorted position = new id; output record and the map from group to
//    new id. (The representatives wait for the step that reads the pairs with
//    the groups' new ids: gathered here in output order they cost 0.08 ms for
//    4.2M, carried along from the scatter on 0.08 ms.)
// Measured (MI355X) against the packing, LSD passes and finalisation they
// replace: 4.2M 12-byte values of a 26.4M-vertex soup 0.32 ms (0.67 ms, twelve
// passes); 65,536 of a 429,165-vertex soup 0.062 ms (0.18 ms); 274,625 32-byte
// values 0.13 ms (0.48 ms, 32 passes). The scattered 16-byte stores of the
// scatter (58 G/s) and 4-byte stores of the map bound the large case, the
// launches and each workgroup's chain of LDS steps the small ones.
//
// The elements are distinct, so no step needs to be stable and their order
// inside a bucket is left to the arrival of atomics: the result does not
// depend on it. Every count stays on the device: grids are sized for U = N.
//
// A batch orders by (mesh id, record): the mesh of an element is the mesh of
// its name, and becomes the first of KW = K + 1 key words.
#pragma once

#include <algorithm>

#include "device_common.hpp"
#include "group_kernels.hpp"

namespace mrx {

// Shape for KW-word keys: buckets of at most CAP elements are sorted in LDS
// (their keys and names take at most 68 KB, two workgroups on a CU), and
// splitters are chosen for an average of TARGET = 0.4 CAP elements. With
// kOversample samples per bucket its size has a relative deviation of 1/4,
// and a bucket exceeds CAP about once in 10^5.
template <int KW>
struct SplitShape {
  static constexpr int BLOCK = 512;
  static constexpr int CAP = KW <= 2 ? 4096 : KW <= 4 ? 3072 : KW <= 5 ? 2560 : KW <= 8 ? 1536 : KW <= 17 ? 1024 : 512;
  static constexpr int E = CAP / BLOCK;
  static constexpr int TARGET = CAP * 2 / 5;
  // samples are sorted in blocks of half the capacity: twice as many
  // workgroups share the one step that has few of them
  static constexpr int SE = E / 2 > 0 ? E / 2 : 1;
  static constexpr int SCAP = SE * BLOCK;
};
constexpr int kOversample = 16;
constexpr int kMaxBuckets = 8192;      // splitter buckets: counters of 32 KB in LDS
constexpr int kMaxSampleBlocks = 32;
constexpr int kSplitRunBlock = 1024;   // k_split_count, k_split_scatter: one workgroup per run of chunks
constexpr int kSplitMaxChunks = 1024;  // chunks of a run
constexpr int kSplitLdsWords = 9 * 1024;  // splitter words k_split_count keeps in LDS
constexpr int kSplitParts = 64;        // parts an oversized bucket is cut into at once

// How U elements are split: F buckets from S = F * os samples.
struct SplitPlan {
  uint32_t buckets, os, samples;
};

// Buckets of about 256 elements up to 512 of them (a short sort on every CU
// rather than a long one on some), then larger ones up to TARGET, then more
// (rounding their number up to whole rounds of the 512 workgroups that the
// chip holds at once gained nothing: 48 and 46 us for a million elements, and
// as much lost to the ranks of more samples).
// Never fewer for more elements.
template <int KW>
__host__ __device__ inline uint32_t split_buckets(int64_t u) {
  if (u <= 512) return 1u;
  if (u <= 512 * 256) return uint32_t((u + 255) / 256);
  const int64_t f = (u + SplitShape<KW>::TARGET - 1) / SplitShape<KW>::TARGET;
  return uint32_t(f < 512 ? 512 : f < kMaxBuckets ? f : kMaxBuckets);
}

template <int KW>
__host__ __device__ inline SplitPlan split_plan(int64_t u) {
  using SH = SplitShape<KW>;
  SplitPlan p{split_buckets<KW>(u), 0u, 0u};
  if (p.buckets == 1) return p;
  // small buckets may vary more in size
  const int64_t t = u / p.buckets;
  const uint32_t os = t * 8 <= SH::CAP ? kOversample / 4 : t * 4 <= SH::CAP ? kOversample / 2 : kOversample;
  const uint32_t most = uint32_t(kMaxSampleBlocks * SH::SCAP) / p.buckets;
  p.os = most < os ? most : os;
  p.samples = p.buckets * p.os;
  return p;
}

// The most samples of any u <= n (not those of n: where the limit on samples
// cuts os, fewer buckets may have more of them in all).
template <int KW>
inline int64_t split_samples_bound(int64_t n) {
  const int64_t f = split_buckets<KW>(n);
  return f == 1 ? 0 : std::min<int64_t>(f * kOversample, int64_t(kMaxSampleBlocks) * SplitShape<KW>::SCAP);
}

// Scratch words of the whole sort of up to n elements in `runs` runs of chunks.
struct SplitScratch {
  int64_t samples, splitters, counts, starts, run_base, digits, words;
};
template <int KW>
inline SplitScratch split_scratch(int64_t n, int64_t runs) {
  const int64_t buckets = split_buckets<KW>(n);
  SplitScratch s{};
  int64_t at = 0;
  auto take = [&](int64_t words) {
    const int64_t r = at;
    at += (words + 3) & ~int64_t(3);
    return r;
  };
  s.samples = take(split_samples_bound<KW>(n) * KW);
  s.splitters = take(buckets * KW);
  s.counts = take(buckets);
  s.starts = take(buckets + 1);
  s.run_base = take(runs * buckets);
  s.digits = take((n + 1) / 2);
  s.words = at;
  return s;
}

struct SplitArgs {
  const uint32_t* sparse;      // [n][K+1] used groups' elements, in their chunks' slots
  const uint2* chunks;         // [tiles] (span start, used groups)
  const uint32_t* range_sums;  // [runs] used groups of each run of chunks
  int64_t tiles, runs, n;
  uint32_t* samples;           // [S][KW] sorted blocks of samples
  uint32_t* splitters;         // [F][KW], entry 0 unused
  uint32_t* counts;            // [F]
  uint32_t* starts;            // [F + 1]
  uint32_t* run_base;          // [runs][F] place of a run's elements in each bucket
  uint16_t* digits;            // [U] bucket of each element, in chunk order
  uint32_t* dense;             // [U][K+1] elements by bucket
  int32_t* cmap;               // [n] by group name: receives the new id
  uint32_t* out_vtx;           // [U][K]
  uint32_t* order;             // batches: [U] group names in output order
  int64_t* out_num;            // nullable
  Control* ctl;                // num_used: written by k_split_sample, read by the others
  const int64_t* mesh_off;     // batches
  const int32_t* mesh_tab;
  int32_t nmesh;
};

// Key words of an element: its record, for a batch with the mesh id first.
template <int K, bool MESH>
__device__ __forceinline__ void split_key(const SplitArgs& a, const uint32_t (&e)[K + 1],
                                          uint32_t (&key)[K + (MESH ? 1 : 0)]) {
  if constexpr (MESH) {
    key[0] = mesh_of(a.mesh_off, a.nmesh, e[K], a.mesh_tab);
#pragma unroll
    for (int w = 0; w < K; ++w) key[w + 1] = e[w];
  } else {
#pragma unroll
    for (int w = 0; w < K; ++w) key[w] = e[w];
  }
}

// Lexicographic comparison with key j of a table whose word w is at
// t[w * stride + j * step]; the first w0 words are known to be equal.
template <int KW, int N>
__device__ __forceinline__ bool key_less(const uint32_t* t, int stride, int step, int j, const uint32_t (&k)[N],
                                         int w0, bool or_equal) {
  bool lt = or_equal, open = true;
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    if (w < w0) continue;
    if (open) {
      const uint32_t x = t[w * stride + j * step];
      if (x != k[w]) {
        lt = x < k[w];
        open = false;
      }
    }
  }
  return lt;  // t[j] < k (or, with or_equal, t[j] <= k)
}

// Sorts n <= CAP elements of NW words by their first KW words (no two equal)
// in LDS: element i * BLOCK + tid is e[i], and after the call word w of the
// element of rank r is lds.x[w * CAP + r].
//
// The elements are compared by a 64-bit window of their key that starts at
// the first bit on which any two of them differ. Up to kSub - 1 of them cut
// the rest into sub-buckets of about 16, and the windows are moved together
// by sub-bucket. Everything in earlier sub-buckets is smaller and everything
// in later ones is larger, so an element's rank may be counted over any
// stretch that holds its sub-bucket: a wave takes 64 neighbours and counts
// over the union of their sub-buckets, a uniform loop over broadcast reads
// of two windows each, without divergence (a loop per lane over its own
// sub-bucket, comparing word by word, took four times as long). Elements
// with equal windows come out as a run, which is then ordered by whole keys.
constexpr int kSub = 128;
template <int NW, int CAP>
struct SortLds {
  union {
    uint32_t x[NW * CAP];                // sorted elements, word-major
    struct {
      alignas(16) uint64_t win[CAP];     // windows
      uint32_t rank[CAP];                // by place in win: rank | copies of the window before it << 16
    } s;
  };
  alignas(16) uint64_t spl[kSub];
  uint32_t ties[CAP / 2];                // elements per rank, two 16-bit counters a word
  uint32_t cnt[kSub];
  uint32_t start[kSub + 1];
  uint32_t first[NW];
  uint32_t w0, diff;
};

template <int KW, int NW, int CAP, int BLOCK, int E>
__device__ void block_sort(const uint32_t (&e)[E][NW], int n, SortLds<NW, CAP>& lds) {
  static_assert(BLOCK == 4 * kSub, "four threads rank a splitter");
  const int tid = threadIdx.x, lane = lane_id();
  __syncthreads();  // the caller's use of lds is over
  if (tid == 0) {
    lds.w0 = KW - 1;
    lds.diff = 0;
#pragma unroll
    for (int w = 0; w < KW; ++w) lds.first[w] = e[0][w];
  }
  if (tid < kSub) lds.cnt[tid] = 0;
  for (int i = tid; i < (n + 1) / 2; i += BLOCK) lds.ties[i] = 0;
  __syncthreads();
  // first word, and first bit of it, on which the elements differ
  int fd = KW;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n) continue;
#pragma unroll
    for (int w = KW - 1; w >= 0; --w)
      if (w < fd && e[i][w] != lds.first[w]) fd = w;
  }
#pragma unroll
  for (int w = 0; w < KW; ++w) {
    if (ballot(fd == w) != 0) {
      if (lane == 0) atomicMin(&lds.w0, uint32_t(w));
      break;
    }
  }
  __syncthreads();
  const int w0 = __builtin_amdgcn_readfirstlane(int(lds.w0));
  uint32_t df = 0;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n) continue;
#pragma unroll
    for (int w = 0; w < KW; ++w)
      if (w == w0) df |= e[i][w] ^ lds.first[w];
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) df |= __shfl_xor(df, o);
  if (lane == 0 && df) atomicOr(&lds.diff, df);
  __syncthreads();
  const int lead = __builtin_amdgcn_readfirstlane(lds.diff ? __clz(int(lds.diff)) : 0);
  uint64_t win[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    win[i] = 0;
#pragma unroll
    for (int w = 0; w < KW; ++w) {
      if (w != w0) continue;
      const uint64_t hi = uint64_t(e[i][w]) << 32 | (w + 1 < KW ? e[i][w + 1 < KW ? w + 1 : w] : 0u);
      const uint32_t lo = w + 2 < KW ? e[i][w + 2 < KW ? w + 2 : w] : 0u;
      win[i] = lead ? hi << lead | lo >> (32 - lead) : hi;
    }
    if (q < n) lds.s.win[q] = win[i];
  }
  // sub-buckets: a power of two with about 16 elements each
  int lg = 0;
  while ((1 << lg) < kSub && (16 << lg) < n) ++lg;
  const int m = 1 << lg;
  const int step = n >> lg;  // splitters are picked all over the elements
  __syncthreads();
  {
    const int c = tid >> 2;
    uint64_t k = 0;
    uint32_t r = 0;
    if (c < m - 1) {
      k = lds.s.win[c * step];
      for (int j = tid & 3; j < m - 1; j += 4) {
        const uint64_t x = lds.s.win[j * step];
        r += (x < k || (x == k && j < c)) ? 1u : 0u;
      }
    }
    r += __shfl_xor(r, 1);
    r += __shfl_xor(r, 2);
    if (c < m - 1 && (tid & 3) == 0) lds.spl[r] = k;
  }
  __syncthreads();
  uint32_t at[E];  // sub-bucket and place in it
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n) continue;
    int sb = 0;  // number of splitters <= the element
    for (int s = m >> 1; s > 0; s >>= 1)
      if (lds.spl[sb + s - 1] <= win[i]) sb += s;
    at[i] = uint32_t(sb) << 16 | atomicAdd(&lds.cnt[sb], 1u);
  }
  __syncthreads();
  if (tid < kWave) {
    static_assert(kSub == 2 * kWave, "two counters per lane");
    const uint32_t a = lds.cnt[2 * tid], b = lds.cnt[2 * tid + 1];
    const uint32_t inc = wave_inclusive_scan(a + b);
    lds.start[2 * tid] = inc - a - b;
    lds.start[2 * tid + 1] = inc - b;
    if (tid == kWave - 1) lds.start[kSub] = inc;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n) continue;
    at[i] = lds.start[at[i] >> 16] + (at[i] & 0xFFFFu);
    lds.s.win[at[i]] = win[i];
  }
  __syncthreads();
  // ranks, 64 neighbours at a time
  bool tied = false;
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q0 = i * BLOCK + (tid & ~(kWave - 1));
    if (q0 >= n) break;
    const int q = q0 + lane;
    // sub-buckets of the first and the last neighbour
    const int ql = min(q0 + kWave, n) - 1;
    int sa = 0, sz = 0;
    for (int s = m >> 1; s > 0; s >>= 1) {
      if (int(lds.start[sa + s]) <= q0) sa += s;
      if (int(lds.start[sz + s]) <= ql) sz += s;
    }
    const int lo = __builtin_amdgcn_readfirstlane(int(lds.start[sa]) & ~1);
    const int hi = __builtin_amdgcn_readfirstlane(int(lds.start[sz + 1]));
    const uint64_t k = lds.s.win[min(q, n - 1)];
    uint32_t r = uint32_t(lo);
    int j = lo;
    const ulonglong2* pw = reinterpret_cast<const ulonglong2*>(lds.s.win);
    for (; j + 8 <= hi; j += 8) {
      ulonglong2 p[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) p[t] = pw[(j >> 1) + t];
#pragma unroll
      for (int t = 0; t < 4; ++t) r += (p[t].x < k ? 1u : 0u) + (p[t].y < k ? 1u : 0u);
    }
    for (; j < hi; ++j) r += lds.s.win[j] < k ? 1u : 0u;
    if (q < n) {
      const uint32_t sh = (r & 1u) * 16;
      const uint32_t d = (atomicAdd(&lds.ties[r >> 1], 1u << sh) >> sh) & 0xFFFFu;
      tied = tied || d != 0;
      lds.s.rank[q] = r | d << 16;
    }
  }
  const bool any_tie = __syncthreads_or(tied) != 0;
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (i * BLOCK + tid < n) at[i] = lds.s.rank[at[i]];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n) continue;
    const uint32_t p = (at[i] & 0xFFFFu) + (at[i] >> 16);
#pragma unroll
    for (int w = 0; w < NW; ++w) lds.x[w * CAP + p] = e[i][w];
  }
  __syncthreads();
  if (!any_tie) return;
  // runs of equal windows by whole keys
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n) continue;
    const int r = int(at[i] & 0xFFFFu);
    const int c = int(lds.ties[r >> 1] >> ((r & 1) * 16) & 0xFFFFu);
    at[i] = uint32_t(r) | (c > 1 ? 1u << 31 : 0u);
    if (c > 1) {
      uint32_t p = 0;
      for (int j = r; j < r + c; ++j) p += key_less<KW>(lds.x, CAP, 1, j, e[i], w0, false) ? 1u : 0u;
      at[i] += p;
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i) {
    if (i * BLOCK + tid >= n || !(at[i] >> 31)) continue;
#pragma unroll
    for (int w = 0; w < NW; ++w) lds.x[w * CAP + (at[i] & 0x7FFFFFFFu)] = e[i][w];
  }
  __syncthreads();
}

// Slot of the element at place j, among nc chunks with places s_base (not
// decreasing) and first slots s_span.
__device__ __forceinline__ int64_t run_slot(const uint32_t* s_base, const uint32_t* s_span, int nc, uint32_t j) {
  int lo = 0, hi = nc - 1;  // last chunk that starts at or before j
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (s_base[mid] <= j) lo = mid; else hi = mid - 1;
  }
  return int64_t(s_span[lo]) + (j - s_base[lo]);
}

// Samples [b * SCAP, (b + 1) * SCAP), sorted. Sample j is element
// floor(j * U / S) in chunk order. Workgroup 0 also stores U. The bucket
// counts are cleared for k_split_count.
template <int K, bool MESH>
__global__ __launch_bounds__(SplitShape<K + (MESH ? 1 : 0)>::BLOCK) void k_split_sample(SplitArgs a) {
  constexpr int KW = K + (MESH ? 1 : 0), S = K + 1;
  using SH = SplitShape<KW>;
  constexpr int BLOCK = SH::BLOCK, CAP = SH::SCAP, E = SH::SE;
  constexpr int kRuns = 2048;
  __shared__ SortLds<KW, CAP> lds;
  __shared__ uint32_t s_wave[BLOCK / kWave];
  __shared__ uint32_t s_tab[kRuns + 2 * 2048];
  // run starts, then the starts and slots of the chunks the samples lie in
  uint32_t* const s_run = s_tab;
  constexpr int kChunks = 2048;
  uint32_t* const s_base = s_tab + kRuns;
  uint32_t* const s_span = s_base + kChunks;
  const int tid = threadIdx.x;
  const int64_t b = blockIdx.x;
  // run starts (at most kRuns runs)
  constexpr int PER = kRuns / BLOCK;
  uint32_t x[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int64_t r = int64_t(tid) * PER + i;
    x[i] = r < a.runs ? a.range_sums[r] : 0u;
    sum += x[i];
  }
  uint32_t u;
  uint32_t acc = block_exclusive_scan<BLOCK>(sum, s_wave, &u);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    s_run[tid * PER + i] = acc;
    acc += x[i];
  }
  if (b == 0 && tid == 0) a.ctl->num_used = int64_t(u);
  const SplitPlan plan = split_plan<KW>(u);
  for (int64_t f = b * BLOCK + tid; f < plan.buckets; f += int64_t(gridDim.x) * BLOCK) a.counts[f] = 0;
  __syncthreads();
  const int64_t j0 = b * CAP;
  const int n = int(min(int64_t(CAP), int64_t(plan.samples) - j0));
  if (n <= 0) return;
  auto place_of = [&](int64_t j) { return uint32_t(uint64_t(j) * u / plan.samples); };
  auto run_of = [&](uint32_t d) {  // last run that starts at or before d
    int lo = 0, hi = int(a.runs) - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_run[mid] <= d) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  // chunks of the runs the samples lie in; where there are too many for LDS
  // (few used values in tens of millions of vertices) each sample walks its run
  const int ra = run_of(place_of(j0)), rz = run_of(place_of(j0 + n - 1));
  const int64_t ta = group_range_start(ra, a.tiles, a.runs);
  const int64_t tc = group_range_start(rz + 1, a.tiles, a.runs) - ta;
  const bool in_lds = tc <= kChunks;
  if (in_lds) {
    constexpr int CPER = kChunks / BLOCK;
    const int per = int((tc + BLOCK - 1) / BLOCK);  // <= CPER
    uint2 c[CPER];
    uint32_t sum_c = 0;
#pragma unroll
    for (int i = 0; i < CPER; ++i) {
      const int t = tid * per + i;
      c[i] = (i < per && t < tc) ? a.chunks[ta + t] : make_uint2(0, 0);
      sum_c += c[i].y;
    }
    uint32_t all;
    uint32_t at = s_run[ra] + block_exclusive_scan<BLOCK>(sum_c, s_wave, &all);
#pragma unroll
    for (int i = 0; i < CPER; ++i) {
      const int t = tid * per + i;
      if (i < per && t < tc) {
        s_span[t] = c[i].x;
        s_base[t] = at;
        at += c[i].y;
      }
    }
    __syncthreads();
  }
  uint32_t e[E][KW];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    if (q >= n) continue;
    const uint32_t d = place_of(j0 + q);
    int64_t slot;
    if (in_lds) {
      slot = run_slot(s_base, s_span, int(tc), d);
    } else {
      const int r = run_of(d);
      uint32_t left = d - s_run[r];
      int64_t t = group_range_start(r, a.tiles, a.runs);
      const int64_t t1 = group_range_start(r + 1, a.tiles, a.runs);
      uint2 c = a.chunks[t];
      while (left >= c.y && t + 1 < t1) {
        left -= c.y;
        c = a.chunks[++t];
      }
      slot = int64_t(c.x) + left;
    }
    uint32_t el[S];
    load_words<S>(a.sparse + min(slot, a.n - 1) * S, el);
    split_key<K, MESH>(a, el, e[i]);
  }
  block_sort<KW, KW, CAP, BLOCK, E>(e, n, lds);
  if (plan.samples <= uint32_t(CAP)) {
    for (int f = 1 + tid; f < int(plan.buckets); f += BLOCK) {
#pragma unroll
      for (int w = 0; w < KW; ++w) a.splitters[int64_t(f) * KW + w] = lds.x[w * CAP + f * int(plan.os)];
    }
    return;
  }
  for (int q = tid; q < n; q += BLOCK) {
#pragma unroll
    for (int w = 0; w < KW; ++w) a.samples[(j0 + q) * KW + w] = lds.x[w * CAP + q];
  }
}

// Global rank of every sample: its place in its own block plus, in each other
// block, the number of smaller samples (a search each, one per lane of a
// 32-lane group, so that the searches' dependent loads overlap).
template <int K, bool MESH>
__global__ __launch_bounds__(256) void k_split_rank(SplitArgs a) {
  constexpr int KW = K + (MESH ? 1 : 0);
  constexpr int CAP = SplitShape<KW>::SCAP;
  static_assert(kMaxSampleBlocks == 32, "one lane per block of samples");
  const SplitPlan plan = split_plan<KW>(a.ctl->num_used);
  const int nb = int((plan.samples + CAP - 1) / CAP);
  if (nb < 2) return;  // the splitters are there already
  const int64_t j = int64_t(blockIdx.x) * 8 + (threadIdx.x >> 5);
  const int bl = threadIdx.x & 31;
  const bool in = j < plan.samples;
  const int own = int(j / CAP);
  uint32_t k[KW];
  uint32_t r = 0;
  if (in) {
#pragma unroll
    for (int w = 0; w < KW; ++w) k[w] = a.samples[j * KW + w];
    if (bl == own) {
      r = uint32_t(j - int64_t(own) * CAP);
    } else if (bl < nb) {
      int lo = 0, hi = min(CAP, int(plan.samples) - bl * CAP);
      const uint32_t* blk = a.samples + int64_t(bl) * CAP * KW;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key_less<KW>(blk, 1, KW, mid, k, 0, false)) lo = mid + 1; else hi = mid;
      }
      r = uint32_t(lo);
    }
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) r += __shfl_xor(r, o);
  if (in && bl == 0 && r > 0 && r % plan.os == 0) {
    const uint32_t f = r / plan.os;
    if (f < plan.buckets) {
#pragma unroll
      for (int w = 0; w < KW; ++w) a.splitters[int64_t(f) * KW + w] = k[w];
    }
  }
}

// The elements of run `run` of chunks: *first is the run's place in chunk
// order, s_base/s_span its chunks' places and slots, *chunks their number.
// Returns the run's elements. The loads of the chunks and of the other runs'
// counts are in flight together and share one exchange: these kernels' chains
// of dependent loads and barriers are what a small order costs.
template <int BLOCK>
__device__ __forceinline__ uint32_t open_run(const SplitArgs& a, int64_t run, uint32_t* s_base, uint32_t* s_span,
                                             uint2* s_wave, uint32_t* first, int* chunks) {
  static_assert(BLOCK >= kSplitMaxChunks, "one chunk per thread");
  constexpr int WAVES = BLOCK / kWave;
  const int tid = threadIdx.x, wave = tid / kWave;
  const int64_t t0 = group_range_start(run, a.tiles, a.runs);
  const int nc = int(group_range_start(run + 1, a.tiles, a.runs) - t0);
  uint2 c = make_uint2(0, 0);
  if (tid < nc) c = a.chunks[t0 + tid];
  uint32_t pre = 0;
  for (int64_t r = tid; r < run; r += BLOCK) pre += a.range_sums[r];
  const uint32_t inc = wave_inclusive_scan(c.y);
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) pre += __shfl_xor(pre, o);
  if (lane_id() == kWave - 1) s_wave[wave] = make_uint2(inc, pre);
  __syncthreads();
  uint32_t at = inc - c.y, total = 0, f = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const uint2 x = s_wave[w];
    if (w < wave) at += x.x;
    total += x.x;
    f += x.y;
  }
  if (tid < nc) {
    s_base[tid] = at;
    s_span[tid] = c.x;
  }
  *first = f;
  *chunks = nc;
  __syncthreads();
  return total;
}

// Bucket of every element of a run of chunks (the number of splitters not
// above it) and where the run's elements go in each bucket. Splitters, or
// every 2^sh-th of them where they are too wide and many, are searched in LDS
// and the last sh steps in memory.
template <int K, bool MESH>
__global__ __launch_bounds__(kSplitRunBlock) void k_split_count(SplitArgs a) {
  constexpr int KW = K + (MESH ? 1 : 0), S = K + 1, BLOCK = kSplitRunBlock;
  __shared__ uint32_t s_spl[kSplitLdsWords];
  __shared__ uint32_t s_cnt[kMaxBuckets];
  __shared__ uint32_t s_base[kSplitMaxChunks], s_span[kSplitMaxChunks];
  __shared__ uint2 s_wave[BLOCK / kWave];
  const int tid = threadIdx.x;
  const int64_t run = blockIdx.x;
  const SplitPlan plan = split_plan<KW>(a.ctl->num_used);
  const int F = int(plan.buckets);
  if (F == 1) {  // nothing to split: every element is in bucket 0
    if (tid == 0) a.run_base[run] = atomicAdd(&a.counts[0], a.range_sums[run]);
    return;
  }
  int sh = 0;
  while (((F - 1) >> sh) * KW > kSplitLdsWords) ++sh;
  const int m = (F - 1) >> sh;  // LDS entry i is splitter (i + 1) << sh
  constexpr int PER = kSplitLdsWords / BLOCK;
  uint32_t spl[PER];  // all in flight at once
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int t = i * BLOCK + tid, j = t / KW, w = t - j * KW;
    spl[i] = t < m * KW ? a.splitters[(int64_t(j + 1) << sh) * KW + w] : 0u;
  }
  for (int f = tid; f < F; f += BLOCK) s_cnt[f] = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int t = i * BLOCK + tid, j = t / KW, w = t - j * KW;
    if (t < m * KW) s_spl[w * m + j] = spl[i];
  }
  uint32_t first;
  int nc;
  const uint32_t total = open_run<BLOCK>(a, run, s_base, s_span, s_wave, &first, &nc);
  constexpr int U = S <= 5 ? 4 : 2;
  for (uint32_t j0 = 0; j0 < total; j0 += BLOCK * U) {
    uint32_t e[U][S];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const uint32_t j = min(j0 + uint32_t(r * BLOCK + tid), total - 1);
      load_words<S>(a.sparse + run_slot(s_base, s_span, nc, j) * S, e[r]);
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const uint32_t j = j0 + uint32_t(r * BLOCK + tid);
      if (j >= total) continue;
      uint32_t k[KW];
      split_key<K, MESH>(a, e[r], k);
      int lo = 0, hi = m;  // LDS entries not above the key
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key_less<KW>(s_spl, m, 1, mid, k, 0, true)) lo = mid + 1; else hi = mid;
      }
      int f = lo << sh;
      if (sh > 0) {
        int b = f, c = min(F, (lo + 1) << sh);  // splitter b is not above the key (b = 0: none), c is
        while (c - b > 1) {
          const int mid = (b + c) >> 1;
          if (key_less<KW>(a.splitters, 1, KW, mid, k, 0, true)) b = mid; else c = mid;
        }
        f = b;
      }
      a.digits[first + j] = uint16_t(f);
      atomicAdd(&s_cnt[f], 1u);
    }
  }
  __syncthreads();
  uint32_t* base = a.run_base + run * int64_t(F);
  for (int f = tid; f < F; f += BLOCK) {
    const uint32_t c = s_cnt[f];
    base[f] = c ? atomicAdd(&a.counts[f], c) : 0u;
  }
}

// The run's elements to their buckets. Workgroup 0 leaves the bucket starts
// for k_split_sort.
template <int K, bool MESH>
__global__ __launch_bounds__(kSplitRunBlock) void k_split_scatter(SplitArgs a) {
  constexpr int KW = K + (MESH ? 1 : 0), S = K + 1, BLOCK = kSplitRunBlock;
  __shared__ uint32_t s_at[kMaxBuckets];
  __shared__ uint32_t s_base[kSplitMaxChunks], s_span[kSplitMaxChunks];
  __shared__ uint2 s_wave2[BLOCK / kWave];
  __shared__ uint32_t s_wave[BLOCK / kWave];
  const int tid = threadIdx.x;
  const int64_t run = blockIdx.x;
  const int64_t u = a.ctl->num_used;
  const SplitPlan plan = split_plan<KW>(u);
  const int F = int(plan.buckets);
  // bucket starts: PER consecutive counts per thread
  constexpr int PER = kMaxBuckets / BLOCK;
  const int per = (F + BLOCK - 1) / BLOCK;  // <= PER
  const uint32_t* base = a.run_base + run * int64_t(F);
  uint32_t c[PER], at[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = tid * per + i;
    c[i] = (i < per && f < F) ? a.counts[f] : 0u;
    at[i] = (i < per && f < F) ? base[f] : 0u;
    sum += c[i];
  }
  uint32_t first;
  int nc;
  const uint32_t total = open_run<BLOCK>(a, run, s_base, s_span, s_wave2, &first, &nc);
  uint32_t all;
  uint32_t acc = block_exclusive_scan<BLOCK>(sum, s_wave, &all);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int f = tid * per + i;
    if (i < per && f < F) {
      if (run == 0) a.starts[f] = acc;
      s_at[f] = acc + at[i];
      acc += c[i];
    }
  }
  if (run == 0 && tid == 0) a.starts[F] = all;
  __syncthreads();
  constexpr int U = S <= 5 ? 4 : 2;
  for (uint32_t j0 = 0; j0 < total; j0 += BLOCK * U) {
    uint32_t e[U][S], f[U];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const uint32_t j = min(j0 + uint32_t(r * BLOCK + tid), total - 1);
      load_words<S>(a.sparse + run_slot(s_base, s_span, nc, j) * S, e[r]);
      f[r] = F > 1 ? min(uint32_t(a.digits[first + j]), uint32_t(F - 1)) : 0u;
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      if (j0 + uint32_t(r * BLOCK + tid) >= total) continue;
      const int64_t p = atomicAdd(&s_at[f[r]], 1u);
      if (p < a.n) store_words<S>(a.dense + p * S, e[r]);
    }
  }
}

// Writes n sorted elements (lds.x: key words, then the name) as output
// vertices [c0, c0 + n).
template <int K, bool MESH, int CAP, int BLOCK>
__device__ __forceinline__ void split_output(const SplitArgs& a, const SortLds<K + (MESH ? 1 : 0) + 1, CAP>& lds,
                                             int64_t c0, int n) {
  constexpr int KW = K + (MESH ? 1 : 0), KO = MESH ? 1 : 0;
  const int tid = threadIdx.x;
  uint32_t* out = a.out_vtx + c0 * K;
  for (int t = tid; t < n * K; t += BLOCK) {
    const int q = t / K, w = t - q * K;
    out[t] = lds.x[(w + KO) * CAP + q];
  }
  for (int q = tid; q < n; q += BLOCK) {
    const uint32_t g = lds.x[KW * CAP + q];
    if (int64_t(g) < a.n) a.cmap[g] = int32_t(c0 + q);
    if constexpr (MESH) a.order[c0 + q] = g;
  }
}

// Sorts bucket f and writes its output vertices. A bucket of more than CAP
// elements (about one in 10^5, or every one where there would be more than
// kMaxBuckets) is cut by quantiles of its first CAP elements, which are as
// good as random, and sorted part by part, each part picked out of the whole
// bucket; a part that does not fit either is narrowed to below one of its
// own elements until it does.
template <int K, bool MESH>
__global__ __launch_bounds__(SplitShape<K + (MESH ? 1 : 0)>::BLOCK, 4) void k_split_sort(SplitArgs a) {
  constexpr int KW = K + (MESH ? 1 : 0), S = K + 1, NW = KW + 1;
  using SH = SplitShape<KW>;
  constexpr int BLOCK = SH::BLOCK, CAP = SH::CAP, E = SH::E;
  __shared__ SortLds<NW, CAP> lds;
  __shared__ uint32_t s_lo[KW], s_hi[KW], s_cnt;
  __shared__ uint32_t s_piv[kSplitParts * KW];
  const int tid = threadIdx.x;
  const int64_t u = a.ctl->num_used;
  if (blockIdx.x == 0 && tid == 0 && a.out_num) *a.out_num = u;
  const SplitPlan plan = split_plan<KW>(u);
  const uint32_t f = blockIdx.x;
  if (f >= plan.buckets) return;
  const int64_t c0 = a.starts[f];
  const int64_t cnt = int64_t(a.starts[f + 1]) - c0;
  if (cnt <= 0 || c0 + cnt > a.n) return;
  auto load_key = [&](int64_t p, uint32_t(&x)[NW]) {
    uint32_t el[S], key[KW];
    load_words<S>(a.dense + p * S, el);
    split_key<K, MESH>(a, el, key);
#pragma unroll
    for (int w = 0; w < KW; ++w) x[w] = key[w];
    x[KW] = el[K];
  };
  // one pass of the loop sorts the bucket, or of an oversized one first the
  // elements its parts are chosen by and then each part, [lo, hi) by key (lo
  // of the first and hi of the last open)
  const int parts = int(min((cnt + CAP / 2 - 1) / (CAP / 2), int64_t(kSplitParts)));
  int part = -1;
  int64_t done = 0;  // elements below lo, which are written
  bool open_lo = true, open_hi = false, narrowed = false;
  int n = int(min(cnt, int64_t(CAP)));
  while (true) {
    uint32_t e[E][NW];
#pragma unroll
    for (int i = 0; i < E; ++i) {
      const int q = i * BLOCK + tid;
      if (q >= n) continue;
      if (part < 0) {
        load_key(c0 + q, e[i]);
      } else {
#pragma unroll
        for (int w = 0; w < NW; ++w) e[i][w] = lds.x[w * CAP + q];
      }
    }
    if (n > 0) block_sort<KW, NW, CAP, BLOCK, E>(e, n, lds);
    if (cnt <= CAP) {
      split_output<K, MESH, CAP, BLOCK>(a, lds, c0, n);
      return;
    }
    if (part < 0) {
      for (int t = tid; t < (parts - 1) * KW; t += BLOCK) {
        const int i = t / KW, w = t - i * KW;
        s_piv[t] = lds.x[w * CAP + int(int64_t(i + 1) * CAP / parts)];
      }
      part = 0;
    } else {
      split_output<K, MESH, CAP, BLOCK>(a, lds, c0 + done, n);
      done += n;
      if (open_hi) return;  // the last part
      if (tid < KW) s_lo[tid] = s_hi[tid];
      open_lo = false;
      if (!narrowed) ++part;
    }
    __syncthreads();
    open_hi = part == parts - 1;
    narrowed = false;
    if (tid < KW && !open_hi) s_hi[tid] = s_piv[part * KW + tid];
    while (true) {
      if (tid == 0) s_cnt = 0;
      __syncthreads();
      // the part's elements, in arrival order, in lds.x (as many as fit)
      for (int64_t p0 = 0; p0 < cnt; p0 += BLOCK) {
        const int64_t p = p0 + tid;
        if (p >= cnt) continue;
        uint32_t x[NW];
        load_key(c0 + p, x);
        const bool above = open_lo || key_less<KW>(s_lo, 1, 0, 0, x, 0, true);
        const bool below = open_hi || !key_less<KW>(s_hi, 1, 0, 0, x, 0, true);
        if (!(above && below)) continue;
        const uint32_t q = atomicAdd(&s_cnt, 1u);
        if (q < uint32_t(CAP)) {
#pragma unroll
          for (int w = 0; w < NW; ++w) lds.x[w * CAP + q] = x[w];
        }
      }
      __syncthreads();
      n = int(s_cnt);
      if (n <= CAP) break;
      // too many: hi becomes one of the picked elements other than lo
      bool is_lo = !open_lo;
      for (int w = 0; w < KW; ++w) is_lo = is_lo && lds.x[w * CAP] == s_lo[w];
      __syncthreads();
      if (tid < KW) s_hi[tid] = lds.x[tid * CAP + (is_lo ? 1 : 0)];
      open_hi = false;
      narrowed = true;
      __syncthreads();
    }
  }
}

}  // namespace mrx
