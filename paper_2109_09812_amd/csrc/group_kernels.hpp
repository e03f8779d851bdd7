// Hash grouping: duplicate detection (Section 2, Steps 2-3) without sorting
// every vertex by its full key.
//
// Section 2 finds duplicates by sorting all N (record, id) pairs by the full
// record; the sort is the dominant cost. Grouping only needs equal records
// to be adjacent. Up to some 26 million vertices they are put in buckets in
// one pass (bucket_kernels.hpp); beyond that, and with k_group below, the N
// pairs are first sorted by a few hash digits of the record (stable, so within
// a bucket of equal hash digits ids stay ascending). Equal records share
// their hash, so every group of duplicates lies inside one bucket, and buckets
// are small enough (a few hundred records) to be grouped in LDS: k_group
// numbers the groups of each bucket in
// order of their first copy, which is the smallest original id (Step 2's
// representative rule), and emits one element per *used* group. Only those U
// elements are then sorted by their full key (Step 3's output order), a
// fraction of the N the plain method sorts.
//
// A group is named by a position: each workgroup owns the buckets that start
// in its chunk, i.e. a span of sorted positions disjoint from every other
// chunk's, and its k-th group (in order of first copy) is called span start +
// k, its k-th used group's element goes to slot span start + k of the
// element buffer. Names stay below N and need no count of earlier chunks, so
// the chunks never wait for each other; the chunks' counts go to per-run
// sums, from which the kernels that order the used groups (split_kernels.hpp)
// find the elements.
//
// A batch groups by (mesh id, record): every mesh owns a range of buckets,
// so its vertices end up at the sorted positions of its own vertex range,
// and a group is named by the position of its first copy instead, which
// lies in that range (the name tells the group's mesh).
//
// A bucket that does not fit the LDS window (many copies of one value, or an
// unlucky hash) is left to k_group_over (bucket_kernels.hpp), which groups it
// by a hash table as those of the one partition pass.
#pragma once

#include "device_common.hpp"
#include "sort_kernels.hpp"

namespace mrx {

// Shape of the grouping kernel for K-word records: a workgroup owns the
// buckets that start inside its chunk of CHUNK sorted positions and reads a
// window of WIN positions (the one before the chunk, the chunk, and room for
// its last bucket to end) into LDS.
template <int K>
struct GroupShape {
  static constexpr int S = K + 1;
  static constexpr int BLOCK = 512;
  static constexpr int WIN = S <= 4 ? 3072 : S <= 6 ? 2048 : S <= 9 ? 1024 : 512;
  static constexpr int CHUNK = WIN * 2 / 3;
  static constexpr int IPT = WIN / BLOCK;
  // open-addressing table of at least 4/3 WIN slots (a window holds at most
  // WIN - 2 distinct records, so probing always meets an empty slot)
  static constexpr int TB = WIN > 2048 ? 12 : WIN > 1024 ? 12 : WIN > 512 ? 11 : 10;
  static constexpr int TS = 1 << TB;
  // average bucket size the host aims for when it picks the hash passes
  static constexpr int TARGET_BUCKET = CHUNK / 4;
  // waves per SIMD the register budget is set for: three workgroups per CU
  // (LDS: keys of the window + the table, at most 53 KB each)
  static constexpr int MIN_WAVES_PER_SIMD = 3 * (BLOCK / 64) / 4;
  static_assert(WIN % BLOCK == 0, "window positions per thread");
  static_assert(TS * 3 >= WIN * 4, "table load");
};

// Per-chunk record of k_group: span start, used groups.
struct GroupArgs {
  const uint32_t* elems;   // [n][K+1] elements in (hash bucket, id) order
  int64_t n;
  uint32_t bucket_mask;    // bucket of a record = hash & bucket_mask
  uint2* pairs;            // [n] (group name, original id) per position
  uint32_t* rep;           // [n] smallest original id of each used group, by name
  int32_t* cmap;           // [n] -1 for unused groups (used ones are set by the key sort's finalisation)
  uint32_t* uelems;        // [n][K+1] (record, group name) of every used group, in its span's slots
  uint2* chunks;           // [chunks] (span start, used groups)
  uint32_t* range_sums;    // [ranges] zeroed: used groups of each run of chunks
                           // k_group_compact_hist takes (spread over many addresses: atomics
                           // on one address from every chunk would serialise)
  int64_t ranges;          // that kernel's grid (group_compact_ranges)
  int32_t* status;
  // batches (k_group<K, true>): vertex offsets [nmesh+1] and their bucket
  // table; the grouping key is then (mesh id, record)
  const int64_t* mesh_off;
  const int32_t* mesh_tab;
  const uint2* mesh_buckets;  // each mesh's hash buckets (mesh_bucket)
  int32_t nmesh;
  // k_group: buckets that run past their chunk's window, left to
  // k_group_over: [chunks] (first position, end), and the chunks that have one
  uint2* over;
  uint32_t* over_list;
  uint32_t* over_count;    // zeroed
  int32_t part;            // of a larger one than two parts the chunk (+ 1), by multiples of `part` inside it
  uint32_t* over_any;      // zeroed; set where there is a larger one
  uint32_t* over_at;       // zeroed
};

// Runs of consecutive chunks, one per workgroup of k_group_compact_hist: few
// (each flushes its digit histograms once), each of at most kCompactMaxChunks.
constexpr int kCompactMaxChunks = 2048;
constexpr int64_t kCompactMinRanges = 512;
__host__ __device__ inline int64_t group_compact_ranges(int64_t tiles) {
  const int64_t by_size = (tiles + kCompactMaxChunks - 1) / kCompactMaxChunks;
  return tiles < kCompactMinRanges ? tiles : (by_size > kCompactMinRanges ? by_size : kCompactMinRanges);
}
// First chunk of run w (of `ranges` runs over `tiles` chunks).
__host__ __device__ inline int64_t group_range_start(int64_t w, int64_t tiles, int64_t ranges) {
  return w * tiles / ranges;
}

// Run of a chunk: the last one whose first chunk is not after it.
__device__ __forceinline__ int64_t group_run_of(int64_t tile, int64_t tiles, int64_t ranges) {
  int64_t w = tile * ranges / tiles;
  while (w + 1 < ranges && group_range_start(w + 1, tiles, ranges) <= tile) ++w;
  while (w > 0 && group_range_start(w, tiles, ranges) > tile) --w;
  return w;
}

template <int K>
__device__ __forceinline__ bool lds_keys_equal(const uint32_t* s_keys, int a, int b, int win) {
  bool eq = true;
#pragma unroll
  for (int w = 0; w < K; ++w) eq = eq && (s_keys[w * win + a] == s_keys[w * win + b]);
  return eq;
}

// MESH (batches): the elements are (record, id) as always, but records are
// told apart by (mesh of id, record): the key held in LDS, hashed and
// compared is KW = K + 1 words with the mesh id first, and the shape is that
// of KW-word records. Each mesh's vertices then occupy its own vertex range
// of sorted positions (its buckets come after those of the meshes before
// it), and a group is named by the sorted position of its first copy, which
// lies in that range: the mesh of a group is the mesh of its name.
// Waves per SIMD the grouping kernel's registers are budgeted for: the
// shape's, except for batches of 1- and 2-word records, whose mesh-id key
// word and lookups would otherwise spill to scratch at that budget.
template <int K, bool MESH>
constexpr int group_min_waves() {
  return MESH && K <= 2 ? GroupShape<K + 1>::MIN_WAVES_PER_SIMD - 1
                        : GroupShape<MESH ? K + 1 : K>::MIN_WAVES_PER_SIMD;
}

// End of the bucket that starts at position b0 (of the last one of a chunk of
// k_group that runs past its window): the elements are in bucket order, so
// every step takes BLOCK probes between the last position known to be in the
// bucket and the first known not to be, three for 10M copies (a walk over
// them took 10 ms).
template <int K, bool MESH, int BLOCK>
__device__ int64_t end_of_bucket(const GroupArgs& a, int64_t b0, uint32_t* s_x) {
  constexpr int S = K + 1;
  const int tid = threadIdx.x;
  uint32_t mesh = 0;
  if constexpr (MESH) mesh = mesh_of(a.mesh_off, a.nmesh, b0, a.mesh_tab);
  auto bucket_at = [&](int64_t p) {
    uint32_t e[S];
    load_words<S>(a.elems + p * S, e);
    if constexpr (MESH) return mesh_bucket(a.mesh_buckets, mesh, hash_mesh_words<K>(mesh, e));
    else return hash_words<K>(e) & a.bucket_mask;
  };
  const uint32_t bucket = bucket_at(b0);
  int64_t in = b0, out = MESH ? min(a.n, a.mesh_off[mesh + 1]) : a.n;  // buckets belong to meshes
  while (out - in > 1) {
    const int64_t step = (out - in + BLOCK) / (BLOCK + 1);
    if (tid == 0) {
      s_x[0] = uint32_t(in);
      s_x[1] = uint32_t(out);
    }
    __syncthreads();
    const int64_t p = in + (tid + 1) * step;
    if (p < out) {
      if (bucket_at(p) == bucket) atomicMax(&s_x[0], uint32_t(p));
      else atomicMin(&s_x[1], uint32_t(p));
    }
    __syncthreads();
    in = s_x[0];
    out = max(int64_t(s_x[1]), in + 1);
    __syncthreads();
  }
  return out;
}

// Node of record e (element i of `recs`) among chains that hang off a table in
// memory, of which every element owns two words, [i * S] the head of chain i
// and [i * S + 1] the next of node i: the node that holds an equal record, or
// i itself, after `publish`. Everything the workgroup's waves tell each other
// through memory goes by agent-scope atomics (L2), in order. Chains
// are only ever prepended to, so a failed insertion re-reads what was added
// and retries.
template <int K, class Publish>
__device__ __forceinline__ uint32_t chain_node(uint32_t* table, const uint32_t* recs, uint32_t heads, uint32_t i,
                                               const uint32_t (&e)[K + 1], Publish publish) {
  constexpr int S = K + 1;
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  uint32_t* const head = table + int64_t(__umulhi(hash_words<K>(e) * 0x9E3779B1u, heads)) * S;
  uint32_t seen = kNone;  // nodes from here on are known not to match
  uint32_t cur = lb_load(head);
  while (true) {
    for (uint32_t q = cur; q != seen && q != kNone; q = lb_load(table + int64_t(q) * S + 1)) {
      bool eq = true;
#pragma unroll
      for (int w = 0; w < K; ++w) eq = eq && recs[int64_t(q) * S + w] == e[w];
      if (eq) return q;
    }
    seen = cur;
    lb_store(table + int64_t(i) * S + 1, cur);
    publish();
    stores_in_l2();  // one workgroup builds the chains
    const uint32_t was = atomicCAS(head, cur, i);
    if (was == cur) return i;
    cur = was;
  }
}

// Groups one bucket of any size, [b0, b1), through chains whose table lies in
// the bucket's slots of `uelems` until its elements are written there; a node
// is the position of some copy and names its group. The record
// at b0 is the likeliest one to have thousands of copies: its copies are told
// by a comparison in registers and touch no table. Bound: the round trips
// of one workgroup's atomics, some 30 elements a microsecond where copies of
// several values meet; only buckets whose records group_span cannot cut by
// their hash come here. Returns
// the number of used groups; their elements start at slot `upre`.
template <int K, bool MESH, int BLOCK>
__device__ uint32_t group_big_bucket(const GroupArgs& a, int64_t b0, int64_t b1, int64_t upre, uint32_t* s_x) {
  constexpr int S = K + 1;
  constexpr int U = S <= 5 ? 4 : 2;  // elements in flight per thread
  constexpr uint32_t kNone = 0xFFFFFFFFu, kUsedBit = 0x80000000u;
  const int tid = threadIdx.x;
  uint32_t hot[S];
  load_words<S>(a.elems + b0 * S, hot);
  const uint32_t cnt = uint32_t(b1 - b0);
  uint32_t* const table = a.uelems + b0 * S;
  for (uint32_t i = tid; i < cnt; i += BLOCK) lb_store(table + int64_t(i) * S, kNone);
  if (tid == 0) {
    lb_store(reinterpret_cast<uint32_t*>(a.cmap) + b0, uint32_t(-1));
    s_x[1] = 0;                      // the hot group is used
    s_x[2] = hot[K] & 0x7FFFFFFFu;   // its smallest id
    s_x[3] = 0;                      // used groups
  }
  stores_in_l2();
  __syncthreads();
  uint32_t* const rep = a.rep;
  uint32_t* const cm = reinterpret_cast<uint32_t*>(a.cmap);
  // ---- every element finds or becomes its group's node
  for (int64_t base = b0; base < b1; base += BLOCK * U) {
    uint32_t e[U][S];
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t p = base + r * BLOCK + tid;
      if (p < b1) load_words<S>(a.elems + p * S, e[r]);
    }
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const int64_t p = base + r * BLOCK + tid;
      if (p >= b1) continue;
      const uint32_t id = e[r][K] & 0x7FFFFFFFu;
      bool is_hot = true;
#pragma unroll
      for (int w = 0; w < K; ++w) is_hot = is_hot && e[r][w] == hot[w];
      uint32_t node = uint32_t(b0);
      if (is_hot) {
        if ((e[r][K] & kUsedBit) && s_x[1] == 0u) s_x[1] = 1u;
        if (id < s_x[2]) atomicMin(&s_x[2], id);
      } else {
        node += chain_node<K>(table, a.elems + b0 * S, cnt, uint32_t(p - b0), e[r], [&] {
          lb_store(rep + p, id);
          lb_store(cm + p, uint32_t(-1));
        });
        if (lb_load(rep + node) > id) atomicMin(rep + node, id);
        if ((e[r][K] & kUsedBit) && lb_load(cm + node) != uint32_t(kUsedMark)) lb_store(cm + node, uint32_t(kUsedMark));
      }
      a.pairs[p] = make_uint2(node, id);
    }
  }
  stores_in_l2();
  __syncthreads();
  if (tid == 0) {
    lb_store(rep + b0, s_x[2]);
    if (s_x[1]) lb_store(cm + b0, uint32_t(kUsedMark));
    stores_in_l2();
  }
  __syncthreads();
  // ---- one element per used group (the table is no longer needed)
  for (int64_t p = b0 + tid; p < b1; p += BLOCK) {
    if (a.pairs[p].x != uint32_t(p) || lb_load(cm + p) != uint32_t(kUsedMark)) continue;
    const int64_t u = upre + atomicAdd(&s_x[3], 1u);
    uint32_t e[S];
    load_words<S>(a.elems + p * S, e);
    e[K] = uint32_t(p);
    store_words<S>(a.uelems + u * S, e);
  }
  __syncthreads();
  return s_x[3];
}

// Merges the `listed` groups (record, name) of a large bucket's parts: of the
// names of one record one stays, with the smallest of their ids and the used
// mark if any is used, and cmap leads from the others to it. The chains'
// table lies in the bucket's elements, whose parts are all done. The elements
// of the used groups, whose number is returned, go to slots from `upre` on,
// at most to half of the bucket's, below the list.
template <int K, int BLOCK>
__device__ uint32_t merge_parts(const GroupArgs& a, const uint32_t* list, uint32_t listed, int64_t b0, int64_t upre,
                                uint32_t* s_x) {
  constexpr int S = K + 1;
  const int tid = threadIdx.x;
  uint32_t* const table = const_cast<uint32_t*>(a.elems) + b0 * S;
  uint32_t* const rep = a.rep;
  uint32_t* const cm = reinterpret_cast<uint32_t*>(a.cmap);
  for (uint32_t j = tid; j < listed; j += BLOCK) lb_store(table + int64_t(j) * S, 0xFFFFFFFFu);
  if (tid == 0) s_x[3] = 0;
  stores_in_l2();
  __syncthreads();
  for (uint32_t j = tid; j < listed; j += BLOCK) {
    uint32_t e[S];
    load_words<S>(list + int64_t(j) * S, e);
    const uint32_t node = chain_node<K>(table, list, listed, j, e, [] {});
    if (node == j) continue;
    const uint32_t name = list[int64_t(node) * S + K], id = lb_load(rep + e[K]);
    if (lb_load(rep + name) > id) atomicMin(rep + name, id);
    if (lb_load(cm + e[K]) == uint32_t(kUsedMark)) lb_store(cm + name, uint32_t(kUsedMark));
    lb_store(cm + e[K], uint32_t(lead_name(name)));
  }
  stores_in_l2();
  __syncthreads();
  for (uint32_t j = tid; j < listed; j += BLOCK) {
    uint32_t e[S];
    load_words<S>(list + int64_t(j) * S, e);
    if (lb_load(cm + e[K]) != uint32_t(kUsedMark)) continue;
    store_words<S>(a.uelems + (upre + atomicAdd(&s_x[3], 1u)) * S, e);
  }
  __syncthreads();
  return s_x[3];
}

template <int K, bool MESH>
__global__ __launch_bounds__(GroupShape<MESH ? K + 1 : K>::BLOCK, (group_min_waves<K, MESH>())) void k_group(
    GroupArgs a) {
  constexpr int KW = MESH ? K + 1 : K;  // key words
  using SH = GroupShape<KW>;
  constexpr int S = K + 1;              // words of an input element
  constexpr int KO = MESH ? 1 : 0;      // first record word of a key
  constexpr int BLOCK = SH::BLOCK, WIN = SH::WIN, CHUNK = SH::CHUNK, IPT = SH::IPT;
  constexpr int TS = SH::TS, TB = SH::TB;
  constexpr int WAVES = BLOCK / kWave;
  constexpr uint32_t kEmpty = 0xFFFFFFFFu;
  constexpr uint32_t kUsedBit = 0x80000000u;
  constexpr int kScratch = WIN > TS ? WIN : TS;

  __shared__ uint32_t s_keys[KW * WIN];     // window keys, word-major
  __shared__ uint32_t s_scratch[kScratch];  // buckets of the window, then the table
  __shared__ uint32_t s_cnt[2][IPT][WAVES];
  __shared__ uint32_t s_sq, s_eq, s_lq;
  __shared__ uint32_t s_big[2];

  const int tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const int64_t n = a.n;
  if (tid == 0) {
    s_sq = WIN;
    s_eq = WIN;
    s_lq = 0;
  }
  const uint32_t tile = blockIdx.x;
  const int64_t c0 = int64_t(tile) * CHUNK;
  const int64_t c1 = min(n, c0 + CHUNK);
  const int qc1 = int(c1 - c0) + 1;  // window slot of position c1

  // ---- window: positions c0 - 1 + q, q in [0, WIN). Each thread keeps, for
  // its own slots, the id (bit 31: referenced) and, until the table is
  // built, the record's hash in `slot`; everything else lives in LDS, so
  // that three workgroups fit on a CU.
  uint32_t ids[IPT], slot[IPT];
  // batches: mesh b's elements sit at sorted positions [mesh_off[b],
  // mesh_off[b+1]) (its buckets follow those of the meshes before it), so a
  // window inside one mesh needs one lookup, and otherwise a position's mesh
  // is looked up instead of its id's
  uint32_t win_mesh[2] = {0u, 1u};
  if constexpr (MESH) {
    const int64_t p0 = max(c0 - 1, int64_t(0)), p1 = min(c0 - 1 + WIN, n) - 1;
    if (p0 <= p1) {
      win_mesh[0] = __builtin_amdgcn_readfirstlane(mesh_of(a.mesh_off, a.nmesh, p0, a.mesh_tab));
      win_mesh[1] = __builtin_amdgcn_readfirstlane(mesh_of(a.mesh_off, a.nmesh, p1, a.mesh_tab));
    }
  }
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int q = i * BLOCK + tid;
    const int64_t pos = c0 - 1 + q;
    uint32_t e[S];
    if (pos >= 0 && pos < n) {
      load_words<S>(a.elems + pos * S, e);
    } else {
#pragma unroll
      for (int w = 0; w < S; ++w) e[w] = 0u;
    }
    uint32_t key[KW];
    if constexpr (MESH) {
      key[0] = (pos < 0 || pos >= n)            ? 0u
               : win_mesh[0] == win_mesh[1] ? win_mesh[0]
                                            : mesh_of(a.mesh_off, a.nmesh, pos, a.mesh_tab);
#pragma unroll
      for (int w = 0; w < K; ++w) key[w + 1] = e[w];
    } else {
#pragma unroll
      for (int w = 0; w < K; ++w) key[w] = e[w];
    }
#pragma unroll
    for (int w = 0; w < KW; ++w) s_keys[w * WIN + q] = key[w];
    ids[i] = e[K];
    slot[i] = hash_words<KW>(key);
    if constexpr (MESH)
      s_scratch[q] = mesh_bucket(a.mesh_buckets, key[0], slot[i]);
    else
      s_scratch[q] = slot[i] & a.bucket_mask;
  }
  __syncthreads();

  // ---- bucket starts: the first (sq) and last (lq) in the chunk and the first
  // at or after position c1 (eq; position n counts as one). A wave's slots are
  // neighbours, so its first and its last lane with one tell it (buckets of two
  // elements, every lane for itself: 0.74 ms instead of 0.52 for 36M vertices).
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int q = i * BLOCK + tid;
    const int64_t pos = c0 - 1 + q;
    const bool start =
        q > 0 && pos <= n && (pos == 0 || pos == n || s_scratch[q] != s_scratch[max(q, 1) - 1]);
    const uint64_t in = ballot(start && q < qc1), after = ballot(start && q >= qc1);
    if (in) {
      const int first = __ffsll((unsigned long long)in) - 1, last = 63 - __clzll((long long)in);
      if (lane == first) atomicMin(&s_sq, uint32_t(q));
      if (lane == last) atomicMax(&s_lq, uint32_t(q));
    }
    if (after && lane == __ffsll((unsigned long long)after) - 1) atomicMin(&s_eq, uint32_t(q));
  }
  __syncthreads();
  const int sq = int(s_sq);
  const bool active = sq < qc1;
  // the chunk's last bucket runs past the window: it is left to k_group_over
  const bool over = active && int(s_eq) >= WIN;
  const int eq = over ? int(s_lq) : int(s_eq);
  for (int i = tid; i < TS; i += BLOCK) s_scratch[i] = kEmpty;  // buckets are no longer needed
  __syncthreads();

  // ---- one table entry per distinct record of the owned span [sq, eq):
  // the smallest window slot holding it (its first copy), bit 31 = used
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int q = i * BLOCK + tid;
    const uint32_t h = slot[i];
    slot[i] = kEmpty;
    if (!active || q < sq || q >= eq) continue;
    uint32_t sl = (h * 0x9E3779B1u) >> (32 - TB);
    for (int probe = 0; probe < TS; ++probe) {
      uint32_t cur = s_scratch[sl];
      if (cur == kEmpty) {
        cur = atomicCAS(&s_scratch[sl], kEmpty, uint32_t(q));
        if (cur == kEmpty) {
          slot[i] = sl;
          break;
        }
      }
      if (lds_keys_equal<KW>(s_keys, int(cur & 0xFFFFu), q, WIN)) {
        atomicMin(&s_scratch[sl], uint32_t(q));
        slot[i] = sl;
        break;
      }
      sl = (sl + 1) & (TS - 1);
    }
  }
  __syncthreads();
  uint32_t headm = 0;  // bit i: slot i of this thread holds its group's first copy
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int q = i * BLOCK + tid;
    if (slot[i] == kEmpty) continue;
    if ((s_scratch[slot[i]] & 0xFFFFu) == uint32_t(q)) headm |= 1u << i;
    if (ids[i] & kUsedBit) atomicOr(&s_scratch[slot[i]], kUsedBit);
  }
  __syncthreads();

  // ---- number the groups (and the used ones) in window order: slot q =
  // i * BLOCK + tid, so round i of every wave precedes round i + 1
  uint32_t uheadm = 0;  // bit i: a head whose group is used
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const bool h = (headm >> i) & 1u;
    const bool uh = h && (s_scratch[slot[i]] & kUsedBit) != 0u;
    uheadm |= uh ? (1u << i) : 0u;
    const uint64_t hm = ballot(h);
    const uint64_t um = ballot(uh);
    if (lane == 0) {
      s_cnt[0][i][wave] = uint32_t(popc64(hm));
      s_cnt[1][i][wave] = uint32_t(popc64(um));
    }
  }
  __syncthreads();
  uint32_t gt = 0, ut = 0;  // totals of the window
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    uint32_t gb = gt, ub = ut;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const uint32_t cg = s_cnt[0][i][w], cu = s_cnt[1][i][w];
      if (w < wave) {
        gb += cg;
        ub += cu;
      }
      gt += cg;
      ut += cu;
    }
    const bool h = (headm >> i) & 1u;
    const uint64_t hm = ballot(h);
    const uint64_t um = ballot((uheadm >> i) & 1u);
    gb += uint32_t(popc64(hm & lanemask_lt()));
    ub += uint32_t(popc64(um & lanemask_lt()));
    // heads leave their group's rank (batches: their window slot) in the low
    // half and their used rank in the high half of the table entry for the
    // other copies; both are below WIN <= 2^16
    const uint32_t q = uint32_t(i * BLOCK + tid);
    if (h) s_scratch[slot[i]] = (MESH ? q : gb) | (ub << 16);
  }

  // names start at the span's first position (batches: the first copy's position)
  const uint32_t span0 = active ? uint32_t(c0 - 1 + sq) : 0u;
  __syncthreads();  // the ranks the heads left in the table are read below
  const uint32_t gpre = span0, upre = span0;

  // ---- outputs of the owned span
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    if (slot[i] == kEmpty) continue;
    const int q = i * BLOCK + tid;
    const int64_t pos = c0 - 1 + q;
    const uint32_t ranks = s_scratch[slot[i]];
    const uint32_t g = MESH ? uint32_t(c0 - 1) + (ranks & 0xFFFFu) : gpre + (ranks & 0xFFFFu);
    const uint32_t org = ids[i] & 0x7FFFFFFFu;
    if (int64_t(g) >= n || pos < 0 || pos >= n) {  // only after a failed wait
      atomicMax(a.status, 7 /* MRX_ERR_INTERNAL */);
      continue;
    }
    a.pairs[pos] = make_uint2(g, org);
    if (!((headm >> i) & 1u)) continue;
    if ((uheadm >> i) & 1u) {
      a.rep[g] = org;
      const uint32_t u = upre + (ranks >> 16);
      if (int64_t(u) >= n) {
        atomicMax(a.status, 7 /* MRX_ERR_INTERNAL */);
        continue;
      }
      uint32_t e[S];
#pragma unroll
      for (int w = 0; w < K; ++w) e[w] = s_keys[(w + KO) * WIN + q];
      e[K] = g;
      store_words<S>(a.uelems + int64_t(u) * S, e);
    } else {
      a.cmap[g] = -1;
    }
  }
  const uint32_t u_own = active ? ut : 0u;
  if (over) {
    const int64_t b0 = c0 - 1 + int(s_lq), b1 = end_of_bucket<K, MESH, BLOCK>(a, b0, s_big);
    const bool large = b1 - b0 > 2 * int64_t(a.part);
    if (tid == 0) {
      a.over[tile] = make_uint2(uint32_t(b0), uint32_t(b1));
      a.over_list[atomicAdd(a.over_count, 1u)] = tile;
      if (large) *a.over_any = 1;
    }
    if (large)
      for (int64_t w = b0 / a.part + 1 + tid; w * a.part < b1; w += BLOCK) a.over_at[w] = tile + 1;
  }
  // ---- the chunk's record and its share of its run's sum
  if (tid == 0) {
    a.chunks[tile] = make_uint2(span0, u_own);
    if (u_own) atomicAdd(&a.range_sums[group_run_of(tile, gridDim.x, a.ranges)], u_own);
  }
}

// Where there are too many vertices for the sample sort (split_kernels.hpp):
// totals of the grouping (every workgroup adds up the runs' sums; workgroup 0
// stores U), then the used groups' elements (slots span start + k of each
// chunk) packed densely into `dense` at the chunk's used-group offset, with
// every key digit of them added to the LDS histograms (flushed once per
// workgroup). A workgroup takes a run of consecutive chunks, whose elements
// are one contiguous stretch of `dense`; each thread maps its dense positions
// back to (chunk, slot) with a search over the run's offsets in LDS.
struct GroupCompactArgs {
  const uint32_t* sparse;     // [n][K+1]
  const uint2* chunks;
  const uint32_t* range_sums; // [ranges] (k_group)
  int64_t tiles;
  int64_t ranges;             // the grid
  int64_t n;
  uint32_t* dense;            // [U][K+1]
  uint32_t* hist;             // [P][2^D] global histograms
  Control* ctl;               // num_used, set here by workgroup 0
};

template <int K, int D, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_group_compact_hist(GroupCompactArgs a) {
  using DG = KeyDigits<K, D>;
  constexpr int S = K + 1;
  constexpr int P = DG::kPasses;
  constexpr int WORDS = P << D;
  // several items in flight per thread, but wide items one at a time: the
  // multi-item register layout of items wider than 4 words is the one that
  // miscounted histograms on the GPU (see items_per_group)
  constexpr int UNROLL = S <= 4 ? 4 : 1;
  constexpr int PER = kCompactMaxChunks / BLOCK;
  __shared__ uint32_t s_h[WORDS];
  __shared__ uint32_t s_base[kCompactMaxChunks + 1];
  __shared__ uint32_t s_span[kCompactMaxChunks];
  __shared__ uint32_t s_wave[BLOCK / kWave];
  const int tid = threadIdx.x;
  const int64_t w = blockIdx.x;
  // the used groups of all runs, and of those before this one
  uint32_t used = 0, before = 0;
  for (int64_t r = tid; r < a.ranges; r += BLOCK) {
    const uint32_t ur = a.range_sums[r];
    used += ur;
    before += r < w ? ur : 0u;
  }
  uint32_t total_used, first;
  (void)block_exclusive_scan<BLOCK>(used, s_wave, &total_used);
  (void)block_exclusive_scan<BLOCK>(before, s_wave, &first);
  if (w == 0 && tid == 0) a.ctl->num_used = int64_t(total_used);
  const int64_t t0 = group_range_start(w, a.tiles, a.ranges);
  const int64_t t1 = group_range_start(w + 1, a.tiles, a.ranges);
  const int nc = int(t1 - t0);  // <= kCompactMaxChunks (group_compact_ranges)
  // the run's chunks: offsets (exclusive prefix of their used counts) and span starts
  uint32_t cnt[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = tid * PER + j;
    uint2 c = make_uint2(0, 0);
    if (i < nc) c = a.chunks[t0 + i];
    cnt[j] = c.y;
    sum += c.y;
    if (i < nc) s_span[i] = c.x;
  }
  uint32_t run_total;
  const uint32_t ex = block_exclusive_scan<BLOCK>(sum, s_wave, &run_total);
  uint32_t acc = first + ex;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int i = tid * PER + j;
    if (i < nc) s_base[i] = acc;
    acc += cnt[j];
  }
  const uint32_t end = first + run_total;
  if (tid == 0) s_base[nc] = end;
  zero_histograms<WORDS, BLOCK>(s_h);  // synchronises
  uint32_t last[P], run[P];
#pragma unroll
  for (int p = 0; p < P; ++p) { last[p] = 0; run[p] = 0; }
  const uint32_t total = end - first;
  for (uint32_t j0 = 0; j0 < total; j0 += BLOCK * UNROLL) {
    uint32_t e[UNROLL][S];
    uint32_t pos[UNROLL];
#pragma unroll
    for (int r = 0; r < UNROLL; ++r) {
      const uint32_t j = j0 + uint32_t(r * BLOCK + tid);
      pos[r] = first + j;
      if (j < total) {
        // chunk of dense position first + j: the last c with s_base[c] <= it
        int lo = 0, hi = nc - 1;
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (s_base[mid] <= pos[r]) lo = mid; else hi = mid - 1;
        }
        const uint32_t slot = s_span[lo] + (pos[r] - s_base[lo]);
        load_words<S>(a.sparse + int64_t(slot) * S, e[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < UNROLL; ++r) {
      if (j0 + uint32_t(r * BLOCK + tid) >= total) continue;
      store_words<S>(a.dense + int64_t(pos[r]) * S, e[r]);
      hist_item<DG, D>(e[r], s_h, last, run);
    }
  }
#pragma unroll
  for (int p = 0; p < P; ++p)
    if (run[p]) atomicAdd(&s_h[p * (1 << D) + last[p]], run[p]);
  flush_histograms<WORDS, BLOCK>(s_h, a.hist);
}

// Plan of the LSD key sort that follows the packing: it reads buf[0], which
// holds the packed elements; passes whose digit is the same for every element
// (dead, from the bucket scan) are skipped. One thread.
static __global__ void k_group_sort_plan(SortBuffers b) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  const uint32_t* dead = b.plan + b.passes + 1;
  uint32_t in = 0u;
  for (int p = 0; p < b.passes; ++p) {
    const bool skip = dead[p] != 0u;
    b.plan[p] = in | (skip ? 2u : 0u);
    if (!skip) in ^= 1u;
  }
  b.plan[b.passes] = in;
}

// After an LSD key sort of the used groups: sorted position c is output
// vertex c (Section 2, Step 3 compacts the sorted array). Writes the record,
// cmap[group] = c, U, and for one mesh the representative: gathered here it
// takes 0.18 ms for the 13.3M used values of an 80M-vertex mesh, where finding
// them among the pairs takes 0.72 longer in the scatter of the map.
struct FinalizeArgs {
  SortBuffers bufs;        // sorted(): [U][K+1] (record, group name)
  int32_t* cmap;           // [n]
  uint32_t* out_vtx;       // [U][K]
  const uint32_t* rep;     // [n]
  int32_t* new2old;        // [U], nullable
  int64_t* out_num;        // nullable
  int64_t cap;             // n
  Control* ctl;
  int32_t* status;
};

template <int K>
__global__ __launch_bounds__(256) void k_group_finalize(FinalizeArgs a) {
  constexpr int S = K + 1;
  const int64_t u = a.ctl->num_used;
  if (blockIdx.x == 0 && threadIdx.x == 0 && a.out_num) *a.out_num = u;
  const uint32_t* sorted = a.bufs.sorted();
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t c = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; c < u && c < a.cap; c += stride) {
    uint32_t e[S];
    load_words<S>(sorted + c * S, e);
#pragma unroll
    for (int w = 0; w < K; ++w) a.out_vtx[c * K + w] = e[w];
    const uint32_t g = e[K];
    if (int64_t(g) >= a.cap) {
      atomicMax(a.status, 7 /* MRX_ERR_INTERNAL */);
      continue;
    }
    a.cmap[g] = int32_t(c);
    if (a.new2old) a.new2old[c] = int32_t(a.rep[g]);
  }
}

}  // namespace mrx
