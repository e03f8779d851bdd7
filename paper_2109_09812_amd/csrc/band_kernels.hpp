// Steps 1 and 4 of a mesh, or of a batch, by vertex bands.
//
// The used marking (Section 2, Step 1), the old2new map and the index remap
// (Step 4) each touch one vertex-indexed table at scattered positions. On
// gfx950 every scattered store costs one fabric request however few bytes it
// writes, and every scattered load fetches a 128-byte line, so these steps
// run at the fabric's request rate. Here the vertex range is cut into bands
// of 2^shift vertices, each small enough that a workgroup holds the band's
// part of the table in LDS, and the index entries and the (group, vertex)
// pairs are first grouped by band:
//  * k_band_partition: a tile of kBandTile index entries groups its valid
//    entries by band in LDS and writes them, band after band, into its own
//    slot part[tile * kBandTile, ...); table[band][tile] = offset << 16 |
//    count within the slot. With positions kept, an entry is
//    pos << kPosShift | (vertex - band start), pos its place in the tile.
//  * k_band_mark: one workgroup per band sets the referenced vertices' bits
//    in an LDS bitmap and writes every flag of the band, 0 or 1, with
//    16-byte stores.
//  * k_pair_partition: the same grouping for the (group, vertex) pairs of
//    Step 3, each carrying the new id of its group: (new id, vertex - band
//    start).
//  * k_band_map: one workgroup per band builds the band's slice of old2new
//    in LDS from its pairs, writes it out whole, then looks up the new id of
//    every index entry of the band and stores it at the entry's slot.
//  * k_band_remap: one workgroup per index tile puts the new ids of its slot
//    back in entry order in LDS and writes its part of out_idx.
// All reads and writes of these kernels are whole runs of a tile slot or a
// band, except the per-(band, tile) slices of the partitions (tens of
// entries each on the meshes this is chosen for).
#pragma once

#include "device_common.hpp"

namespace mrx {

constexpr int kBandBlock = 1024;                    // k_band_map, k_band_remap
constexpr int kIdxPartBlock = 512;                  // index partition
constexpr int kIdxPartItems = 64;
constexpr int kBandTile = kIdxPartBlock * kIdxPartItems;  // 32768 entries: offsets and counts fit 16 bits
constexpr int kMaxBands = 1024;
constexpr int kPairBlock = 1024;  // 512 threads of 32 pairs: 0.204 against 0.197 ms for 26.4M pairs
constexpr int kPairItems = 16;
constexpr int kPairTile = kPairBlock * kPairItems;  // 16384 pairs (128 KB staged)
// Up to some million entries, tiles of a quarter of that: the partitions and
// the remap of 4.2M entries would otherwise run on 128 workgroups, half the
// GPU, one to a CU (index partition of 4.2M entries 44 -> 23 us).
constexpr int kFineIdxItems = 16, kFineBandTile = kIdxPartBlock * kFineIdxItems;
constexpr int kFinePairBlock = 512, kFinePairItems = 8, kFinePairTile = kFinePairBlock * kFinePairItems;
constexpr int kMinBandShift = 12;                   // bands start 16-byte aligned
constexpr int kMinFineShift = 8;
constexpr int kMaxMarkShift = 19;                   // a band's bitmap: at most 64 KB
constexpr int kMaxMapShift = 15;                    // a band's old2new slice: 128 KB
constexpr int kPosShift = 17;                       // entry = pos << 17 | vertex - band start
constexpr int kBandErrIndex = 3;                    // MRX_ERR_INDEX_OUT_OF_RANGE
constexpr int kBandErrInternal = 7;                 // MRX_ERR_INTERNAL

struct BandArgs {
  const int32_t* idx;          // [m] index entries (may be the memory `part` points to)
  int64_t m;                   // capacity in entries (num_elems * arity)
  int32_t arity;
  int64_t n;                   // vertices
  const int64_t* live_elems;   // device, nullable: only the first *live_elems elements count
  int32_t shift;               // band of vertex v = v >> shift
  int32_t nb;                  // ceil(n / 2^shift) <= kMaxBands
  int32_t vec;                 // idx is 16-byte aligned
  int32_t keep_pos;            // entries carry their position in the tile (shift <= kPosShift)
  int64_t tiles;               // ceil(m / tile size)
  int32_t fine;                // tiles of kFineBandTile entries instead of kBandTile
  uint32_t* part;              // [m]
  uint32_t* table;             // [nb][tiles]
  uint32_t* tile_valid;        // [tiles], nullable: valid entries of each tile
  uint8_t* used;               // [n], 16-byte aligned
  int32_t* status;
  // batches: entries are mesh-local; vertex and element offsets [nmesh + 1]
  // and the bucket table of the latter (mesh_of)
  const int64_t* vtx_off;
  const int64_t* elem_off;
  const int32_t* elem_tab;
  int32_t nmesh;
};

__device__ __forceinline__ int64_t live_entries(const int64_t* live_elems, int64_t m, int32_t arity) {
  return live_elems ? min(m, *live_elems * arity) : m;
}

template <int ITEMS, bool BATCHED>
__global__ __launch_bounds__(kIdxPartBlock) void k_band_partition(BandArgs a) {
  constexpr int B = kIdxPartBlock, kBandTile = B * ITEMS;
  static_assert(ITEMS % 4 == 0, "entries are loaded four at a time");
  static_assert(kBandTile <= (1 << (32 - kPosShift)), "positions fit above the vertex offset");
  __shared__ uint32_t s_cnt[kMaxBands];
  __shared__ uint32_t s_off[kMaxBands];
  __shared__ uint32_t s_stage[kBandTile];
  __shared__ uint32_t s_wave[B / kWave];
  const int tid = threadIdx.x;
  for (int b = tid; b < kMaxBands; b += B) s_cnt[b] = 0;
  __syncthreads();
  const int64_t m = live_entries(a.live_elems, a.m, a.arity);
  const int64_t tile = blockIdx.x;
  const int64_t base = tile * kBandTile;
  // entry 4 * (i * B + tid) + c of the tile goes to v[4 * i + c]
  int32_t v[ITEMS];
  if (a.vec && base + kBandTile <= m) {
    const int4* p = reinterpret_cast<const int4*>(a.idx + base);
#pragma unroll
    for (int i = 0; i < ITEMS / 4; ++i) {
      const int4 q = stream_load(p + i * B + tid);
      v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < ITEMS / 4; ++i)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t k = base + 4 * (int64_t(i) * B + tid) + c;
        v[4 * i + c] = k < m ? stream_load(a.idx + k) : -1;
      }
  }
  bool bad = false;
  int64_t first = 0, count = a.n;  // vertex range of the entries' mesh
  bool one_mesh = true;
  if constexpr (BATCHED) {
    // one lookup for a tile inside one mesh
    const int64_t e0 = base / a.arity, e1 = (min(base + kBandTile, m) - 1) / a.arity;
    const uint32_t b0 = mesh_of(a.elem_off, a.nmesh, e0, a.elem_tab), b1 = mesh_of(a.elem_off, a.nmesh, e1, a.elem_tab);
    one_mesh = b0 == b1;
    first = a.vtx_off[b0];
    count = a.vtx_off[b0 + 1] - first;
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const int64_t k = base + 4 * (int64_t(i / 4) * B + tid) + (i % 4);
    if constexpr (BATCHED) {
      if (k < m) {
        if (!one_mesh) {
          const uint32_t b = mesh_of(a.elem_off, a.nmesh, uint32_t(k) / uint32_t(a.arity), a.elem_tab);
          first = a.vtx_off[b];
          count = a.vtx_off[b + 1] - first;
        }
        v[i] = v[i] >= 0 && int64_t(v[i]) < count && first >= 0 ? int32_t(first + v[i]) : -1;
      }
    }
    if (k < m && (v[i] < 0 || int64_t(v[i]) >= a.n)) {
      bad = true;
      v[i] = -1;
    }
  }
  if (bad) atomicMax(a.status, kBandErrIndex);
  uint32_t r[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (v[i] >= 0) r[i] = atomicAdd(&s_cnt[v[i] >> a.shift], 1u);
  __syncthreads();
  constexpr int PER = kMaxBands / B;
  uint32_t loc[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    loc[j] = sum;
    sum += s_cnt[tid * PER + j];
  }
  uint32_t valid;
  const uint32_t ex = block_exclusive_scan<B>(sum, s_wave, &valid);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = tid * PER + j;
    s_off[b] = ex + loc[j];
    if (b < a.nb) a.table[size_t(b) * size_t(a.tiles) + size_t(tile)] = ((ex + loc[j]) << 16) | s_cnt[b];
  }
  if (tid == 0 && a.tile_valid) a.tile_valid[tile] = valid;
  __syncthreads();
  const uint32_t mask = (1u << a.shift) - 1u;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (v[i] >= 0) {
      const uint32_t pos = 4u * uint32_t((i / 4) * B + tid) + uint32_t(i % 4);
      const uint32_t local = uint32_t(v[i]) & mask;
      s_stage[s_off[uint32_t(v[i]) >> a.shift] + r[i]] = a.keep_pos ? (pos << kPosShift) | local : local;
    }
  __syncthreads();
  for (uint32_t j = tid; j < valid; j += B) stream_store(a.part + base + j, s_stage[j]);
}

__device__ __forceinline__ uint32_t spread_bits4(uint32_t x) {  // bit i -> byte i (i < 4)
  return (x & 1u) | ((x & 2u) << 7) | ((x & 4u) << 14) | ((x & 8u) << 21);
}

// Walks the band's row of a partition table: fn(entry, place) for every entry
// of the band. Slices are `tile_size` apart; word positions fit 32 bits
// (fewer than 2^31 entries). The slices of BLOCK tiles at a time are cut into
// units of up to 16 entries, listed in LDS, and every 16 lanes take a unit,
// BATCH of them in flight: the work is spread evenly whether the entries are
// scattered (tens of entries in every slice) or in order (nearly all of a
// band's entries in one or two slices). With one wave per slice and 64 slices
// per wave, 160 tiles kept 3 of 16 waves busy and long slices one: 0.13 ms to
// mark and 0.13 ms to map the 5.4M ordered entries of a 1M-vertex mesh, which
// take 0.033 (with the hash histograms) and 0.018 ms now; the map of the 25M
// scattered entries of a 26.4M-vertex soup 0.22 -> 0.18 ms.
template <int BLOCK>
struct BandWalk {
  static constexpr int UNITS = 4 * BLOCK;
  uint32_t unit[UNITS];  // slice | number of the unit in it << 10
  uint32_t at[BLOCK];    // first entry of a slice
  uint32_t cnt[BLOCK];
  uint32_t wave[BLOCK / kWave];
};

template <int BLOCK, int BATCH, class Load, class Fn>
__device__ __forceinline__ void for_band_entries(const uint32_t* __restrict__ row, int64_t tiles, int tile_size,
                                                 BandWalk<BLOCK>& w, Load load, Fn fn) {
  static_assert(BLOCK <= 1024, "slices are numbered in 10 bits");
  constexpr int UNITS = BandWalk<BLOCK>::UNITS, GROUPS = BLOCK / 16;
  const int tid = threadIdx.x, lane = lane_id();
  for (int64_t t0 = 0; t0 < tiles; t0 += BLOCK) {
    const uint32_t e = t0 + tid < tiles ? row[t0 + tid] : 0u;
    const uint32_t cnt = e & 0xFFFFu;
    const int units = int((cnt + 15) >> 4);
    uint32_t total;
    const int first = int(block_exclusive_scan<BLOCK>(uint32_t(units), w.wave, &total));
    w.at[tid] = uint32_t(t0 + tid) * uint32_t(tile_size) + (e >> 16);
    w.cnt[tid] = cnt;
    for (int w0 = 0; w0 < int(total); w0 += UNITS) {
      if (w0 > 0) __syncthreads();  // the units before are done
      const int lo = max(first, w0), hi = min(first + units, w0 + UNITS);
      if (units <= 4) {
        for (int k = lo; k < hi; ++k) w.unit[k - w0] = uint32_t(tid) | uint32_t(k - first) << 10;
      }
      for (uint64_t many = ballot(units > 4 && lo < hi); many; many &= many - 1) {
        const int src = __ffsll((unsigned long long)many) - 1;
        const int l = __shfl(lo, src), h = __shfl(hi, src), f = __shfl(first, src);
        const uint32_t slice = uint32_t(tid - lane + src);
        for (int k = l + lane; k < h; k += kWave) w.unit[k - w0] = slice | uint32_t(k - f) << 10;
      }
      __syncthreads();
      const int nu = min(int(total) - w0, UNITS);
      for (int u0 = 0; u0 < nu; u0 += GROUPS * BATCH) {
        uint32_t at[BATCH];
        bool ok[BATCH];
        decltype(load(0u)) x[BATCH];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {  // unconditional loads, all in flight at once
          const int u = u0 + b * GROUPS + (tid >> 4);
          const uint32_t c = w.unit[min(u, nu - 1)];
          const uint32_t in = (c >> 10) * 16 + uint32_t(tid & 15), n = w.cnt[c & 1023u];
          ok[b] = u < nu && in < n;
          at[b] = w.at[c & 1023u] + min(in, n - 1);
          x[b] = load(at[b]);
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b)
          if (ok[b]) fn(x[b], at[b]);
      }
    }
  }
  __syncthreads();
}

// One band of k_band_mark; s_bits holds (1 << shift) / 32 words of LDS.
template <int BLOCK>
__device__ __forceinline__ void band_mark_body(const BandArgs& a, int64_t band, uint32_t* s_bits,
                                               BandWalk<BLOCK>& walk) {
  const int tid = threadIdx.x;
  const int words = (1 << a.shift) / 32;
  for (int w = tid; w < words; w += BLOCK) s_bits[w] = 0;
  __syncthreads();
  const int64_t lo = band << a.shift;
  const uint32_t mask = (1u << a.shift) - 1u;
  const uint32_t* part = a.part;
  for_band_entries<BLOCK, 8>(
      a.table + size_t(band) * size_t(a.tiles), a.tiles, a.fine ? kFineBandTile : kBandTile, walk,
      [&](uint32_t at) { return stream_load(part + at); },
      [&](uint32_t e, uint32_t) {
        const uint32_t l = e & mask;
        atomicOr(&s_bits[l >> 5], 1u << (l & 31));
      });
  __syncthreads();
  const int64_t hi = min(a.n, lo + (int64_t(1) << a.shift));
  for (int64_t q = lo + int64_t(tid) * 16; q < hi; q += int64_t(BLOCK) * 16) {
    const uint32_t w = (s_bits[(q - lo) >> 5] >> ((q - lo) & 31)) & 0xFFFFu;
    if (q + 16 <= hi) {
      const uint4 o = {spread_bits4(w), spread_bits4(w >> 4), spread_bits4(w >> 8), spread_bits4(w >> 12)};
      stream_store(reinterpret_cast<uint4*>(a.used + q), o);
    } else {
      for (int64_t t = q; t < hi; ++t) a.used[t] = uint8_t((w >> (t - q)) & 1u);
    }
  }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_band_mark(BandArgs a) {
  extern __shared__ uint32_t s_bits[];
  __shared__ BandWalk<BLOCK> s_walk;
  band_mark_body<BLOCK>(a, blockIdx.x, s_bits, s_walk);
}

// Buffers of the sort-all path are decided on the device: with from_sort
// set, the pairs are read from sort.spare() and the partition is written
// into sort.sorted() (free once the flag scan has run) instead of the plain
// pointers.
struct PairPartArgs {
  const uint2* pairs;          // [n] (group, vertex) pairs of Step 3
  const int32_t* cmap;         // [G] new id of each group, negative if the group is unused (after hash grouping
                               // -1, or led_name)
  int64_t n;
  int32_t shift;
  int32_t nb;
  int64_t tiles;               // ceil(n / tile size)
  uint2* part;                 // [n] (new id or -1, vertex - band start)
  uint32_t* table;             // [nb][tiles]
  int32_t* status;
  const uint32_t* rep;         // [n] representative of each used group, by name
  int32_t* new2old;            // nullable (hash grouping): receives them, at the groups' new ids
  const uint32_t* large;       // null after sort-all; not 0: there were large buckets (led_name)
  SortBuffers sort;
  int32_t from_sort;
  // batches: new ids and representatives become mesh-local (a pair's mesh is
  // that of its position, see k_scatter_old2new)
  const int64_t* vtx_off;
  const int64_t* out_off;
  const int32_t* vtx_tab;
  int32_t nmesh;
};

// The group ids of a tile of pairs are clustered (sorted, or grouped by
// hash bucket), so the cmap reads hit cache lines other lanes fetched.
template <int BLOCK, int kPairItems, bool BATCHED>
__global__ __launch_bounds__(BLOCK) void k_pair_partition(PairPartArgs a) {
  constexpr int kPairTile = BLOCK * kPairItems;
  __shared__ uint32_t s_cnt[kMaxBands];
  __shared__ uint32_t s_off[kMaxBands];
  __shared__ uint2 s_stage[kPairTile];
  __shared__ uint32_t s_wave[BLOCK / kWave];
  const int tid = threadIdx.x;
  for (int b = tid; b < kMaxBands; b += BLOCK) s_cnt[b] = 0;
  __syncthreads();
  const bool led = a.large && *a.large != 0;  // requested before the pairs
  const uint2* pairs = a.from_sort ? reinterpret_cast<const uint2*>(a.sort.spare()) : a.pairs;
  uint2* out = a.from_sort ? reinterpret_cast<uint2*>(a.sort.sorted()) : a.part;
  const int64_t tile = blockIdx.x;
  const int64_t base = tile * kPairTile;
  // every load unconditional (clamped positions), so that all of them are
  // in flight at once: first the pairs, then the new ids of their groups
  const uint32_t last = uint32_t(a.n - 1);
  uint2 p[kPairItems];
#pragma unroll
  for (int i = 0; i < kPairItems; ++i)
    p[i] = stream_load(pairs + min(uint32_t(base + int64_t(i) * BLOCK + tid), last));
  int32_t val[kPairItems];
#pragma unroll
  for (int i = 0; i < kPairItems; ++i) val[i] = a.cmap[min(p[i].x, last)];
  // representatives: the pair of one takes its group's place in new2old (the
  // entry is 0xFFFFFFFF for all other pairs)
  uint32_t at[kPairItems];
#pragma unroll
  for (int i = 0; i < kPairItems; ++i) {
    at[i] = 0xFFFFFFFFu;
    if (a.new2old) at[i] = a.rep[min(p[i].x, last)];
  }
  if (led) {
    // names that lead to another of their group
#pragma unroll
    for (int i = 0; i < kPairItems; ++i) {
      if (val[i] >= -1 || p[i].x > last) continue;
      p[i].x = led_name(val[i]);
      val[i] = a.cmap[min(p[i].x, last)];
      if (a.new2old) at[i] = a.rep[min(p[i].x, last)];
    }
  }
  uint32_t vtx[kPairItems];
  bool bad = false;
  int64_t out0 = 0, vtx0 = 0;  // output and vertex offsets of the pairs' mesh
  bool one_mesh = true;
  if constexpr (BATCHED) {
    const uint32_t b0 = mesh_of(a.vtx_off, a.nmesh, base, a.vtx_tab);
    const uint32_t b1 = mesh_of(a.vtx_off, a.nmesh, min(base + kPairTile, a.n) - 1, a.vtx_tab);
    one_mesh = b0 == b1;
    out0 = a.out_off[b0];
    vtx0 = a.vtx_off[b0];
  }
#pragma unroll
  for (int i = 0; i < kPairItems; ++i) {
    const int64_t k = base + int64_t(i) * BLOCK + tid;
    const bool ok = p[i].x <= last && p[i].y <= last;
    if (k < a.n && !ok) bad = true;  // only after a failed wait
    vtx[i] = k < a.n && ok ? p[i].y : 0xFFFFFFFFu;
    if constexpr (BATCHED) {
      if (!one_mesh && k < a.n) {
        const uint32_t b = mesh_of(a.vtx_off, a.nmesh, k, a.vtx_tab);
        out0 = a.out_off[b];
        vtx0 = a.vtx_off[b];
      }
    }
    at[i] = at[i] == p[i].y && k < a.n && ok && uint32_t(val[i]) <= last ? uint32_t(val[i]) : 0xFFFFFFFFu;
    p[i].y -= uint32_t(vtx0);
    if constexpr (BATCHED) val[i] = val[i] < 0 ? -1 : int32_t(val[i] - out0);
  }
  if (bad) atomicMax(a.status, kBandErrInternal);
  uint32_t r[kPairItems];
#pragma unroll
  for (int i = 0; i < kPairItems; ++i)
    if (vtx[i] != 0xFFFFFFFFu) r[i] = atomicAdd(&s_cnt[vtx[i] >> a.shift], 1u);
  __syncthreads();
  constexpr int PER = kMaxBands / BLOCK;
  uint32_t loc[PER], sum = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    loc[j] = sum;
    sum += s_cnt[tid * PER + j];
  }
  uint32_t valid;
  const uint32_t ex = block_exclusive_scan<BLOCK>(sum, s_wave, &valid);
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int b = tid * PER + j;
    s_off[b] = ex + loc[j];
    if (b < a.nb) a.table[size_t(b) * size_t(a.tiles) + size_t(tile)] = ((ex + loc[j]) << 16) | s_cnt[b];
  }
  __syncthreads();
  const uint32_t mask = (1u << a.shift) - 1u;
#pragma unroll
  for (int i = 0; i < kPairItems; ++i)
    if (vtx[i] != 0xFFFFFFFFu)
      s_stage[s_off[vtx[i] >> a.shift] + r[i]] = make_uint2(uint32_t(val[i] < 0 ? -1 : val[i]), vtx[i] & mask);
  __syncthreads();
  for (uint32_t j = tid; j < valid; j += BLOCK) stream_store(out + base + j, s_stage[j]);
  // scattered, so last: nothing waits behind them
#pragma unroll
  for (int i = 0; i < kPairItems; ++i)
    if (at[i] != 0xFFFFFFFFu) a.new2old[at[i]] = int32_t(p[i].y);
}

struct BandMapArgs {
  const uint2* ppart;          // pair partition
  const uint32_t* ptable;
  int64_t ptiles;
  const uint32_t* ipart;       // index partition (entries with positions)
  const uint32_t* itable;
  int64_t itiles;
  int64_t n;
  int32_t shift;               // <= kMaxMapShift
  int32_t nb;
  int32_t* old2new;            // [n]
  int32_t* values;             // [m]: new id of the entry at the same place in ipart
  SortBuffers sort;            // with from_sort: ppart = sort.sorted(), values = sort.spare()
  int32_t from_sort;
};

template <int kBandBlock, int SHIFT, bool FINE>
__global__ __launch_bounds__(kBandBlock) void k_band_map(BandMapArgs a) {
  __shared__ alignas(16) int32_t s_map[1 << SHIFT];  // a.shift <= SHIFT
  __shared__ BandWalk<kBandBlock> s_walk;
  const int tid = threadIdx.x;
  // the slices of neighbouring bands are neighbours in every tile's slot and
  // share its cache lines
  const int64_t band = die_tile(blockIdx.x, a.nb);
  if (band < 0) return;
  const int64_t lo = band << a.shift;
  const int64_t hi = min(a.n, lo + (int64_t(1) << a.shift));
  const int len = int(hi - lo);
  // vertices whose pair went missing (only after a failed wait) map to -1
  for (int i = tid; i < len; i += kBandBlock) s_map[i] = -1;
  __syncthreads();
  const uint2* ppart = a.from_sort ? reinterpret_cast<const uint2*>(a.sort.sorted()) : a.ppart;
  for_band_entries<kBandBlock, 8>(
      a.ptable + size_t(band) * size_t(a.ptiles), a.ptiles, FINE ? kFinePairTile : kPairTile, s_walk,
      [&](uint32_t at) { return stream_load(ppart + at); },
      [&](uint2 p, uint32_t) { s_map[p.y] = int32_t(p.x); });
  int32_t* out = a.old2new + lo;
  if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) {
    for (int i = 4 * tid; i < len; i += 4 * kBandBlock) {
      if (i + 4 <= len) {
        stream_store(reinterpret_cast<int4*>(out + i), make_int4(s_map[i], s_map[i + 1], s_map[i + 2], s_map[i + 3]));
      } else {
        for (int t = i; t < len; ++t) out[t] = s_map[t];
      }
    }
  } else {
    for (int i = tid; i < len; i += kBandBlock) out[i] = s_map[i];
  }
  const uint32_t mask = (1u << a.shift) - 1u;
  const uint32_t* ipart = a.ipart;
  int32_t* values = a.from_sort ? reinterpret_cast<int32_t*>(a.sort.spare()) : a.values;
  for_band_entries<kBandBlock, 8>(
      a.itable + size_t(band) * size_t(a.itiles), a.itiles, FINE ? kFineBandTile : kBandTile, s_walk,
      [&](uint32_t at) { return stream_load(ipart + at); },
      [&](uint32_t e, uint32_t at) { stream_store(values + at, s_map[e & mask]); });
}

struct BandRemapArgs {
  const uint32_t* ipart;       // index partition (may be out_idx itself)
  const int32_t* values;       // new ids in ipart's layout
  const uint32_t* tile_valid;  // [tiles]
  int64_t m;
  int32_t arity;
  const int64_t* live_elems;   // device, nullable
  int32_t* out_idx;            // [m]
  SortBuffers sort;            // with from_sort: values = sort.spare()
  int32_t from_sort;
};

// Entries dropped by the partition (out of range) come out as -1.
template <int kBandBlock, int kBandTile>
__global__ __launch_bounds__(kBandBlock) void k_band_remap(BandRemapArgs a) {
  __shared__ int32_t s_out[kBandTile];
  const int tid = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const int64_t base = tile * kBandTile;
  for (int j = tid; j < kBandTile; j += kBandBlock) s_out[j] = -1;
  __syncthreads();
  const uint32_t valid = a.tile_valid[tile];
  const int32_t* values = a.from_sort ? reinterpret_cast<const int32_t*>(a.sort.spare()) : a.values;
  if (valid > 0) {
    // unconditional loads (clamped positions), all in flight at once
    constexpr int PER = kBandTile / kBandBlock;
    uint32_t e[PER];
    int32_t x[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t j = min(uint32_t(i * kBandBlock + tid), valid - 1);
      e[i] = a.ipart[base + j];
      x[i] = stream_load(values + base + j);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (uint32_t(i * kBandBlock + tid) < valid) s_out[e[i] >> kPosShift] = x[i];
  }
  __syncthreads();  // every read of this tile's slot precedes the writes below
  const int64_t m = live_entries(a.live_elems, a.m, a.arity);
  const int len = int(min(int64_t(kBandTile), m - base));
  for (int j = tid; j < len; j += kBandBlock) stream_store(a.out_idx + base + j, s_out[j]);
}

// Launches, each with the block shape its kernel is written for.
static inline void launch_band_partition(const BandArgs& a, hipStream_t s) {
  if (a.tiles <= 0) return;
  if (a.nmesh > 0)
    hipLaunchKernelGGL((k_band_partition<kFineIdxItems, true>), dim3(a.tiles), dim3(kIdxPartBlock), 0, s, a);
  else if (a.fine)
    hipLaunchKernelGGL((k_band_partition<kFineIdxItems, false>), dim3(a.tiles), dim3(kIdxPartBlock), 0, s, a);
  else
    hipLaunchKernelGGL((k_band_partition<kIdxPartItems, false>), dim3(a.tiles), dim3(kIdxPartBlock), 0, s, a);
}

// Small bands (Step 4 follows): many short workgroups; large bands: few,
// each reading many entries.
static inline void launch_band_mark(const BandArgs& a, bool small_bands, hipStream_t s) {
  const size_t bits_lds = (size_t(1) << a.shift) / 8;
  if (small_bands)
    hipLaunchKernelGGL(k_band_mark<256>, dim3(a.nb), dim3(256), bits_lds, s, a);
  else
    hipLaunchKernelGGL(k_band_mark<1024>, dim3(a.nb), dim3(1024), bits_lds, s, a);
}

static inline void launch_pair_partition(const PairPartArgs& a, bool fine, hipStream_t s) {
  if (a.tiles <= 0) return;
  if (a.nmesh > 0)
    hipLaunchKernelGGL((k_pair_partition<kFinePairBlock, kFinePairItems, true>), dim3(a.tiles), dim3(kFinePairBlock), 0, s, a);
  else if (fine)
    hipLaunchKernelGGL((k_pair_partition<kFinePairBlock, kFinePairItems, false>), dim3(a.tiles), dim3(kFinePairBlock), 0, s, a);
  else
    hipLaunchKernelGGL((k_pair_partition<kPairBlock, kPairItems, false>), dim3(a.tiles), dim3(kPairBlock), 0, s, a);
}

// Fine bands hold at most 2^14 vertices, in 32 or 64 KB of LDS, so that
// several of their workgroups share a CU.
constexpr int kMaxFineShift = 14;
static inline void launch_band_map(const BandMapArgs& a, bool fine, hipStream_t s) {
  const dim3 nb(die_grid(a.nb));
  if (fine && a.shift <= 13)
    hipLaunchKernelGGL((k_band_map<512, 13, true>), nb, dim3(512), 0, s, a);
  else if (fine && a.shift <= kMaxFineShift)
    hipLaunchKernelGGL((k_band_map<512, kMaxFineShift, true>), nb, dim3(512), 0, s, a);
  else if (fine)
    hipLaunchKernelGGL((k_band_map<kBandBlock, kMaxMapShift, true>), nb, dim3(kBandBlock), 0, s, a);
  else
    hipLaunchKernelGGL((k_band_map<kBandBlock, kMaxMapShift, false>), nb, dim3(kBandBlock), 0, s, a);
}

static inline void launch_band_remap(const BandRemapArgs& a, int64_t tiles, bool fine, hipStream_t s) {
  if (tiles <= 0) return;
  if (fine)
    hipLaunchKernelGGL((k_band_remap<512, kFineBandTile>), dim3(tiles), dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((k_band_remap<kBandBlock, kBandTile>), dim3(tiles), dim3(kBandBlock), 0, s, a);
}

}  // namespace mrx
