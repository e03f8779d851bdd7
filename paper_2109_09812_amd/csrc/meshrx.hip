// meshrx C ABI: argument validation, workspace layout and the launch
// sequence of the re-indexing pipeline (Section 2, Steps 1-4), plus the
// attribute gather and its backward.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <vector>

#include "../../include/meshrx.h"
#include "band_kernels.hpp"
#include "edit_kernels.hpp"
#include "mesh_ranges.hpp"
#include "registry.hpp"

namespace mrx {

// Zero a 16-byte aligned byte range (the per-call control state) and the
// caller's status word.
__global__ void k_fill_zero(uint4* __restrict__ p, int64_t n16, int32_t* status, int64_t* count,
                            int64_t* count2) {
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (status) *status = 0;
    if (count) *count = 0;
    if (count2) *count2 = 0;
  }
}

// Batch epilogue: out_off[b] = number of used groups of meshes < b, read
// from cmap at the first sorted position of mesh b (a head, since heads
// break at mesh starts).
__global__ void k_batch_offsets(const int64_t* __restrict__ vtx_off, int32_t nmesh, SortBuffers bufs,
                                const int32_t* __restrict__ cmap, const Control* ctl,
                                const int64_t* __restrict__ total_used, int64_t n,
                                int64_t* __restrict__ out_off) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b > nmesh) return;
  const int64_t p = vtx_off[b];
  int64_t r = *total_used;
  if (b < nmesh && p >= 0 && p < n) {
    const uint2* pairs = reinterpret_cast<const uint2*>(bufs.spare());
    const uint32_t g = pairs[p].x;
    if (int64_t(g) < ctl->num_groups) {
      const int32_t c = cmap[g];
      r = c >= 0 ? c : ~c;
    }
  }
  out_off[b] = r;
}

// Output offsets of a batch after its hash grouping, from a list in mesh
// order of group names, which lie in their mesh's vertex range (the last word
// of every `stride`): those of the packed used groups before an LSD key sort,
// or those of the output vertices. Mesh b's outputs start at the
// number of entries below vtx_off[b] (a binary search per mesh).
__global__ void k_batch_offsets_dense(const uint32_t* __restrict__ dense, int32_t stride, const Control* ctl,
                                      const int64_t* vtx_off, int32_t nmesh, int64_t* out_off) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b > nmesh) return;
  const int64_t u = ctl->num_used;
  const int64_t start = vtx_off[b];
  int64_t lo = 0, hi = u;  // first packed position whose name is >= start
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (int64_t(dense[mid * stride + stride - 1]) < start) lo = mid + 1; else hi = mid;
  }
  out_off[b] = lo;
}

__global__ void k_localize_new2old(int32_t* __restrict__ new2old, const int64_t* __restrict__ total_used,
                                   const int64_t* __restrict__ vtx_off, int32_t nmesh,
                                   const int32_t* __restrict__ vtx_tab) {
  const int64_t u = *total_used;
  const int64_t stride = int64_t(gridDim.x) * blockDim.x;
  for (int64_t j = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < u; j += stride) {
    const int32_t g = new2old[j];
    new2old[j] = g - int32_t(vtx_off[mesh_of(vtx_off, nmesh, g, vtx_tab)]);
  }
}

// tab[q] = mesh of packed id min(q << kMeshTabShift, total - 1), q in [0, nq),
// the bucket table that lets mesh_of search a handful of meshes. `more`: a
// second table in the same launch (nq = 0: none).
struct MeshTable {
  const int64_t* off;
  int64_t total;
  int32_t* tab;
  int64_t nq;
};
__global__ void k_mesh_table(MeshTable t, MeshTable more, int32_t nmesh) {
  int64_t q = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (q >= t.nq) {
    q -= t.nq;
    t = more;
  }
  if (q >= t.nq) return;
  t.tab[q] = int32_t(mesh_of(t.off, nmesh, min(q << kMeshTabShift, t.total - 1)));
}

// Workspace of mrx_reindex_mesh_noalloc: a fixed array in the library's code
// object, one copy per GPU the library runs on, kept until the process ends.
// In host code this name denotes a host-side stand-in, not device memory:
// host code only ever uses the device address that hipGetSymbolAddress
// returns for it (scratch_of_current_device).
static __device__ __align__(256) unsigned char scratch[MRX_NOALLOC_SCRATCH_BYTES];

namespace {

// ---------------------------------------------------------------- profiling
struct ProfRecord {
  const char* name;  // null: end of a call
  hipEvent_t event;
};

struct Profiler {
  std::mutex mu;
  bool on = false;
  std::vector<hipEvent_t> pool;
  size_t next = 0;
  std::vector<ProfRecord> recs;

  hipEvent_t take() {
    if (next == pool.size()) {
      hipEvent_t e = nullptr;
      if (hipEventCreate(&e) != hipSuccess) return nullptr;
      pool.push_back(e);
    }
    return pool[next++];
  }
};

Profiler& profiler() {
  static Profiler p;
  return p;
}

// Records a timing event on the stream before a kernel launch (name != null)
// or after the last launch of a call (name == null). Kernel i of a call runs
// between its mark and the next one, since the stream executes in order.
void prof_mark(const char* name, hipStream_t s) {
  Profiler& p = profiler();
  if (!p.on) return;
  std::lock_guard<std::mutex> g(p.mu);
  hipEvent_t e = p.take();
  if (!e) return;
  if (hipEventRecord(e, s) != hipSuccess) return;
  p.recs.push_back(ProfRecord{name, e});
}

constexpr int64_t kMaxCount = int64_t(INT32_MAX);  // ids and counts are int32
constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

const std::vector<SortVariant>& variants_for(int K) {
  static std::vector<SortVariant> table[17];
  static std::once_flag once;
  std::call_once(once, [] {
    void (*reg[16])(std::vector<SortVariant>&) = {
        register_k1, register_k2, register_k3, register_k4, register_k5, register_k6,
        register_k7, register_k8, register_k9, register_k10, register_k11, register_k12,
        register_k13, register_k14, register_k15, register_k16};
    for (int k = 1; k <= 16; ++k) reg[k - 1](table[k]);
  });
  static const std::vector<SortVariant> empty;
  return (K >= 1 && K <= 16) ? table[K] : empty;
}

// Sort passes use 32-bit look-back words unless a count could reach 2^30
// (or the caller asks for the 64-bit words).
constexpr int64_t kCompactLookbackLimit = int64_t(1) << 30;
bool wide_lookback(int64_t n, const mrx_tuning* t) {
  return n >= kCompactLookbackLimit || (t && (t->flags & MRX_TUNING_WIDE_LOOKBACK));
}

// Picks the variant a tuning asks for; all-zero shape (or NULL) = variant 0.
// Unknown flag bits are rejected.
const SortVariant* pick_variant(int K, const mrx_tuning* t) {
  const auto& vs = variants_for(K);
  if (vs.empty()) return nullptr;
  constexpr int32_t known = MRX_TUNING_WIDE_LOOKBACK | MRX_TUNING_CLAIMED_TILES | MRX_TUNING_SORT_ALL |
                             MRX_TUNING_HASH_GROUPS | MRX_TUNING_BANDS;
  if (t && (t->flags & ~known) != 0) return nullptr;
  if (t && (t->flags & MRX_TUNING_SORT_ALL) && (t->flags & MRX_TUNING_HASH_GROUPS)) return nullptr;
  if (!t || (t->digit_bits == 0 && t->block_threads == 0 && t->items_per_thread == 0)) return &vs[0];
  for (const auto& v : vs)
    if (v.D == t->digit_bits && v.block == t->block_threads && v.ipt == t->items_per_thread) return &v;
  return nullptr;
}

int bits_for(int64_t x) {  // bits needed to represent values 0..x
  int b = 0;
  while (x > 0) { ++b; x >>= 1; }
  return b;
}

// Hash grouping for a single mesh of n vertices? Its look-back words hold
// counts below 2^30. By default from the smallest meshes that do not fit one
// workgroup (use_small) on: 21,905 12-byte vertices take 60 us in 11 launches,
// 199 us in the 19 of the sort of all vertices.
constexpr int64_t kHashMinDefault = int64_t(1) << 10;
// For batches, and where the workspace was sized for the sort of all vertices
// of a mesh of fewer vertices than this: from 2^16 on.
constexpr int64_t kHashMinBatch = int64_t(1) << 16;
bool use_hash_groups(int64_t n, int32_t nmesh, const mrx_tuning* t) {
  if (nmesh != 1 || n >= kCompactLookbackLimit) return false;
  if (t && (t->flags & MRX_TUNING_SORT_ALL)) return false;
  if (t && (t->flags & MRX_TUNING_HASH_GROUPS)) return true;
  return n >= kHashMinDefault;
}

// The whole mesh in one workgroup? Only when nothing in the tuning asks for a
// kernel shape, a strategy or bands.
bool use_small(const SortVariant& v, int64_t n, int64_t m, const mrx_tuning* t) {
  if (t && (t->digit_bits != 0 || (t->flags & (MRX_TUNING_SORT_ALL | MRX_TUNING_HASH_GROUPS | MRX_TUNING_BANDS)) != 0))
    return false;
  return n <= v.small_vertices && m <= v.small_entries;
}

// Hash grouping for a batch (key = (mesh id, record))? By default from 2^16
// vertices in all, as for single meshes.
bool use_batched_hash(int64_t n, int32_t nmesh, const mrx_tuning* t) {
  if (nmesh < 2 || n <= 0 || n >= kCompactLookbackLimit) return false;
  if (t && (t->flags & MRX_TUNING_SORT_ALL)) return false;
  if (t && (t->flags & MRX_TUNING_HASH_GROUPS)) return true;
  return n >= kHashMinBatch;
}

// Hash passes: enough D-bit hash digits that a bucket averages at most the
// grouping kernel's target size (1 to 3 passes).
int hash_passes(int64_t n, int D, int target_bucket) {
  int bits = 0;
  while ((n >> bits) > target_bucket) ++bits;
  return std::max(1, std::min(3, (bits + D - 1) / D));
}

// Steps 1 and 4 by vertex bands (band_kernels.hpp) for one mesh. kMarkOnly:
// the marking alone (the index partition in a sort buffer that is free until
// the marking is done: C on the hash-grouping path, B on the sort-all path);
// kMarkAndMap: the marking, old2new and the remap, with the index partition
// in out_idx (its slots become the remapped tiles) and the new ids of the
// entries in a free sort buffer (C, or the sort-all path's spare buffer once
// the pairs in it are partitioned). Chosen when there are enough entries to pay for the extra
// launches on the hash-grouping path (or MRX_TUNING_BANDS asks for it, on
// either path), at most kMaxBands bands of at
// most 2^kMaxMarkShift (marking) or 2^kMaxMapShift (map) vertices, and C
// holds m words. Below about 2^20 entries the five extra launches cost more
// than the scattered accesses they replace (a 390K-entry soup: 0.28 against
// 0.22 ms).
enum BandMode { kBandNone = 0, kMarkOnly = 1, kMarkAndMap = 2 };
constexpr int64_t kBandMinEntries = int64_t(1) << 20;
struct BandPlan {
  int mode = kBandNone;
  bool fine = false;  // the smaller tiles, and bands to match
  int shift = 0, nb = 0;
  int64_t itiles = 0, ptiles = 0;
  size_t words() const {  // index table + tile counts (+ pair table)
    if (mode == kBandNone) return 0;
    return size_t(nb) * size_t(itiles) + size_t(itiles) + (mode == kMarkAndMap ? size_t(nb) * size_t(ptiles) : 0);
  }
};
BandPlan band_plan(int64_t n, int64_t m, int s, bool force, bool automatic) {
  BandPlan b;
  if (n <= 0 || m <= 0 || (!force && (!automatic || m < kBandMinEntries)) || m > n * int64_t(s)) return b;
  int want = kMinBandShift;  // about 256 bands where the band size allows it
  while (((n - 1) >> want) + 1 > 256) ++want;
  for (int mode : {int(kMarkAndMap), int(kMarkOnly)}) {
    const int shift = std::min(want, mode == kMarkAndMap ? kMaxMapShift : kMaxMarkShift);
    const int64_t nb = ((n - 1) >> shift) + 1;
    if (nb > kMaxBands) continue;
    b.mode = mode;
    b.shift = shift;
    b.nb = int(nb);
    b.itiles = (m + kBandTile - 1) / kBandTile;
    b.ptiles = mode == kMarkAndMap ? (n + kPairTile - 1) / kPairTile : 0;
    return b;
  }
  return b;
}

// On the hash path, up to kFineMaxEntries index entries: tiles of a quarter of
// the size and up to 512 bands, so that a slice still holds 16 entries where
// they are scattered. Their larger tables lie behind the sample sort's
// scratch, where there is room.
constexpr int64_t kFineMaxEntries = int64_t(1) << 23;
BandPlan fine_band_plan(const BandPlan& coarse, int64_t n, int64_t m) {
  if (coarse.mode != kMarkAndMap || m > kFineMaxEntries) return coarse;
  BandPlan b = coarse;
  b.fine = true;
  b.shift = kMinFineShift;
  while (((n - 1) >> b.shift) + 1 > 512) ++b.shift;
  if (b.shift > kMaxFineShift) return coarse;
  b.nb = int(((n - 1) >> b.shift) + 1);
  b.itiles = (m + kFineBandTile - 1) / kFineBandTile;
  b.ptiles = (n + kFinePairTile - 1) / kFinePairTile;
  return b;
}

// Bands of a batch (hash path), over the packed vertex ids: always the
// smaller tiles, since a tile's entries and pairs lie in the vertex ranges of
// its few meshes and so in few bands, whatever the number of bands. For
// meshes of 2^12 vertices and more on average: the scattered accesses of
// smaller ones stay within a few cache lines each (4,096 meshes of 400
// vertices: 308 us a call without bands, 342 with; 256 meshes of 80,000:
// 1,788 and 1,666).
BandPlan batch_band_plan(int64_t n, int64_t m, int s, int32_t nmesh) {
  BandPlan b;
  if (m < kBandMinEntries || m > n * int64_t(s) || n < int64_t(nmesh) << 12) return b;
  b.shift = kMinFineShift;
  while (((n - 1) >> b.shift) + 1 > 512 && b.shift < kMaxMapShift) ++b.shift;
  if (((n - 1) >> b.shift) + 1 > kMaxBands) return b;
  b.mode = kMarkAndMap;
  b.fine = true;
  b.nb = int(((n - 1) >> b.shift) + 1);
  b.itiles = (m + kFineBandTile - 1) / kFineBandTile;
  b.ptiles = (n + kFinePairTile - 1) / kFinePairTile;
  return b;
}

struct Layout {
  int K = 0, S = 0, P_key = 0, P_mesh = 0, P_hash = 0;  // P_hash > 0: hash grouping
  BandPlan band;                                         // hash grouping only
  int64_t tiles_sort = 0, tiles_scan = 0, tiles_group = 0;
  bool mesh_hash = false;  // hash grouping of a batch (key = (mesh id, record))
  // zeroed region
  size_t ctl = 0, counters = 0, hist = 0, plan = 0, lookback = 0, scan_lookback = 0, elem_lookback = 0,
         used_v = 0, used_g = 0, hist_hash = 0, plan_hash = 0, dead_hash = 0, group_chunks = 0, group_ranges = 0,
         zero_end = 0;
  int64_t tiles_elem = 0;
  // scratch
  size_t buf_a = 0, buf_b = 0, buf_c = 0, uniq = 0, rep = 0, cmap = 0, vtx_tab = 0, elem_tab = 0, band_tab = 0,
         mesh_bk = 0, total = 0;
  int64_t vtx_tab_n = 0, elem_tab_n = 0;
};

// Element tiles of the sub-mesh selection (k_select_elements).
constexpr int kSelectBlock = 256;
constexpr int kSelectIpt = 16;
constexpr int kSelectTile = kSelectBlock * kSelectIpt;

// num_idx bounds the element count of a sub-mesh selection (arity >= 1).
Layout make_layout(int64_t n, int64_t num_idx, int K, int32_t nmesh, const SortVariant& v,
                   const mrx_tuning* tuning) {
  Layout L;
  L.K = K;
  L.S = K + 1;
  L.P_key = (32 * K + v.D - 1) / v.D;
  L.P_mesh = nmesh > 1 ? (bits_for(int64_t(nmesh) - 1) + v.D - 1) / v.D : 0;
  int ph_mesh = 0;
  if (use_batched_hash(n, nmesh, tuning)) {
    // every mesh's bucket count is at most 1 + 2 n_b / target (k_mesh_buckets)
    const int64_t buckets = int64_t(nmesh) + 2 * n / v.group_mesh_target_bucket + 1;
    ph_mesh = (bits_for(buckets) + v.D - 1) / v.D;
    L.mesh_hash = ph_mesh <= 3;  // more than 2^24 buckets: sort all
  }
  if (L.mesh_hash)
    L.P_hash = ph_mesh;
  else
    L.P_hash = use_hash_groups(n, nmesh, tuning) ? hash_passes(n, v.D, v.group_target_bucket) : 0;
  L.tiles_sort = (n + v.tile() - 1) / v.tile();
  L.tiles_scan = (n + kScanTile - 1) / kScanTile;
  const int group_chunk = L.mesh_hash ? v.group_mesh_chunk : v.group_chunk;
  L.tiles_group = L.P_hash ? (n + group_chunk - 1) / group_chunk : 0;
  const int P = L.P_key + L.P_mesh;
  size_t off = 0;
  L.ctl = off;      off = align_up(off + sizeof(Control));
  // tile counters of every look-back launch of a call (claimed tiles)
  L.counters = off; off = align_up(off + sizeof(uint32_t) * size_t(P + L.P_hash + 8));
  L.hist = off;     off = align_up(off + sizeof(uint32_t) * size_t(P) * size_t(v.radix()));
  L.plan = off;     off = align_up(off + sizeof(uint32_t) * size_t(2 * P + 1));  // SortBuffers::plan
  // sort look-back: tiles x radix 64-bit words, or two alternating buffers of
  // 32-bit words in the same bytes; flag scan and compaction have their own
  const int64_t lb_words = std::max<int64_t>(L.tiles_sort * v.radix(), 1);
  L.lookback = off; off = align_up(off + sizeof(uint64_t) * size_t(lb_words));
  L.scan_lookback = off; off = align_up(off + sizeof(uint64_t) * size_t(L.tiles_scan + 1));
  L.tiles_elem = (num_idx + kSelectTile - 1) / kSelectTile;
  L.elem_lookback = off; off = align_up(off + sizeof(uint64_t) * size_t(L.tiles_elem + 1));
  L.used_g = off;   off = align_up(off + size_t(n));
  if (L.P_hash) {
    L.hist_hash = off; off = align_up(off + sizeof(uint32_t) * size_t(L.P_hash) * size_t(v.radix()));
    L.plan_hash = off; off = align_up(off + sizeof(uint32_t) * size_t(2 * L.P_hash + 1));
    L.dead_hash = off; off = align_up(off + sizeof(uint32_t) * size_t(L.P_hash));
    // a record of each chunk and the bucket it left to k_group_over
    L.group_chunks = off; off = align_up(off + sizeof(uint2) * 2 * size_t(L.tiles_group));
    L.group_ranges = off; off = align_up(off + sizeof(uint32_t) * 3 * size_t(group_compact_ranges(L.tiles_group)));
  }
  // last, so that a call whose Step 1 writes every flag (by bands) can leave
  // it out of the clearing
  L.used_v = off;   off = align_up(off + size_t(n));
  L.zero_end = off;
  L.buf_a = off;    off = align_up(off + sizeof(uint32_t) * size_t(n) * L.S);
  L.buf_b = off;    off = align_up(off + sizeof(uint32_t) * size_t(n) * L.S);
  if (L.P_hash) {
    L.buf_c = off;  off = align_up(off + sizeof(uint32_t) * size_t(n) * L.S);
  }
  if (nmesh == 1) {
    // by default only with hash grouping, the strategy for meshes whose
    // copies (and so index entries) are scattered; on the sort-all path,
    // which the autotuner keeps for meshes stored in order (the paper's quad
    // grid: 0.46 ms without bands, 0.75 ms with), only when asked for
    L.band = band_plan(n, num_idx, L.S, tuning && (tuning->flags & MRX_TUNING_BANDS), L.P_hash > 0);
    L.band_tab = off; off = align_up(off + sizeof(uint32_t) * L.band.words());
  }
  L.uniq = off;     off = align_up(off + sizeof(uint32_t) * size_t(n) * K);
  L.rep = off;      off = align_up(off + sizeof(int32_t) * size_t(n));
  L.cmap = off;     off = align_up(off + sizeof(int32_t) * size_t(n));
  // bucket tables of the element offsets (batch, merge) and vertex offsets
  // (batch) for mesh_of; the element table is small enough to always reserve
  L.elem_tab_n = (std::max<int64_t>(num_idx, 1) - 1) / (int64_t(1) << kMeshTabShift) + 2;
  L.elem_tab = off; off = align_up(off + sizeof(int32_t) * size_t(L.elem_tab_n));
  if (nmesh > 1) {
    L.vtx_tab_n = (std::max<int64_t>(n, 1) - 1) / (int64_t(1) << kMeshTabShift) + 2;
    L.vtx_tab = off;  off = align_up(off + sizeof(int32_t) * size_t(L.vtx_tab_n));
  }
  if (L.mesh_hash) {
    L.mesh_bk = off;  off = align_up(off + sizeof(uint2) * size_t(nmesh));
  }
  L.total = off;
  return L;
}

// True if [a, a+na) and [b, b+nb) overlap (empty ranges never do).
bool overlaps(const void* a, size_t na, const void* b, size_t nb) {
  if (!a || !b || na == 0 || nb == 0) return false;
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + nb && y < x + na;
}

bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

struct Buffer {
  const void* p;
  size_t bytes;
};

// No two listed buffers may overlap.
bool disjoint(std::initializer_list<Buffer> list) {
  std::vector<Buffer> v(list);
  for (size_t i = 0; i < v.size(); ++i)
    for (size_t j = i + 1; j < v.size(); ++j)
      if (overlaps(v[i].p, v[i].bytes, v[j].p, v[j].bytes)) return false;
  return true;
}

int64_t grid_for(int64_t work, int block, int64_t cap = 8192) {
  return std::max<int64_t>(1, std::min<int64_t>((work + block - 1) / block, cap));
}

// Digit location of LSD key bit `bit` (0 = least significant bit of the last
// word): word masks select the word holding it and the next more
// significant word.
void set_digit(SortPassArgs& a, int K, int bit) {
  a.lo_word = K - 1 - bit / 32;
  a.hi_word = a.lo_word - 1;  // -1: none
  a.shift = bit % 32;
}

int64_t rand_grid(int64_t work, int items = kRandItems) {
  return std::max<int64_t>(1, (work + kRandBlock * items - 1) / (kRandBlock * items));
}

// Few entries, so few used values among many (also bucket_plan)?
bool few_used(int64_t n, int64_t m) { return m < n / 8; }

// The scatter's items per thread: with 16 a mesh of 429,165 vertices has 105
// workgroups on 256 CUs (17.9 us; 9.4 us with 4), 4,096 parts of 1.05 million
// 256 (27.4 and 14.3 us). `stage_rep`: representatives of most vertices'
// groups are wanted.
template <bool BATCHED, typename... A>
void launch_scatter_old2new(hipStream_t s, bool stage_rep, SortBuffers sb, const uint2* pairs, const int32_t* cmap,
                            int64_t n, const A&... rest) {
  const dim3 block(kRandBlock), few(rand_grid(n, kScatterFew)), many(rand_grid(n, kScatterItems));
  if (rand_grid(n, kScatterItems) < 4 * 256)
    hipLaunchKernelGGL((k_scatter_old2new<BATCHED, kScatterFew, false>), few, block, 0, s, sb, pairs, cmap, n, rest...);
  else if (stage_rep)
    hipLaunchKernelGGL((k_scatter_old2new<BATCHED, kScatterItems, true>), many, block, 0, s, sb, pairs, cmap, n,
                       rest...);
  else
    hipLaunchKernelGGL((k_scatter_old2new<BATCHED, kScatterItems, false>), many, block, 0, s, sb, pairs, cmap, n,
                       rest...);
}

// Entries of the bucket table of `total` ids (0: none), as laid out by
// make_layout or fewer.
int64_t mesh_table_size(int64_t total) { return total > 0 ? (total - 1) / (int64_t(1) << kMeshTabShift) + 2 : 0; }

void launch_mesh_tables(const MeshTable& t, const MeshTable& more, int32_t nmesh, hipStream_t s) {
  const int64_t nq = t.nq + more.nq;
  if (nq > 0) hipLaunchKernelGGL(k_mesh_table, dim3((nq + 255) / 256), dim3(256), 0, s, t, more, nmesh);
}

mrx_status check_launch() {
  return hipGetLastError() == hipSuccess ? MRX_OK : MRX_ERR_HIP;
}

// Shared validation of the re-index calls (everything before any HIP call).
mrx_status validate_common(const void* vtx, int64_t num_vtx, int32_t vtx_bytes, const int32_t* idx,
                           int64_t num_elems, int32_t arity, const void* out_vtx,
                           const int32_t* out_idx, const int32_t* old2new, const void* workspace,
                           size_t workspace_bytes) {
  if (vtx_bytes < 4 || vtx_bytes > 64 || vtx_bytes % 4 != 0) return MRX_ERR_INVALID_ARGUMENT;
  if (arity < 1 || num_vtx < 0 || num_elems < 0) return MRX_ERR_INVALID_ARGUMENT;
  if (num_vtx > kMaxCount) return MRX_ERR_TOO_LARGE;
  if (num_elems > kMaxCount / arity) return MRX_ERR_TOO_LARGE;
  const int64_t m = num_elems * arity;
  if (num_vtx > 0 && (!vtx || !out_vtx || !old2new)) return MRX_ERR_INVALID_ARGUMENT;
  if (m > 0 && (!idx || !out_idx)) return MRX_ERR_INVALID_ARGUMENT;
  if (!aligned(vtx, 4) || !aligned(out_vtx, 4) || !aligned(idx, 4) || !aligned(out_idx, 4) ||
      !aligned(old2new, 4))
    return MRX_ERR_INVALID_ARGUMENT;
  if (workspace_bytes > 0 && (!workspace || !aligned(workspace, kAlign))) return MRX_ERR_INVALID_ARGUMENT;
  return MRX_OK;
}

// Checks shared by every single-mesh call; on success *layout describes the
// workspace. `extra` lists caller buffers of the call that must not overlap
// any of the others (NULL entries are ignored).
mrx_status validate_single(const void* vtx, int64_t num_vtx, int32_t vtx_bytes, const int32_t* idx,
                           int64_t num_elems, int32_t arity, const void* out_vtx, const int32_t* out_idx,
                           const int32_t* old2new, const int32_t* new2old, const int64_t* out_num_vtx,
                           const int32_t* dev_status, const void* workspace, size_t workspace_bytes,
                           const mrx_tuning* tuning, std::initializer_list<Buffer> extra,
                           const SortVariant** variant, Layout* layout) {
  mrx_status st = validate_common(vtx, num_vtx, vtx_bytes, idx, num_elems, arity, out_vtx, out_idx,
                                  old2new, workspace, workspace_bytes);
  if (st != MRX_OK) return st;
  // dev_status is required: it is the only channel for data errors and for
  // a cross-workgroup wait that gave up (results invalid)
  if (!out_num_vtx || !aligned(out_num_vtx, 8) || !aligned(new2old, 4) || !dev_status ||
      !aligned(dev_status, 4))
    return MRX_ERR_INVALID_ARGUMENT;
  const int K = vtx_bytes / 4;
  const SortVariant* vp = pick_variant(K, tuning);
  if (!vp) return MRX_ERR_UNSUPPORTED;
  const int64_t n = num_vtx, m = num_elems * arity;
  Layout L = make_layout(n, m, K, 1, *vp, tuning);
  if (workspace_bytes < L.total && n < kHashMinBatch && !(tuning && (tuning->flags & MRX_TUNING_HASH_GROUPS))) {
    // a workspace that holds the sort of all vertices will do
    mrx_tuning all = tuning ? *tuning : mrx_tuning{};
    all.flags |= MRX_TUNING_SORT_ALL;
    L = make_layout(n, m, K, 1, *vp, &all);
  }
  if (workspace_bytes < L.total) return MRX_ERR_WORKSPACE_TOO_SMALL;
  const size_t vb = size_t(n) * vtx_bytes, ib = size_t(m) * 4, nb = size_t(n) * 4;
  std::vector<Buffer> outs = {{out_idx, ib}, {vtx, vb}, {out_vtx, vb}, {old2new, nb},
                              {new2old, new2old ? nb : 0}, {out_num_vtx, 8},
                              {dev_status, 4u}, {workspace, L.total}};
  for (const Buffer& b : extra) outs.push_back(b);
  for (size_t i = 0; i < outs.size(); ++i)
    for (size_t j = i + 1; j < outs.size(); ++j)
      if (overlaps(outs[i].p, outs[i].bytes, outs[j].p, outs[j].bytes)) return MRX_ERR_INVALID_ARGUMENT;
  // idx may be out_idx itself, but may not overlap any other buffer
  if (idx != out_idx)
    for (size_t j = 0; j < outs.size(); ++j)
      if (overlaps(idx, ib, outs[j].p, outs[j].bytes)) return MRX_ERR_INVALID_ARGUMENT;
  *variant = vp;
  *layout = L;
  return MRX_OK;
}

// Order of the used groups by record after the grouping (for a batch by (mesh
// id, record)): the sample sort, for up to kSplitMax vertices, else an LSD
// sort of the packed elements. Both leave the output records, cmap and U.
struct OrderArgs {
  uint32_t* X;               // [n][K+1], free
  uint32_t* C;               // [n][K+1], the used groups' elements in their chunks' slots
  uint32_t* scratch;         // [n * K] words
  const uint2* chunks;
  const uint32_t* range_sums;
  int64_t ranges;
  int32_t* cmap;
  uint32_t* out_vtx;
  int64_t* out_num;          // nullable
  Control* ctl;
  int32_t* status;
  uint32_t* hist;            // LSD sort: zeroed histograms, plan, look-back words, tile counters
  uint32_t* plan;
  uint64_t* lookback;
  bool wide;
  uint32_t* counter;         // nullable
  int gp;                    // passes of the call so far
  const uint32_t* rep;       // one mesh: representatives and, nullable, new2old for the LSD sort to write
  int32_t* new2old;
  const int64_t* vtx_off;    // batches
  const int32_t* mesh_tab;
  int32_t nmesh;
  int64_t* out_off;          // holds the meshes' ordered vertex offsets and receives the output offsets
};

// The sample sort's buckets and samples are sized for tens of millions of
// used values: with kMaxBuckets buckets, 67M 12-byte values average two of
// the sort kernel's capacities per bucket, where cutting buckets again still
// costs less than twelve passes over the data.
constexpr int64_t kSplitMax = int64_t(1) << 26;
bool split_applies(const SortVariant& v, const Layout& L, int64_t n, int K) {
  const int64_t runs = group_compact_ranges(L.tiles_group);
  const SplitSort& sp = L.mesh_hash ? v.split_mesh : v.split;
  return n <= kSplitMax && L.tiles_group <= runs * kSplitMaxChunks && sp.scratch(n, runs).words <= n * int64_t(K);
}

void order_used_groups(const SortVariant& v, const Layout& L, int64_t n, int K, const OrderArgs& o, hipStream_t s) {
  const bool mesh = L.mesh_hash;
  if (split_applies(v, L, n, K)) {
    const SplitSort& sp = mesh ? v.split_mesh : v.split;
    const SplitScratch at = sp.scratch(n, o.ranges);
    SplitArgs a{};
    a.sparse = o.C;
    a.chunks = o.chunks;
    a.range_sums = o.range_sums;
    a.tiles = L.tiles_group;
    a.runs = o.ranges;
    a.n = n;
    a.samples = o.scratch + at.samples;
    a.splitters = o.scratch + at.splitters;
    a.counts = o.scratch + at.counts;
    a.starts = o.scratch + at.starts;
    a.run_base = o.scratch + at.run_base;
    a.digits = reinterpret_cast<uint16_t*>(o.scratch + at.digits);
    a.dense = o.X;
    a.cmap = o.cmap;
    a.out_vtx = o.out_vtx;
    a.order = o.C;  // free once scattered
    a.out_num = o.out_num;
    a.ctl = o.ctl;
    a.mesh_off = o.out_off;
    a.mesh_tab = o.mesh_tab;
    a.nmesh = o.nmesh;
    prof_mark("split_sample", s);
    sp.sample(a, s);
    if (sp.ranked(n)) {
      prof_mark("split_rank", s);
      sp.rank(a, s);
    }
    prof_mark("split_count", s);
    sp.count(a, s);
    prof_mark("split_scatter", s);
    sp.scatter(a, s);
    prof_mark("split_sort", s);
    sp.sort(a, s);
    if (mesh) {
      prof_mark("batch_offsets", s);
      hipLaunchKernelGGL(k_batch_offsets_dense, dim3((o.nmesh + 1 + 255) / 256), dim3(256), 0, s,
                         static_cast<const uint32_t*>(a.order), 1, static_cast<const Control*>(o.ctl),
                         static_cast<const int64_t*>(o.out_off), o.nmesh, o.out_off);
    }
    return;
  }
  const int P = L.P_key + (mesh ? L.P_mesh : 0);
  uint32_t* const lb32[2] = {reinterpret_cast<uint32_t*>(o.lookback),
                             reinterpret_cast<uint32_t*>(o.lookback) + size_t(L.tiles_sort) * v.radix()};
  const SortBuffers sb{{o.X, o.C}, o.plan, P};
  const GroupCompactArgs gc{o.C, o.chunks, o.range_sums, L.tiles_group, o.ranges, n, o.X, o.hist, o.ctl};
  prof_mark("compact_histogram", s);
  v.group_compact_hist(gc, s);
  if (mesh) {
    prof_mark("batch_offsets", s);
    hipLaunchKernelGGL(k_batch_offsets_dense, dim3((o.nmesh + 1 + 255) / 256), dim3(256), 0, s,
                       static_cast<const uint32_t*>(o.X), int32_t(K + 1), static_cast<const Control*>(o.ctl),
                       static_cast<const int64_t*>(o.out_off), o.nmesh, o.out_off);
    prof_mark("mesh_histogram", s);
    v.mesh_hist(o.out_off, o.nmesh, L.P_mesh, o.hist + size_t(L.P_key) * v.radix(), s);
  }
  prof_mark("scan_buckets", s);
  v.scan(o.hist, P, n, &o.ctl->num_used, o.plan + P + 1, s);
  prof_mark("sort_plan", s);
  hipLaunchKernelGGL(k_group_sort_plan, dim3(1), dim3(64), 0, s, sb);
  int gp = o.gp;
  for (int p = 0; p < P; ++p, ++gp) {
    SortPassArgs a{};
    a.bufs = sb;
    a.pass = p;
    a.bucket_base = o.hist + size_t(p) * v.radix();
    a.lookback = o.wide ? static_cast<void*>(o.lookback) : static_cast<void*>(lb32[gp & 1]);
    a.lookback_next = lb32[(gp + 1) & 1];
    a.tile_counter = o.counter ? o.counter + p : nullptr;
    a.ctl = o.ctl;
    a.status = o.status;
    a.n = n;
    a.n_dev = &o.ctl->num_used;
    a.mesh_off = o.vtx_off;
    a.mesh_tab = o.mesh_tab;
    a.nmesh = o.nmesh;
    a.tag = uint32_t(gp + 1);
    int mode = kPassKey;
    if (p < L.P_key) {
      set_digit(a, K, p * v.D);
    } else {
      a.shift = (p - L.P_key) * v.D;
      mode = kPassMesh;
    }
    prof_mark(mode == kPassMesh ? "onesweep_mesh" : "onesweep", s);
    v.pass(a, mode, o.wide, L.tiles_sort, s);
  }
  FinalizeArgs fa{};
  fa.bufs = sb;
  fa.cmap = o.cmap;
  fa.out_vtx = o.out_vtx;
  fa.rep = o.rep;
  fa.new2old = o.new2old;
  fa.out_num = o.out_num;
  fa.cap = n;
  fa.ctl = o.ctl;
  fa.status = o.status;
  prof_mark("finalize", s);
  v.finalize(fa, grid_for(n, 256, 4096), s);
}

// Where the bucket path (bucket_kernels.hpp) keeps its state: starts, totals,
// chunk records and run sums in the look-back words, which nothing else uses
// on that path, and the counts in the buffer that takes the pairs.
struct BucketState {
  BucketPlan plan;           // buckets = 0: the call sorts by hash digits instead
  BucketArgs args{};
  uint2* chunks = nullptr;
  uint32_t* range_sums = nullptr;
  int64_t ranges = 0;
};

// What the grouping of large buckets keeps in the zeroed flags of the sort of
// all vertices (n bytes, at least 256, which hash grouping leaves alone): a
// word that says whether there are any, two words of state per part and, on
// the digit path, one more and the list of the chunks that left a bucket.
LargeBuckets large_buckets(int64_t n, uint32_t* words, GroupArgs* g) {
  const LargeBuckets l{large_part(n), large_helpers(n), words, words + 2};
  g->part = l.part;
  g->over_any = words;
  g->over_count = words + 1;
  g->over_at = l.state + 2 * (l.helpers + 1);
  g->over_list = g->over_at + l.helpers + 1;
  return l;
}

BucketState bucket_state(const SortVariant& v, Layout L, int64_t n, int64_t m, int K, int32_t nmesh,
                         uint32_t* lookback, uint32_t* matrix) {
  BucketState b;
  const BucketGroup& g = nmesh > 1 ? v.bucket_mesh : v.bucket;
  const BucketPlan p = g.plan(n, m, nmesh, n * int64_t(K + 1));
  const int64_t F = p.buckets;
  const int64_t ranges = group_compact_ranges(F);
  if (F == 0 || F > (nmesh > 1 ? kBucketMaxMesh : kBucketMax) ||
      4 * F + 2 + ranges > 2 * L.tiles_sort * int64_t(v.radix()))
    return b;
  L.tiles_group = F;
  if (!split_applies(v, L, n, K)) return b;
  b.plan = p;
  b.chunks = reinterpret_cast<uint2*>(lookback);
  b.args.starts = lookback + 2 * F;
  b.args.totals = b.args.starts + F + 1;
  b.range_sums = b.args.totals + F;
  b.ranges = ranges;
  b.args.n = n;
  b.args.buckets = int32_t(F);
  b.args.tiles = p.tiles;
  b.args.tile = kBucketBlock * p.ept;
  b.args.stride = int32_t((F + 1) / 2 * 2);
  b.args.counts = reinterpret_cast<uint16_t*>(matrix);
  b.args.base = matrix + p.count_words();
  return b;
}

// Elements into their buckets (in args.elems) and the buckets grouped.
void group_buckets(BucketState& b, const BucketGroup& g, const MarkArgs* mark, const BandArgs* band, GroupArgs ga,
                   const LargeBuckets& large, hipStream_t s) {
  b.args.most = 2 * uint32_t(large.part);
  b.args.large = ga.over_any;
  prof_mark(mark || band ? "mark_bucket_count" : "bucket_count", s);
  g.count(b.args, mark, band, s);
  prof_mark("bucket_offsets", s);
  const dim3 columns((b.args.buckets + kOffsetCols - 1) / kOffsetCols), block(kOffsetCols * kOffsetRuns);
  if (b.args.nmesh > 0)
    hipLaunchKernelGGL(k_bucket_offsets<true>, columns, block, 0, s, b.args);
  else
    hipLaunchKernelGGL(k_bucket_offsets<false>, columns, block, 0, s, b.args);
  prof_mark("bucket_scatter", s);
  g.scatter(b.args, s);
  ga.elems = b.args.elems;
  ga.chunks = b.chunks;
  ga.range_sums = b.range_sums;
  ga.ranges = b.ranges;
  const GroupBucketArgs a{ga, b.args.starts, b.args.buckets, b.plan.target, large};
  prof_mark("group", s);
  g.group(a, s);
}

// The hash-grouping launch sequence of one mesh (see group_kernels.hpp):
//   Step 1 (marking, by vertex bands or by scattered stores) with the
//   hash-digit histograms; stable sort of (record, id | used << 31) by
//   P_hash hash digits into X; grouping of each hash bucket (pairs
//   (group, id) into Y, one (record, group) element per used group into its
//   chunk's slots of C); order of the used groups by record, with the output
//   records and the map from group to new id (order_used_groups); Step 4
//   (old2new, with new2old, and the index remap, by vertex bands or by
//   scattered accesses).
// Buffers: A and B hold the hash passes (X = the last one written, Y = the
// other), C the used groups' slots (before the grouping: Step 1's index
// partition when only the marking goes by bands); the ordering works in X and
// C; by bands, Step 4 then partitions the pairs into X and puts the index
// entries' new ids in C.
mrx_status launch_hash(const SortVariant& v, const Layout& layout, const void* vtx, int64_t num_vtx,
                       int32_t vtx_bytes, const int32_t* idx, int64_t num_elems, int32_t arity,
                       const int64_t* live_elems, void* out_vtx, int32_t* out_idx, int32_t* old2new,
                       int32_t* new2old, int64_t* out_num_vtx, int32_t* dev_status, void* workspace,
                       const mrx_tuning* tuning, void* stream_, bool state_zeroed) {
  Layout L = layout;
  const int K = vtx_bytes / 4;
  const int64_t n = num_vtx, m = num_elems * arity;
  const int ph = L.P_hash;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream_);
  char* ws = static_cast<char*>(workspace);
  Control* ctl = reinterpret_cast<Control*>(ws + L.ctl);
  uint32_t* counters = reinterpret_cast<uint32_t*>(ws + L.counters);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
  uint32_t* plan = reinterpret_cast<uint32_t*>(ws + L.plan);
  uint32_t* hist_hash = reinterpret_cast<uint32_t*>(ws + L.hist_hash);
  uint32_t* plan_hash = reinterpret_cast<uint32_t*>(ws + L.plan_hash);
  uint32_t* dead_hash = reinterpret_cast<uint32_t*>(ws + L.dead_hash);
  uint64_t* lookback = reinterpret_cast<uint64_t*>(ws + L.lookback);
  uint2* group_chunks = reinterpret_cast<uint2*>(ws + L.group_chunks);
  uint32_t* group_range_sums = reinterpret_cast<uint32_t*>(ws + L.group_ranges);
  const bool wide = wide_lookback(n, tuning);
  const bool claimed = tuning && (tuning->flags & MRX_TUNING_CLAIMED_TILES);
  uint32_t* const lb32[2] = {reinterpret_cast<uint32_t*>(lookback),
                             reinterpret_cast<uint32_t*>(lookback) + size_t(L.tiles_sort) * v.radix()};
  uint8_t* used_v = reinterpret_cast<uint8_t*>(ws + L.used_v);
  uint32_t* buf[3] = {reinterpret_cast<uint32_t*>(ws + L.buf_a), reinterpret_cast<uint32_t*>(ws + L.buf_b),
                      reinterpret_cast<uint32_t*>(ws + L.buf_c)};
  int32_t* rep = reinterpret_cast<int32_t*>(ws + L.rep);
  int32_t* cmap = reinterpret_cast<int32_t*>(ws + L.cmap);
  int32_t* status = dev_status;
  int counter = 0;  // next tile counter (claimed tiles)
  auto next_counter = [&]() { return claimed ? counters + counter++ : nullptr; };

  // one partition pass where the buckets suffice, else two or three stable
  // passes by hash digits; the order of the used groups takes either's chunks
  BucketState bs = bucket_state(v, L, n, m, K, 1, reinterpret_cast<uint32_t*>(lookback), buf[1]);
  const bool bucketed = bs.plan.buckets > 0;
  if (bucketed) L.tiles_group = bs.plan.buckets;
  const int64_t group_ranges = group_compact_ranges(L.tiles_group);
  if (!state_zeroed) {
    // band marking writes every used flag: those need no clearing
    const int64_t words = int64_t((L.band.mode != kBandNone ? L.used_v : L.zero_end) / 16);
    prof_mark("fill_zero", s);
    hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(words, 256, 4096)), dim3(256), 0, s,
                       reinterpret_cast<uint4*>(ws), words, dev_status, out_num_vtx,
                       static_cast<int64_t*>(nullptr));
  }
  // Step 1 and the hash-digit histograms: Step 1 by vertex bands (the index
  // partition in out_idx, or in C, which the grouping fills only later),
  // else scattered byte stores beside the histograms
  BandPlan bp = L.band;
  uint32_t* band_tab = reinterpret_cast<uint32_t*>(ws + L.band_tab);
  if (split_applies(v, L, n, K)) {
    const BandPlan fine = fine_band_plan(L.band, n, m);
    const int64_t used = v.split.scratch(n, group_ranges).words;
    if (fine.fine && used + int64_t(fine.words()) <= n * int64_t(K)) {
      bp = fine;
      band_tab = reinterpret_cast<uint32_t*>(ws + L.uniq) + used;
    }
  }
  const MarkArgs mark{idx, m, arity, n, nullptr, nullptr, 0, nullptr, live_elems, used_v, status};
  uint32_t* ipart = bp.mode == kMarkAndMap ? reinterpret_cast<uint32_t*>(out_idx) : buf[2];
  uint32_t* itable = band_tab;
  uint32_t* itile_valid = itable + size_t(bp.nb) * size_t(bp.itiles);
  uint32_t* ptable = itile_valid + bp.itiles;
  const BandArgs ba{idx, m, arity, n, live_elems, bp.shift, bp.nb, aligned(idx, 16) ? 1 : 0,
                    bp.mode == kMarkAndMap ? 1 : 0, bp.itiles, bp.fine ? 1 : 0, ipart, itable, itile_valid, used_v,
                    status, nullptr, nullptr, nullptr, 0};
  if (bp.mode != kBandNone) {
    prof_mark("band_partition", s);
    launch_band_partition(ba, s);
  }
  if (bp.mode == kMarkOnly) {
    prof_mark("band_mark", s);
    launch_band_mark(ba, false, s);
  }
  const bool band_mark = bp.mode == kMarkAndMap, scatter_mark = m > 0 && bp.mode == kBandNone;
  if (!bucketed) {
    prof_mark(band_mark ? "band_mark_histogram" : scatter_mark ? "mark_histogram" : "hash_histogram", s);
    if (band_mark)
      v.band_mark_hash_hist(ba, static_cast<const uint32_t*>(vtx), n, ph, hist_hash, s);
    else
      v.hash_hist(scatter_mark ? &mark : nullptr, static_cast<const uint32_t*>(vtx), n, ph, hist_hash, s);
  }
  if (n > 0) {
    uint32_t* X = buf[0];
    uint32_t* Y = buf[1];
    int gp = 0;  // index of the pass in the call (look-back buffer parity, tag)
    GroupArgs g{};
    g.n = n;
    g.rep = reinterpret_cast<uint32_t*>(rep);
    g.cmap = cmap;
    g.uelems = buf[2];
    g.status = status;
    const LargeBuckets large = large_buckets(n, reinterpret_cast<uint32_t*>(ws + L.used_g), &g);
    if (bucketed) {
      bs.args.vtx = static_cast<const uint32_t*>(vtx);
      bs.args.used = used_v;
      bs.args.elems = X;
      g.pairs = reinterpret_cast<uint2*>(Y);
      group_chunks = bs.chunks;
      group_range_sums = bs.range_sums;
      group_buckets(bs, v.bucket, scatter_mark ? &mark : nullptr, band_mark ? &ba : nullptr, g, large, s);
    } else {
      // stable sort by the hash digits; every hash pass runs (dead flags go to
      // a word nobody reads), so the elements end in X = buf[(ph - 1) & 1]
      prof_mark("scan_buckets", s);
      v.scan(hist_hash, ph, n, nullptr, dead_hash, s);
      const SortBuffers sbh{{buf[0], buf[1]}, plan_hash, ph};
      for (int p = 0; p < ph; ++p, ++gp) {
        SortPassArgs a{};
        a.vtx = static_cast<const uint32_t*>(vtx);
        a.bufs = sbh;
        a.pass = p;
        a.used = used_v;
        a.bucket_base = hist_hash + size_t(p) * v.radix();
        a.lookback = wide ? static_cast<void*>(lookback) : static_cast<void*>(lb32[gp & 1]);
        a.lookback_next = lb32[(gp + 1) & 1];
        a.tile_counter = next_counter();
        a.ctl = ctl;
        a.status = status;
        a.n = n;
        a.lo_word = a.hi_word = -1;
        a.shift = p * v.D;
        a.tag = uint32_t(gp + 1);
        prof_mark(p == 0 ? "onesweep_hash_first" : "onesweep_hash", s);
        v.pass(a, p == 0 ? kPassFirstHash : kPassHash, wide, L.tiles_sort, s);
      }
      X = buf[(ph - 1) & 1];
      Y = buf[((ph - 1) & 1) ^ 1];
      // group each hash bucket
      g.elems = X;
      g.pairs = reinterpret_cast<uint2*>(Y);
      g.bucket_mask = ph * v.D >= 32 ? 0xFFFFFFFFu : (1u << (ph * v.D)) - 1u;
      g.chunks = group_chunks;
      g.range_sums = group_range_sums;
      g.ranges = group_ranges;
      g.over = group_chunks + L.tiles_group;
      prof_mark("group", s);
      v.group(g, L.tiles_group, s);
      prof_mark("group_over", s);
      v.group_over(g, large, L.tiles_group, s);
    }
    uint2* pairs = reinterpret_cast<uint2*>(Y);
    OrderArgs o{};
    o.X = X;
    o.C = buf[2];
    o.scratch = reinterpret_cast<uint32_t*>(ws + L.uniq);
    o.chunks = group_chunks;
    o.range_sums = group_range_sums;
    o.ranges = group_ranges;
    o.cmap = cmap;
    o.out_vtx = static_cast<uint32_t*>(out_vtx);
    o.ctl = ctl;
    o.status = status;
    o.hist = hist;
    o.plan = plan;
    o.lookback = lookback;
    o.wide = wide;
    o.counter = claimed ? counters + counter : nullptr;
    o.gp = gp;
    o.out_num = out_num_vtx;
    o.rep = reinterpret_cast<const uint32_t*>(rep);
    o.new2old = new2old;
    order_used_groups(v, L, n, K, o, s);
    if (!split_applies(v, L, n, K)) new2old = nullptr;  // written
    // Step 4's map (and, by bands, the remap)
    if (bp.mode == kMarkAndMap) {
      // X and C are free again: X takes the partitioned pairs, C the new ids
      // of the index entries
      const PairPartArgs pa{static_cast<const uint2*>(pairs), cmap, n, bp.shift, bp.nb, bp.ptiles,
                            reinterpret_cast<uint2*>(X), ptable, status,
                            reinterpret_cast<const uint32_t*>(rep), new2old, g.over_any, SortBuffers{}, 0,
                            nullptr, nullptr, nullptr, 0};
      prof_mark("pair_partition", s);
      launch_pair_partition(pa, bp.fine, s);
      const BandMapArgs ma{reinterpret_cast<const uint2*>(X), ptable, bp.ptiles, ipart, itable, bp.itiles, n,
                           bp.shift, bp.nb, old2new, reinterpret_cast<int32_t*>(buf[2])};
      prof_mark("band_map", s);
      launch_band_map(ma, bp.fine, s);
      const BandRemapArgs ra{ipart, reinterpret_cast<const int32_t*>(buf[2]), itile_valid, m, arity, live_elems,
                             out_idx};
      prof_mark("band_remap", s);
      launch_band_remap(ra, bp.itiles, bp.fine, s);
      prof_mark(nullptr, s);
      return check_launch();
    }
    prof_mark("old2new", s);
    launch_scatter_old2new<false>(s, new2old && !few_used(n, m), SortBuffers{{nullptr, nullptr}, nullptr, 0},
                                  static_cast<const uint2*>(pairs), cmap, n, nullptr, nullptr, 0, nullptr, old2new,
                                  reinterpret_cast<const uint32_t*>(rep), new2old,
                                  static_cast<const uint32_t*>(g.over_any));
  }
  // Step 4: remap the index array
  if (m > 0) {
    prof_mark("remap", s);
    hipLaunchKernelGGL((k_remap<false>), dim3(rand_grid(m)), dim3(kRandBlock), 0, s, idx, m, arity, n,
                       nullptr, nullptr, 0, nullptr, live_elems, old2new, out_idx);
  }
  prof_mark(nullptr, s);
  return check_launch();
}

// The single-mesh launch sequence (Section 2, Steps 1-4). live_elems
// (device, nullable) limits the index array to its first *live_elems
// elements; num_elems is then only a capacity.
mrx_status launch_single(const SortVariant& v, const Layout& L, const void* vtx, int64_t num_vtx,
                         int32_t vtx_bytes, const int32_t* idx, int64_t num_elems, int32_t arity,
                         const int64_t* live_elems, void* out_vtx, int32_t* out_idx, int32_t* old2new,
                         int32_t* new2old, int64_t* out_num_vtx, int32_t* dev_status, void* workspace,
                         const mrx_tuning* tuning, void* stream_, bool state_zeroed = false) {
  if (use_small(v, num_vtx, num_elems * arity, tuning)) {
    hipStream_t s = reinterpret_cast<hipStream_t>(stream_);
    const SmallArgs a{static_cast<const uint32_t*>(vtx), int32_t(num_vtx), idx, int32_t(num_elems * arity), arity,
                      live_elems, static_cast<uint32_t*>(out_vtx), out_idx, old2new, new2old, out_num_vtx,
                      dev_status, state_zeroed ? 1 : 0};
    prof_mark("small", s);
    v.small(a, s);
    prof_mark(nullptr, s);
    return check_launch();
  }
  if (L.P_hash)
    return launch_hash(v, L, vtx, num_vtx, vtx_bytes, idx, num_elems, arity, live_elems, out_vtx, out_idx,
                       old2new, new2old, out_num_vtx, dev_status, workspace, tuning, stream_, state_zeroed);
  const int K = vtx_bytes / 4;
  const int64_t n = num_vtx, m = num_elems * arity;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream_);
  char* ws = static_cast<char*>(workspace);
  Control* ctl = reinterpret_cast<Control*>(ws + L.ctl);
  uint32_t* counters = reinterpret_cast<uint32_t*>(ws + L.counters);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
  uint32_t* plan = reinterpret_cast<uint32_t*>(ws + L.plan);
  uint64_t* lookback = reinterpret_cast<uint64_t*>(ws + L.lookback);
  uint64_t* scan_lookback = reinterpret_cast<uint64_t*>(ws + L.scan_lookback);
  const bool wide = wide_lookback(n, tuning);
  const bool claimed = tuning && (tuning->flags & MRX_TUNING_CLAIMED_TILES);
  uint32_t* const lb32[2] = {reinterpret_cast<uint32_t*>(lookback),
                             reinterpret_cast<uint32_t*>(lookback) + size_t(L.tiles_sort) * v.radix()};
  uint8_t* used_v = reinterpret_cast<uint8_t*>(ws + L.used_v);
  uint8_t* used_g = reinterpret_cast<uint8_t*>(ws + L.used_g);
  uint32_t* buf[2] = {reinterpret_cast<uint32_t*>(ws + L.buf_a), reinterpret_cast<uint32_t*>(ws + L.buf_b)};
  uint32_t* uniq = reinterpret_cast<uint32_t*>(ws + L.uniq);
  int32_t* rep = reinterpret_cast<int32_t*>(ws + L.rep);
  int32_t* cmap = reinterpret_cast<int32_t*>(ws + L.cmap);
  int32_t* status = dev_status;

  const BandPlan& bp = L.band;
  // per-call state: look-back words, tile counters, histograms, flags, G
  // (already cleared when a preceding step of the same call used it; band
  // marking writes every used flag, so those need no clearing)
  if (!state_zeroed) {
    const int64_t words = int64_t((bp.mode != kBandNone ? L.used_v : L.zero_end) / 16);
    prof_mark("fill_zero", s);
    hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(words, 256, 4096)), dim3(256), 0, s,
                       reinterpret_cast<uint4*>(ws), words, dev_status, out_num_vtx,
                       static_cast<int64_t*>(nullptr));
  }
  // Step 1: mark referenced vertices (and report out-of-range entries): by
  // vertex bands (the index partition in out_idx, or in B, which the sort
  // first writes in its second pass), else with the digit histograms of
  // Step 2 in the same launch where it applies
  const MarkArgs mark{idx, m, arity, n, nullptr, nullptr, 0, nullptr, live_elems, used_v, status};
  uint32_t* band_tab = reinterpret_cast<uint32_t*>(ws + L.band_tab);
  uint32_t* ipart = bp.mode == kMarkAndMap ? reinterpret_cast<uint32_t*>(out_idx) : buf[1];
  uint32_t* itable = band_tab;
  uint32_t* itile_valid = itable + size_t(bp.nb) * size_t(bp.itiles);
  uint32_t* ptable = itile_valid + bp.itiles;
  const bool fused = bp.mode == kBandNone && v.mark_hist_applies(n, m);
  if (bp.mode != kBandNone) {
    const BandArgs ba{idx, m, arity, n, live_elems, bp.shift, bp.nb, aligned(idx, 16) ? 1 : 0,
                      bp.mode == kMarkAndMap ? 1 : 0, bp.itiles, 0, ipart, itable, itile_valid, used_v, status, nullptr,
                      nullptr, nullptr, 0};
    prof_mark("band_partition", s);
    launch_band_partition(ba, s);
    prof_mark("band_mark", s);
    launch_band_mark(ba, bp.mode == kMarkAndMap, s);
  } else if (fused) {
    prof_mark("mark_histogram", s);
    v.mark_hist(mark, false, static_cast<const uint32_t*>(vtx), n, hist, s);
  } else if (m > 0) {
    prof_mark("mark_used", s);
    hipLaunchKernelGGL((k_mark_used<false>), dim3(rand_grid(m)), dim3(kRandBlock), 0, s, mark);
  }
  if (n > 0) {
    // Step 2: stable LSD radix sort of (record, id | used << 31)
    if (!fused) {
      prof_mark("histogram", s);
      v.hist(static_cast<const uint32_t*>(vtx), n, hist, s);
    }
    prof_mark("scan_buckets", s);
    v.scan(hist, L.P_key, n, nullptr, plan + L.P_key + 1, s);
    const SortBuffers sb{{buf[0], buf[1]}, plan, L.P_key};
    for (int p = 0; p < L.P_key; ++p) {
      SortPassArgs a{};
      a.vtx = static_cast<const uint32_t*>(vtx);
      a.bufs = sb;
      a.pass = p;
      a.used = used_v;
      a.bucket_base = hist + size_t(p) * v.radix();
      a.lookback = wide ? static_cast<void*>(lookback) : static_cast<void*>(lb32[p & 1]);
      a.lookback_next = lb32[(p + 1) & 1];
      a.tile_counter = claimed ? counters + p : nullptr;
      a.ctl = ctl;
      a.status = status;
      a.n = n;
      set_digit(a, K, p * v.D);
      a.tag = uint32_t(p + 1);
      prof_mark(p == 0 ? "onesweep_first" : "onesweep", s);
      v.pass(a, p == 0 ? kPassFirst : kPassKey, wide, L.tiles_sort, s);
    }
    // Step 2 flags + prefix sum, Step 3/4 scatters
    FlagScanArgs f{};
    f.bufs = sb;
    f.n = n;
    f.uniq = uniq;
    f.rep = rep;
    f.used_g = used_g;
    f.lookback = scan_lookback;
    f.tile_counter = claimed ? counters + L.P_key : nullptr;
    f.ctl = ctl;
    f.status = status;
    f.tag = uint32_t(L.P_key + 1);
    prof_mark("flag_scan", s);
    v.flag_scan(f, false, L.tiles_scan, s);
    // Step 3 on used groups only: compaction
    CompactArgs c{};
    c.used_g = used_g;
    c.uniq = uniq;
    c.rep = rep;
    c.K = K;
    c.out_vtx = static_cast<uint32_t*>(out_vtx);
    c.new2old = new2old;
    c.cmap = cmap;
    c.out_num = out_num_vtx;
    c.cap = n;
    c.lookback = scan_lookback;
    c.tile_counter = claimed ? counters + L.P_key + 1 : nullptr;
    c.ctl = ctl;
    c.status = status;
    c.tag = uint32_t(L.P_key + 2);
    prof_mark("compact", s);
    hipLaunchKernelGGL((k_compact<kScanBlock, kScanIpt>), dim3(L.tiles_scan), dim3(kScanBlock), 0, s, c);
    if (bp.mode == kMarkAndMap) {
      // Step 4 by vertex bands: the pairs (in the spare buffer) partitioned
      // into the sorted buffer, the index entries' new ids into the spare one
      PairPartArgs pa{};
      pa.cmap = cmap;
      pa.n = n;
      pa.shift = bp.shift;
      pa.nb = bp.nb;
      pa.tiles = bp.ptiles;
      pa.table = ptable;
      pa.status = status;
      pa.sort = sb;
      pa.from_sort = 1;
      prof_mark("pair_partition", s);
      launch_pair_partition(pa, false, s);
      BandMapArgs ma{};
      ma.ptable = ptable;
      ma.ptiles = bp.ptiles;
      ma.ipart = ipart;
      ma.itable = itable;
      ma.itiles = bp.itiles;
      ma.n = n;
      ma.shift = bp.shift;
      ma.nb = bp.nb;
      ma.old2new = old2new;
      ma.sort = sb;
      ma.from_sort = 1;
      prof_mark("band_map", s);
      launch_band_map(ma, false, s);
      BandRemapArgs ra{};
      ra.ipart = ipart;
      ra.tile_valid = itile_valid;
      ra.m = m;
      ra.arity = arity;
      ra.live_elems = live_elems;
      ra.out_idx = out_idx;
      ra.sort = sb;
      ra.from_sort = 1;
      prof_mark("band_remap", s);
      launch_band_remap(ra, bp.itiles, false, s);
      prof_mark(nullptr, s);
      return check_launch();
    }
    prof_mark("old2new", s);
    launch_scatter_old2new<false>(s, false, sb, static_cast<const uint2*>(nullptr), cmap, n, nullptr, nullptr, 0,
                                  nullptr, old2new, static_cast<const uint32_t*>(nullptr), static_cast<int32_t*>(nullptr),
                                  static_cast<const uint32_t*>(nullptr));
  }
  // Step 4: remap the index array
  if (m > 0) {
    prof_mark("remap", s);
    hipLaunchKernelGGL((k_remap<false>), dim3(rand_grid(m)), dim3(kRandBlock), 0, s, idx, m, arity, n,
                       nullptr, nullptr, 0, nullptr, live_elems, old2new, out_idx);
  }
  prof_mark(nullptr, s);
  return check_launch();
}

// The hash-grouping launch sequence of a batch: launch_hash's, with
// vertices told apart by (mesh id, record). The hash digits are those of a
// bucket of the vertex's mesh (each mesh owns a range of buckets, in mesh
// order), so the hash-ordered elements are grouped by mesh; the grouping
// compares (mesh id, record) and names each group by a sorted position of
// one of its copies, which lies in its mesh's vertex range; the used groups
// are ordered by (mesh id, record), the mesh of an element being that of its
// name. New ids are numbered over the whole batch and made mesh-local by the
// old2new scatter.
mrx_status launch_batched_hash(const SortVariant& v, const Layout& layout, const void* vtx, const int64_t* vtx_offsets,
                               int64_t n, int32_t vtx_bytes, const int32_t* idx, const int64_t* elem_offsets,
                               int64_t total_elems, int32_t arity, int32_t num_meshes, void* out_vtx,
                               int64_t* out_vtx_offsets, int32_t* out_idx, int32_t* old2new, int32_t* new2old,
                               int32_t* dev_status, void* workspace, const mrx_tuning* tuning, void* stream_) {
  Layout L = layout;
  const int K = vtx_bytes / 4;
  const int64_t m = total_elems * arity;
  const int ph = L.P_hash;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream_);
  char* ws = static_cast<char*>(workspace);
  Control* ctl = reinterpret_cast<Control*>(ws + L.ctl);
  uint32_t* counters = reinterpret_cast<uint32_t*>(ws + L.counters);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
  uint32_t* plan = reinterpret_cast<uint32_t*>(ws + L.plan);
  uint32_t* hist_hash = reinterpret_cast<uint32_t*>(ws + L.hist_hash);
  uint32_t* plan_hash = reinterpret_cast<uint32_t*>(ws + L.plan_hash);
  uint32_t* dead_hash = reinterpret_cast<uint32_t*>(ws + L.dead_hash);
  uint64_t* lookback = reinterpret_cast<uint64_t*>(ws + L.lookback);
  uint2* group_chunks = reinterpret_cast<uint2*>(ws + L.group_chunks);
  uint32_t* group_range_sums = reinterpret_cast<uint32_t*>(ws + L.group_ranges);
  const bool wide = wide_lookback(n, tuning);
  const bool claimed = tuning && (tuning->flags & MRX_TUNING_CLAIMED_TILES);
  uint32_t* const lb32[2] = {reinterpret_cast<uint32_t*>(lookback),
                             reinterpret_cast<uint32_t*>(lookback) + size_t(L.tiles_sort) * v.radix()};
  uint8_t* used_v = reinterpret_cast<uint8_t*>(ws + L.used_v);
  uint32_t* buf[3] = {reinterpret_cast<uint32_t*>(ws + L.buf_a), reinterpret_cast<uint32_t*>(ws + L.buf_b),
                      reinterpret_cast<uint32_t*>(ws + L.buf_c)};
  int32_t* rep = reinterpret_cast<int32_t*>(ws + L.rep);
  int32_t* cmap = reinterpret_cast<int32_t*>(ws + L.cmap);
  int32_t* vtab = reinterpret_cast<int32_t*>(ws + L.vtx_tab);
  int32_t* etab = L.elem_tab_n ? reinterpret_cast<int32_t*>(ws + L.elem_tab) : nullptr;
  uint2* mbk = reinterpret_cast<uint2*>(ws + L.mesh_bk);
  int32_t* status = dev_status;
  int counter = 0;  // next tile counter (claimed tiles)
  auto next_counter = [&]() { return claimed ? counters + counter++ : nullptr; };

  BucketState bs = bucket_state(v, L, n, m, K, num_meshes, reinterpret_cast<uint32_t*>(lookback), buf[1]);
  const bool bucketed = bs.plan.buckets > 0;
  if (bucketed) L.tiles_group = bs.plan.buckets;
  const int64_t group_ranges = group_compact_ranges(L.tiles_group);

  prof_mark("fill_zero", s);
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(int64_t(L.zero_end / 16), 256, 4096)), dim3(256), 0, s,
                     reinterpret_cast<uint4*>(ws), int64_t(L.zero_end / 16), dev_status,
                     static_cast<int64_t*>(nullptr), static_cast<int64_t*>(nullptr));
  // n > 0 and num_meshes > 1 here (use_batched_hash). The grouping and the
  // ordering go by the ordered offsets, which the output offsets' array holds
  // until those are known; Steps 1 and 4, which check every place they touch,
  // by the caller's.
  const int64_t* ordered = out_vtx_offsets;
  prof_mark("mesh_buckets", s);
  if (bucketed)
    hipLaunchKernelGGL(k_mesh_buckets<false>, dim3(1), dim3(kMeshBucketBlock), 0, s, vtx_offsets, num_meshes, n,
                       bs.plan.target, out_vtx_offsets, mbk);
  else
    hipLaunchKernelGGL(k_mesh_buckets<true>, dim3(1), dim3(kMeshBucketBlock), 0, s, vtx_offsets, num_meshes, n,
                       int32_t(v.group_mesh_target_bucket), out_vtx_offsets, mbk);
  prof_mark("mesh_tables", s);
  if (total_elems <= 0) etab = nullptr;
  launch_mesh_tables({ordered, n, vtab, L.vtx_tab_n}, {elem_offsets, total_elems, etab, mesh_table_size(total_elems)},
                     num_meshes, s);
  // Step 1 by vertex bands, or by scattered byte stores beside the
  // bucket-digit histograms of the stable sort of (record, id | used << 31)
  // by the buckets of (mesh id, record)
  BandPlan bp;
  uint32_t* band_tab = nullptr;
  if (split_applies(v, L, n, K) && etab) {
    const BandPlan want = batch_band_plan(n, m, K + 1, num_meshes);
    const int64_t used = v.split_mesh.scratch(n, group_ranges).words;
    if (want.mode != kBandNone && used + int64_t(want.words()) <= n * int64_t(K)) {
      bp = want;
      band_tab = reinterpret_cast<uint32_t*>(ws + L.uniq) + used;
    }
  }
  const bool bands = bp.mode == kMarkAndMap;
  uint32_t* ipart = reinterpret_cast<uint32_t*>(out_idx);
  uint32_t* itable = band_tab;
  uint32_t* itile_valid = itable + size_t(bp.nb) * size_t(bp.itiles);
  uint32_t* ptable = itile_valid + bp.itiles;
  const BandArgs ba{idx, m, arity, n, nullptr, bp.shift, bp.nb, aligned(idx, 16) ? 1 : 0, 1, bp.itiles, 1,
                    ipart, itable, itile_valid, used_v, status, vtx_offsets, elem_offsets, etab, num_meshes};
  if (bands) {
    prof_mark("band_partition", s);
    launch_band_partition(ba, s);
  }
  const MarkArgs mark{idx, m, arity, n, vtx_offsets, elem_offsets, num_meshes, etab, nullptr, used_v, status};
  const bool scatter_mark = m > 0 && !bands;
  uint32_t* X = buf[0];
  uint32_t* Y = buf[1];
  int gp = 0;  // index of the pass in the call (look-back buffer parity, tag)
  GroupArgs g{};
  g.n = n;
  g.rep = reinterpret_cast<uint32_t*>(rep);
  g.cmap = cmap;
  g.uelems = buf[2];
  g.status = status;
  g.mesh_off = ordered;
  g.mesh_tab = vtab;
  g.mesh_buckets = mbk;
  g.nmesh = num_meshes;
  const LargeBuckets large = large_buckets(n, reinterpret_cast<uint32_t*>(ws + L.used_g), &g);
  if (bucketed) {
    bs.args.vtx = static_cast<const uint32_t*>(vtx);
    bs.args.used = used_v;
    bs.args.elems = X;
    bs.args.mesh_off = ordered;
    bs.args.mesh_tab = vtab;
    bs.args.mesh_buckets = mbk;
    bs.args.nmesh = num_meshes;
    g.pairs = reinterpret_cast<uint2*>(Y);
    group_chunks = bs.chunks;
    group_range_sums = bs.range_sums;
    group_buckets(bs, v.bucket_mesh, scatter_mark ? &mark : nullptr, bands ? &ba : nullptr, g, large, s);
  } else {
    if (bands) {
      prof_mark("band_mark", s);
      launch_band_mark(ba, true, s);
    }
    prof_mark(scatter_mark ? "mark_histogram" : "hash_histogram", s);
    v.hash_mesh_hist(scatter_mark ? &mark : nullptr, static_cast<const uint32_t*>(vtx), n, ordered, num_meshes,
                     vtab, mbk, ph, hist_hash, s);
    prof_mark("scan_buckets", s);
    v.scan(hist_hash, ph, n, nullptr, dead_hash, s);
    const SortBuffers sbh{{buf[0], buf[1]}, plan_hash, ph};
    for (int p = 0; p < ph; ++p, ++gp) {
      SortPassArgs a{};
      a.vtx = static_cast<const uint32_t*>(vtx);
      a.bufs = sbh;
      a.pass = p;
      a.used = used_v;
      a.bucket_base = hist_hash + size_t(p) * v.radix();
      a.lookback = wide ? static_cast<void*>(lookback) : static_cast<void*>(lb32[gp & 1]);
      a.lookback_next = lb32[(gp + 1) & 1];
      a.tile_counter = next_counter();
      a.ctl = ctl;
      a.status = status;
      a.n = n;
      a.mesh_off = ordered;
      a.mesh_tab = vtab;
      a.mesh_buckets = mbk;
      a.nmesh = num_meshes;
      a.lo_word = a.hi_word = -1;
      a.shift = p * v.D;
      a.tag = uint32_t(gp + 1);
      prof_mark(p == 0 ? "onesweep_hash_first" : "onesweep_hash", s);
      v.pass(a, p == 0 ? kPassFirstHashMesh : kPassHashMesh, wide, L.tiles_sort, s);
    }
    X = buf[(ph - 1) & 1];
    Y = buf[((ph - 1) & 1) ^ 1];
    // group each bucket by (mesh id, record)
    g.elems = X;
    g.pairs = reinterpret_cast<uint2*>(Y);
    g.chunks = group_chunks;
    g.range_sums = group_range_sums;
    g.ranges = group_ranges;
    g.over = group_chunks + L.tiles_group;
    prof_mark("group", s);
    v.group_mesh(g, L.tiles_group, s);
    prof_mark("group_over", s);
    v.group_over_mesh(g, large, L.tiles_group, s);
  }
  uint2* pairs = reinterpret_cast<uint2*>(Y);

  OrderArgs o{};
  o.X = X;
  o.C = buf[2];
  o.scratch = reinterpret_cast<uint32_t*>(ws + L.uniq);
  o.chunks = group_chunks;
  o.range_sums = group_range_sums;
  o.ranges = group_ranges;
  o.cmap = cmap;
  o.out_vtx = static_cast<uint32_t*>(out_vtx);
  o.ctl = ctl;
  o.status = status;
  o.hist = hist;
  o.plan = plan;
  o.lookback = lookback;
  o.wide = wide;
  o.counter = claimed ? counters + counter : nullptr;
  o.gp = gp;
  o.vtx_off = vtx_offsets;
  o.mesh_tab = vtab;
  o.nmesh = num_meshes;
  o.out_off = out_vtx_offsets;
  order_used_groups(v, L, n, K, o, s);

  // Step 4's map and new2old, both mesh-local, remap
  if (bands) {
    const PairPartArgs pa{static_cast<const uint2*>(pairs), cmap, n, bp.shift, bp.nb, bp.ptiles,
                          reinterpret_cast<uint2*>(X), ptable, status,
                          reinterpret_cast<const uint32_t*>(rep), new2old, g.over_any, SortBuffers{}, 0,
                          vtx_offsets, out_vtx_offsets, vtab, num_meshes};
    prof_mark("pair_partition", s);
    launch_pair_partition(pa, true, s);
    const BandMapArgs ma{reinterpret_cast<const uint2*>(X), ptable, bp.ptiles, ipart, itable, bp.itiles, n,
                         bp.shift, bp.nb, old2new, reinterpret_cast<int32_t*>(buf[2]), SortBuffers{}, 0};
    prof_mark("band_map", s);
    launch_band_map(ma, true, s);
    const BandRemapArgs ra{ipart, reinterpret_cast<const int32_t*>(buf[2]), itile_valid, m, arity, nullptr, out_idx,
                           SortBuffers{}, 0};
    prof_mark("band_remap", s);
    launch_band_remap(ra, bp.itiles, true, s);
    prof_mark(nullptr, s);
    return check_launch();
  }
  prof_mark("old2new", s);
  launch_scatter_old2new<true>(s, new2old && !few_used(n, m), SortBuffers{{nullptr, nullptr}, nullptr, 0},
                               static_cast<const uint2*>(pairs), cmap,
                               n, vtx_offsets, static_cast<const int64_t*>(out_vtx_offsets), num_meshes,
                               static_cast<const int32_t*>(vtab), old2new, reinterpret_cast<const uint32_t*>(rep),
                               new2old, static_cast<const uint32_t*>(g.over_any));
  if (m > 0) {
    prof_mark("remap", s);
    hipLaunchKernelGGL((k_remap<true>), dim3(rand_grid(m)), dim3(kRandBlock), 0, s, idx, m, arity, n, vtx_offsets,
                       elem_offsets, num_meshes, static_cast<const int32_t*>(etab),
                       static_cast<const int64_t*>(nullptr), old2new, out_idx);
  }
  prof_mark(nullptr, s);
  return check_launch();
}

// Device address of `scratch` on the current device, looked up once per
// device (the first call on that device) and kept.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

mrx_status scratch_of_current_device(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return MRX_ERR_HIP;
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return MRX_ERR_HIP;
    g_scratch_addr[dev] = p;
  }
  *out = g_scratch_addr[dev];
  return MRX_OK;
}

}  // namespace
}  // namespace mrx

using namespace mrx;

extern "C" {

int32_t mrx_abi_version(void) { return MRX_ABI_VERSION; }

const char* mrx_status_string(int32_t s) {
  switch (s) {
    case MRX_OK: return "MRX_OK";
    case MRX_ERR_INVALID_ARGUMENT: return "MRX_ERR_INVALID_ARGUMENT";
    case MRX_ERR_WORKSPACE_TOO_SMALL: return "MRX_ERR_WORKSPACE_TOO_SMALL";
    case MRX_ERR_INDEX_OUT_OF_RANGE: return "MRX_ERR_INDEX_OUT_OF_RANGE";
    case MRX_ERR_TOO_LARGE: return "MRX_ERR_TOO_LARGE";
    case MRX_ERR_HIP: return "MRX_ERR_HIP";
    case MRX_ERR_UNSUPPORTED: return "MRX_ERR_UNSUPPORTED";
    case MRX_ERR_INTERNAL: return "MRX_ERR_INTERNAL";
    case MRX_ERR_NOALLOC_TOO_LARGE: return "MRX_ERR_NOALLOC_TOO_LARGE";
    default: return "MRX_UNKNOWN_STATUS";
  }
}

int32_t mrx_tuning_count(int32_t vtx_bytes) {
  if (vtx_bytes < 4 || vtx_bytes > 64 || vtx_bytes % 4) return 0;
  return int32_t(variants_for(vtx_bytes / 4).size());
}

mrx_status mrx_tuning_get(int32_t vtx_bytes, int32_t i, mrx_tuning* out) {
  if (!out || i < 0 || i >= mrx_tuning_count(vtx_bytes)) return MRX_ERR_INVALID_ARGUMENT;
  const SortVariant& v = variants_for(vtx_bytes / 4)[i];
  out->digit_bits = v.D;
  out->block_threads = v.block;
  out->items_per_thread = v.ipt;
  out->flags = 0;
  return MRX_OK;
}

mrx_status mrx_profile_enable(int32_t on) {
  Profiler& p = profiler();
  std::lock_guard<std::mutex> g(p.mu);
  if (on) {
    p.recs.clear();
    p.next = 0;
  }
  p.on = on != 0;
  return MRX_OK;
}

// Named marks, each followed by the mark that ends its kernel.
static std::vector<std::pair<size_t, size_t>> prof_pairs(const Profiler& p) {
  std::vector<std::pair<size_t, size_t>> out;
  for (size_t i = 0; i + 1 < p.recs.size(); ++i)
    if (p.recs[i].name) out.emplace_back(i, i + 1);
  return out;
}

int32_t mrx_profile_count(void) {
  Profiler& p = profiler();
  std::lock_guard<std::mutex> g(p.mu);
  return int32_t(prof_pairs(p).size());
}

mrx_status mrx_profile_get(int32_t i, const char** name, float* ms) {
  Profiler& p = profiler();
  ProfRecord a, b;
  {
    std::lock_guard<std::mutex> g(p.mu);
    const auto pairs = prof_pairs(p);
    if (i < 0 || size_t(i) >= pairs.size() || !ms) return MRX_ERR_INVALID_ARGUMENT;
    a = p.recs[pairs[size_t(i)].first];
    b = p.recs[pairs[size_t(i)].second];
  }
  if (name) *name = a.name;
  if (hipEventSynchronize(b.event) != hipSuccess) return MRX_ERR_HIP;
  return hipEventElapsedTime(ms, a.event, b.event) == hipSuccess ? MRX_OK : MRX_ERR_HIP;
}

mrx_status mrx_reindex_workspace_size(int64_t num_vtx, int32_t vtx_bytes, int64_t num_idx,
                                      int32_t num_meshes, const mrx_tuning* tuning, size_t* bytes) {
  if (!bytes) return MRX_ERR_INVALID_ARGUMENT;
  if (vtx_bytes < 4 || vtx_bytes > 64 || vtx_bytes % 4 != 0) return MRX_ERR_INVALID_ARGUMENT;
  if (num_vtx < 0 || num_idx < 0 || num_meshes < 1) return MRX_ERR_INVALID_ARGUMENT;
  if (num_vtx > kMaxCount || num_idx > kMaxCount) return MRX_ERR_TOO_LARGE;
  const SortVariant* v = pick_variant(vtx_bytes / 4, tuning);
  if (!v) return MRX_ERR_UNSUPPORTED;
  *bytes = make_layout(num_vtx, num_idx, vtx_bytes / 4, num_meshes, *v, tuning).total;
  return MRX_OK;
}


mrx_status mrx_reindex_mesh(const void* vtx, int64_t num_vtx, int32_t vtx_bytes, const int32_t* idx,
                            int64_t num_elems, int32_t arity, void* out_vtx, int32_t* out_idx,
                            int32_t* old2new, int32_t* new2old, int64_t* out_num_vtx,
                            int32_t* dev_status, void* workspace, size_t workspace_bytes,
                            const mrx_tuning* tuning, void* stream) {
  const SortVariant* v = nullptr;
  Layout L;
  mrx_status st = validate_single(vtx, num_vtx, vtx_bytes, idx, num_elems, arity, out_vtx, out_idx, old2new,
                                  new2old, out_num_vtx, dev_status, workspace, workspace_bytes, tuning, {},
                                  &v, &L);
  if (st != MRX_OK) return st;
  return launch_single(*v, L, vtx, num_vtx, vtx_bytes, idx, num_elems, arity, nullptr, out_vtx, out_idx,
                       old2new, new2old, out_num_vtx, dev_status, workspace, tuning, stream);
}

mrx_status mrx_reindex_mesh_noalloc(const void* vtx, int64_t num_vtx, int32_t vtx_bytes, const int32_t* idx,
                                    int64_t num_elems, int32_t arity, void* out_vtx, int32_t* out_idx,
                                    int32_t* old2new, int32_t* new2old, int64_t* out_num_vtx,
                                    int32_t* dev_status, const mrx_tuning* tuning, void* stream) {
  // the stream must belong to the current device: its kernels get that
  // device's copy of the array
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess) return MRX_ERR_HIP;
  if (stream) {
    hipDevice_t sd = -1;
    if (hipStreamGetDevice(reinterpret_cast<hipStream_t>(stream), &sd) != hipSuccess) return MRX_ERR_HIP;
    if (int(sd) != cur) return MRX_ERR_INVALID_ARGUMENT;
  }
  void* ws = nullptr;
  mrx_status st = scratch_of_current_device(&ws);
  if (st != MRX_OK) return st;
  const SortVariant* v = nullptr;
  Layout L;
  st = validate_single(vtx, num_vtx, vtx_bytes, idx, num_elems, arity, out_vtx, out_idx, old2new, new2old,
                       out_num_vtx, dev_status, ws, MRX_NOALLOC_SCRATCH_BYTES, tuning, {}, &v, &L);
  if (st == MRX_ERR_WORKSPACE_TOO_SMALL) return MRX_ERR_NOALLOC_TOO_LARGE;
  if (st != MRX_OK) return st;
  return launch_single(*v, L, vtx, num_vtx, vtx_bytes, idx, num_elems, arity, nullptr, out_vtx, out_idx,
                       old2new, new2old, out_num_vtx, dev_status, ws, tuning, stream);
}

mrx_status mrx_reindex_mesh_batched(const void* vtx, const int64_t* vtx_offsets, int64_t total_vtx,
                                    int32_t vtx_bytes, const int32_t* idx, const int64_t* elem_offsets,
                                    int64_t total_elems, int32_t arity, int32_t num_meshes,
                                    void* out_vtx, int64_t* out_vtx_offsets, int32_t* out_idx,
                                    int32_t* old2new, int32_t* new2old, int32_t* dev_status,
                                    void* workspace, size_t workspace_bytes,
                                    const mrx_tuning* tuning, void* stream_) {
  mrx_status st = validate_common(vtx, total_vtx, vtx_bytes, idx, total_elems, arity, out_vtx, out_idx,
                                  old2new, workspace, workspace_bytes);
  if (st != MRX_OK) return st;
  if (num_meshes < 1 || !vtx_offsets || !elem_offsets || !out_vtx_offsets ||
      !aligned(vtx_offsets, 8) || !aligned(elem_offsets, 8) || !aligned(out_vtx_offsets, 8) ||
      !aligned(new2old, 4) || !dev_status || !aligned(dev_status, 4))
    return MRX_ERR_INVALID_ARGUMENT;
  const int K = vtx_bytes / 4;
  const SortVariant* vp = pick_variant(K, tuning);
  if (!vp) return MRX_ERR_UNSUPPORTED;
  const SortVariant& v = *vp;
  const int64_t n = total_vtx, m = total_elems * arity;
  const Layout L = make_layout(n, m, K, num_meshes, v, tuning);
  if (workspace_bytes < L.total) return MRX_ERR_WORKSPACE_TOO_SMALL;
  const size_t vb = size_t(n) * vtx_bytes, ib = size_t(m) * 4, nb = size_t(n) * 4,
               ob = size_t(num_meshes + 1) * 8;
  if (!disjoint({{vtx, vb}, {out_vtx, vb}, {old2new, nb}, {new2old, new2old ? nb : 0},
                 {out_vtx_offsets, ob}, {dev_status, 4u}, {workspace, L.total},
                 {vtx_offsets, ob}, {elem_offsets, ob}, {idx == out_idx ? nullptr : idx, ib}}) ||
      !disjoint({{out_idx, ib}, {vtx, vb}, {out_vtx, vb}, {old2new, nb}, {new2old, new2old ? nb : 0},
                 {out_vtx_offsets, ob}, {dev_status, 4u}, {workspace, L.total},
                 {vtx_offsets, ob}, {elem_offsets, ob}}) ||
      (idx != out_idx && overlaps(idx, ib, out_idx, ib)))  // in place, or not at all
    return MRX_ERR_INVALID_ARGUMENT;

  if (L.mesh_hash)
    return launch_batched_hash(v, L, vtx, vtx_offsets, n, vtx_bytes, idx, elem_offsets, total_elems, arity,
                               num_meshes, out_vtx, out_vtx_offsets, out_idx, old2new, new2old, dev_status,
                               workspace, tuning, stream_);
  hipStream_t s = reinterpret_cast<hipStream_t>(stream_);
  char* ws = static_cast<char*>(workspace);
  Control* ctl = reinterpret_cast<Control*>(ws + L.ctl);
  uint32_t* counters = reinterpret_cast<uint32_t*>(ws + L.counters);
  uint32_t* hist = reinterpret_cast<uint32_t*>(ws + L.hist);
  uint32_t* plan = reinterpret_cast<uint32_t*>(ws + L.plan);
  uint64_t* lookback = reinterpret_cast<uint64_t*>(ws + L.lookback);
  uint64_t* scan_lookback = reinterpret_cast<uint64_t*>(ws + L.scan_lookback);
  const bool wide = wide_lookback(n, tuning);
  const bool claimed = tuning && (tuning->flags & MRX_TUNING_CLAIMED_TILES);
  uint32_t* const lb32[2] = {reinterpret_cast<uint32_t*>(lookback),
                             reinterpret_cast<uint32_t*>(lookback) + size_t(L.tiles_sort) * v.radix()};
  uint8_t* used_v = reinterpret_cast<uint8_t*>(ws + L.used_v);
  uint8_t* used_g = reinterpret_cast<uint8_t*>(ws + L.used_g);
  uint32_t* buf[2] = {reinterpret_cast<uint32_t*>(ws + L.buf_a), reinterpret_cast<uint32_t*>(ws + L.buf_b)};
  uint32_t* uniq = reinterpret_cast<uint32_t*>(ws + L.uniq);
  int32_t* rep = reinterpret_cast<int32_t*>(ws + L.rep);
  int32_t* cmap = reinterpret_cast<int32_t*>(ws + L.cmap);
  int32_t* status = dev_status;
  const int P = L.P_key + L.P_mesh;
  int32_t* vtab = L.vtx_tab_n ? reinterpret_cast<int32_t*>(ws + L.vtx_tab) : nullptr;
  int32_t* etab = L.elem_tab_n ? reinterpret_cast<int32_t*>(ws + L.elem_tab) : nullptr;

  prof_mark("fill_zero", s);
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(int64_t(L.zero_end / 16), 256, 4096)), dim3(256), 0, s,
                     reinterpret_cast<uint4*>(ws), int64_t(L.zero_end / 16), dev_status,
                     static_cast<int64_t*>(nullptr), static_cast<int64_t*>(nullptr));
  if (n <= 0) vtab = nullptr;
  if (total_elems <= 0) etab = nullptr;
  if (vtab || etab) prof_mark("mesh_tables", s);
  launch_mesh_tables({vtx_offsets, n, vtab, vtab ? L.vtx_tab_n : 0},
                     {elem_offsets, total_elems, etab, mesh_table_size(total_elems)}, num_meshes, s);
  const MarkArgs mark{idx, m, arity, n, vtx_offsets, elem_offsets, num_meshes, etab, nullptr, used_v, status};
  const bool fused = v.mark_hist_applies(n, m);
  if (fused) {
    prof_mark("mark_histogram", s);
    v.mark_hist(mark, true, static_cast<const uint32_t*>(vtx), n, hist, s);
  } else if (m > 0) {
    prof_mark("mark_used", s);
    hipLaunchKernelGGL((k_mark_used<true>), dim3(rand_grid(m)), dim3(kRandBlock), 0, s, mark);
  }
  if (n > 0) {
    if (!fused) {
      prof_mark("histogram", s);
      v.hist(static_cast<const uint32_t*>(vtx), n, hist, s);
    }
    prof_mark("mesh_histogram", s);
    v.mesh_hist(vtx_offsets, num_meshes, L.P_mesh, hist + size_t(L.P_key) * v.radix(), s);
    prof_mark("scan_buckets", s);
    v.scan(hist, P, n, nullptr, plan + P + 1, s);
    const SortBuffers sb{{buf[0], buf[1]}, plan, P};
    for (int p = 0; p < P; ++p) {
      SortPassArgs a{};
      a.vtx = static_cast<const uint32_t*>(vtx);
      a.bufs = sb;
      a.pass = p;
      a.used = used_v;
      a.bucket_base = hist + size_t(p) * v.radix();
      a.lookback = wide ? static_cast<void*>(lookback) : static_cast<void*>(lb32[p & 1]);
      a.lookback_next = lb32[(p + 1) & 1];
      a.tile_counter = claimed ? counters + p : nullptr;
      a.ctl = ctl;
      a.status = status;
      a.n = n;
      a.mesh_off = vtx_offsets;
      a.mesh_tab = vtab;
      a.nmesh = num_meshes;
      a.tag = uint32_t(p + 1);
      int mode = kPassKey;
      if (p < L.P_key) {
        set_digit(a, K, p * v.D);
        if (p == 0) mode = kPassFirst;
      } else {
        a.shift = (p - L.P_key) * v.D;
        mode = kPassMesh;
      }
      prof_mark(mode == kPassFirst ? "onesweep_first" : mode == kPassMesh ? "onesweep_mesh" : "onesweep", s);
      v.pass(a, mode, wide, L.tiles_sort, s);
    }
    FlagScanArgs f{};
    f.bufs = sb;
    f.n = n;
    f.uniq = uniq;
    f.rep = rep;
    f.used_g = used_g;
    f.lookback = scan_lookback;
    f.tile_counter = claimed ? counters + P : nullptr;
    f.ctl = ctl;
    f.status = status;
    f.mesh_off = vtx_offsets;
    f.mesh_tab = vtab;
    f.nmesh = num_meshes;
    f.tag = uint32_t(P + 1);
    prof_mark("flag_scan", s);
    v.flag_scan(f, true, L.tiles_scan, s);
    CompactArgs c{};
    c.used_g = used_g;
    c.uniq = uniq;
    c.rep = rep;
    c.K = K;
    c.out_vtx = static_cast<uint32_t*>(out_vtx);
    c.new2old = new2old;
    c.cmap = cmap;
    c.out_num = &ctl->num_used;
    c.cap = n;
    c.lookback = scan_lookback;
    c.tile_counter = claimed ? counters + P + 1 : nullptr;
    c.ctl = ctl;
    c.status = status;
    c.tag = uint32_t(P + 2);
    prof_mark("compact", s);
    hipLaunchKernelGGL((k_compact<kScanBlock, kScanIpt>), dim3(L.tiles_scan), dim3(kScanBlock), 0, s, c);
    prof_mark("batch_offsets", s);
    hipLaunchKernelGGL(k_batch_offsets, dim3((num_meshes + 1 + 255) / 256), dim3(256), 0, s, vtx_offsets,
                       num_meshes, sb, static_cast<const int32_t*>(cmap), static_cast<const Control*>(ctl),
                       static_cast<const int64_t*>(&ctl->num_used), n, out_vtx_offsets);
    prof_mark("old2new", s);
    launch_scatter_old2new<true>(s, false, sb, static_cast<const uint2*>(nullptr), cmap, n, vtx_offsets,
                                 out_vtx_offsets, num_meshes, static_cast<const int32_t*>(vtab), old2new,
                                 static_cast<const uint32_t*>(nullptr), static_cast<int32_t*>(nullptr),
                                 static_cast<const uint32_t*>(nullptr));
    if (new2old) {
      prof_mark("localize_new2old", s);
      hipLaunchKernelGGL(k_localize_new2old, dim3(grid_for(n, 256)), dim3(256), 0, s, new2old,
                         &ctl->num_used, vtx_offsets, num_meshes, static_cast<const int32_t*>(vtab));
    }
  } else {
    prof_mark("batch_offsets", s);
    hipLaunchKernelGGL(k_batch_offsets, dim3((num_meshes + 1 + 255) / 256), dim3(256), 0, s, vtx_offsets,
                       num_meshes, SortBuffers{{nullptr, nullptr}, nullptr, 0}, static_cast<const int32_t*>(cmap),
                       static_cast<const Control*>(ctl), static_cast<const int64_t*>(&ctl->num_used), n,
                       out_vtx_offsets);
  }
  if (m > 0) {
    prof_mark("remap", s);
    hipLaunchKernelGGL((k_remap<true>), dim3(rand_grid(m)), dim3(kRandBlock), 0, s, idx, m, arity, n,
                       vtx_offsets, elem_offsets, num_meshes, static_cast<const int32_t*>(etab),
                       static_cast<const int64_t*>(nullptr), old2new, out_idx);
  }
  prof_mark(nullptr, s);
  return check_launch();
}

mrx_status mrx_merge_meshes(const void* vtx, const int64_t* vtx_offsets, int64_t total_vtx, int32_t vtx_bytes,
                            const int32_t* idx, const int64_t* elem_offsets, int64_t total_elems,
                            int32_t arity, int32_t num_meshes, void* out_vtx, int32_t* out_idx,
                            int32_t* old2new, int32_t* new2old, int64_t* out_num_vtx, int32_t* dev_status,
                            void* workspace, size_t workspace_bytes, const mrx_tuning* tuning,
                            void* stream) {
  if (num_meshes < 1 || !vtx_offsets || !elem_offsets || !aligned(vtx_offsets, 8) ||
      !aligned(elem_offsets, 8))
    return MRX_ERR_INVALID_ARGUMENT;
  const size_t ob = sizeof(int64_t) * (size_t(num_meshes) + 1);
  const SortVariant* v = nullptr;
  Layout L;
  mrx_status st = validate_single(vtx, total_vtx, vtx_bytes, idx, total_elems, arity, out_vtx, out_idx,
                                  old2new, new2old, out_num_vtx, dev_status, workspace, workspace_bytes,
                                  tuning, {{vtx_offsets, ob}, {elem_offsets, ob}}, &v, &L);
  if (st != MRX_OK) return st;
  // the offsets must not overlap each other either
  if (overlaps(vtx_offsets, ob, elem_offsets, ob)) return MRX_ERR_INVALID_ARGUMENT;
  const int64_t m = total_elems * arity;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  if (m > 0) {
    int32_t* etab = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + L.elem_tab);
    prof_mark("mesh_tables", s);
    launch_mesh_tables({elem_offsets, total_elems, etab, mesh_table_size(total_elems)}, {}, num_meshes, s);
    prof_mark("offset_indices", s);
    hipLaunchKernelGGL(k_offset_indices, dim3((m + 255) / 256), dim3(256), 0, s, idx, m, arity, vtx_offsets,
                       elem_offsets, num_meshes, static_cast<const int32_t*>(etab), out_idx);
  }
  return launch_single(*v, L, vtx, total_vtx, vtx_bytes, out_idx, total_elems, arity, nullptr, out_vtx,
                       out_idx, old2new, new2old, out_num_vtx, dev_status, workspace, tuning, stream);
}

mrx_status mrx_extract_submesh(const void* vtx, int64_t num_vtx, int32_t vtx_bytes, const int32_t* idx,
                               int64_t num_elems, int32_t arity, const uint8_t* keep, void* out_vtx,
                               int32_t* out_idx, int64_t* out_num_elems, int32_t* old2new, int32_t* new2old,
                               int64_t* out_num_vtx, int32_t* dev_status, void* workspace,
                               size_t workspace_bytes, const mrx_tuning* tuning, void* stream) {
  if (!out_num_elems || !aligned(out_num_elems, 8)) return MRX_ERR_INVALID_ARGUMENT;
  if (num_elems > 0 && (!keep || idx == out_idx)) return MRX_ERR_INVALID_ARGUMENT;
  const SortVariant* v = nullptr;
  Layout L;
  mrx_status st = validate_single(vtx, num_vtx, vtx_bytes, idx, num_elems, arity, out_vtx, out_idx, old2new,
                                  new2old, out_num_vtx, dev_status, workspace, workspace_bytes, tuning,
                                  {{keep, size_t(num_elems)}, {out_num_elems, 8}}, &v, &L);
  if (st != MRX_OK) return st;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  Control* ctl = reinterpret_cast<Control*>(ws + L.ctl);
  // per-call state for the selection and the re-index that follows it
  prof_mark("fill_zero", s);
  hipLaunchKernelGGL(k_fill_zero, dim3(grid_for(int64_t(L.zero_end / 16), 256, 4096)), dim3(256), 0, s,
                     reinterpret_cast<uint4*>(ws), int64_t(L.zero_end / 16), dev_status, out_num_vtx,
                     out_num_elems);
  if (num_elems > 0) {
    SelectArgs a{};
    a.keep = keep;
    a.idx = idx;
    a.num_elems = num_elems;
    a.arity = arity;
    a.out = out_idx;
    a.out_count = out_num_elems;
    a.lookback = reinterpret_cast<uint64_t*>(ws + L.elem_lookback);
    a.tile_counter = (tuning && (tuning->flags & MRX_TUNING_CLAIMED_TILES))
                         ? reinterpret_cast<uint32_t*>(ws + L.counters) + L.P_key + L.P_mesh + L.P_hash + 7
                         : nullptr;
    a.ctl = ctl;
    a.status = dev_status;
    a.tag = 1;
    const int64_t tiles = (num_elems + kSelectTile - 1) / kSelectTile;
    prof_mark("select_elements", s);
    hipLaunchKernelGGL((k_select_elements<kSelectBlock, kSelectIpt>), dim3(tiles), dim3(kSelectBlock), 0, s, a);
  }
  return launch_single(*v, L, vtx, num_vtx, vtx_bytes, out_idx, num_elems, arity, out_num_elems, out_vtx,
                       out_idx, old2new, new2old, out_num_vtx, dev_status, workspace, tuning, stream,
                       /*state_zeroed=*/true);
}

}  // extern "C"
