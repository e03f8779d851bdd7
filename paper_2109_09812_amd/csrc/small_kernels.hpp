// A small mesh in one launch.
//
// The general launch sequence costs a dozen dependent launches, 5-10 us each
// however few vertices there are. A mesh whose vertices fit the LDS of one
// workgroup is re-indexed by that workgroup alone: used bits and a table of
// distinct records in LDS, the used ones ordered by the block sort of
// split_kernels.hpp, both maps and the remap from LDS. Nothing in the
// workspace is touched and nothing needs clearing. Bound by the one
// workgroup's chain of LDS steps and memory round trips: 1,689 12-byte vertices
// and 1,536 entries take 15 us, where the sort of all vertices by key
// bytes that served them took 154 us of kernels in 20 launches.
#pragma once

#include "band_kernels.hpp"
#include "scan_kernels.hpp"
#include "split_kernels.hpp"

namespace mrx {

template <int K>
struct SmallShape {
  using SH = SplitShape<K>;
  static constexpr int BLOCK = SH::BLOCK, CAP = SH::CAP, E = SH::E;
  static constexpr int TB = CAP > 3072 ? 13 : CAP > 1536 ? 12 : 11;  // table: at least 4/3 CAP slots
  static constexpr int TS = 1 << TB;
  static_assert(TS * 3 >= CAP * 4, "table load");
  // most index entries: the one workgroup reads them twice, 2,048 at a time,
  // about 1 us each; beyond this the marking and remap of a full grid pay
  // for their launches
  static constexpr int MAX_ENTRIES = 8 * CAP;
};

struct SmallArgs {
  const uint32_t* vtx;         // [n][K]
  int32_t n;                   // <= CAP
  const int32_t* idx;          // [m], may be out_idx
  int32_t m;                   // capacity in entries
  int32_t arity;
  const int64_t* live_elems;   // device, nullable
  uint32_t* out_vtx;
  int32_t* out_idx;
  int32_t* old2new;
  int32_t* new2old;            // nullable
  int64_t* out_num;
  int32_t* status;             // receives MRX_OK or the index error, unless `keep_status`
  int32_t keep_status;         // an earlier step of the call owns the status word: only raise it
};

template <int K>
__global__ __launch_bounds__(SmallShape<K>::BLOCK) void k_small(SmallArgs a) {
  using SH = SmallShape<K>;
  constexpr int BLOCK = SH::BLOCK, CAP = SH::CAP, E = SH::E, TS = SH::TS, TB = SH::TB, NW = K + 1;
  constexpr uint32_t kEmpty = 0xFFFFFFFFu, kUsedBit = 0x80000000u;
  constexpr uint16_t kUnused = 0xFFFFu;
  constexpr int UN = 4;
  __shared__ SortLds<NW, CAP> lds;
  __shared__ uint32_t s_key[K * CAP];      // records, word-major
  __shared__ uint32_t s_tab[TS];           // smallest vertex of a distinct record, bit 31: used
  __shared__ uint32_t s_used[CAP / 32];
  __shared__ uint16_t s_map[CAP];          // new id: of representatives, then of every vertex
  __shared__ uint32_t s_n, s_bad;
  const int tid = threadIdx.x;
  const int n = a.n;
  const int m = int(live_entries(a.live_elems, a.m, a.arity));
  if (tid == 0) s_n = s_bad = 0;
  for (int i = tid; i < TS; i += BLOCK) s_tab[i] = kEmpty;
  for (int i = tid; i < CAP / 32; i += BLOCK) s_used[i] = 0;
  for (int t = tid; t < n * K; t += BLOCK) {
    const int v = t / K, w = t - v * K;
    s_key[w * CAP + v] = a.vtx[t];
  }
  __syncthreads();
  // ---- Step 1: used bits
  bool bad = false;
  for (int k0 = 0; k0 < m; k0 += UN * BLOCK) {
    int32_t v[UN];
#pragma unroll
    for (int r = 0; r < UN; ++r) {
      const int k = k0 + r * BLOCK + tid;
      v[r] = k < m ? a.idx[k] : -1;
    }
#pragma unroll
    for (int r = 0; r < UN; ++r) {
      if (k0 + r * BLOCK + tid >= m) continue;
      if (v[r] < 0 || v[r] >= n) bad = true;
      else atomicOr(&s_used[v[r] >> 5], 1u << (v[r] & 31));
    }
  }
  if (bad) s_bad = 1;
  // ---- distinct records, named by their smallest vertex
  uint32_t slot[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    slot[i] = 0;
    if (q >= n) continue;
    uint32_t key[K];
#pragma unroll
    for (int w = 0; w < K; ++w) key[w] = s_key[w * CAP + q];
    uint32_t sl = (hash_words<K>(key) * 0x9E3779B1u) >> (32 - TB);
    for (int probe = 0; probe < TS; ++probe) {
      uint32_t cur = s_tab[sl];
      if (cur == kEmpty) {
        cur = atomicCAS(&s_tab[sl], kEmpty, uint32_t(q));
        if (cur == kEmpty) break;
      }
      if (lds_keys_equal<K>(s_key, int(cur), q, CAP)) {
        atomicMin(&s_tab[sl], uint32_t(q));
        break;
      }
      sl = (sl + 1) & (TS - 1);
    }
    slot[i] = sl;
  }
  __syncthreads();
  uint32_t heads = 0;  // bit i: vertex i * BLOCK + tid is its record's smallest copy
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    if (q >= n) continue;
    if ((s_tab[slot[i]] & ~kUsedBit) == uint32_t(q)) heads |= 1u << i;
    if (s_used[q >> 5] >> (q & 31) & 1u) atomicOr(&s_tab[slot[i]], kUsedBit);
  }
  __syncthreads();
  // ---- Steps 2-3: the used ones in order
#pragma unroll
  for (int i = 0; i < E; ++i)
    if ((heads >> i & 1u) && (s_tab[slot[i]] & kUsedBit)) lds.x[atomicAdd(&s_n, 1u)] = uint32_t(i * BLOCK + tid);
  __syncthreads();
  const int u = int(s_n);
  uint32_t e[E][NW];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    if (q >= u) continue;
    const uint32_t v = lds.x[q];
#pragma unroll
    for (int w = 0; w < K; ++w) e[i][w] = s_key[w * CAP + v];
    e[i][K] = v;
  }
  if (u > 0) block_sort<K, NW, CAP, BLOCK, E>(e, u, lds);
  for (int t = tid; t < u * K; t += BLOCK) {
    const int q = t / K, w = t - q * K;
    a.out_vtx[t] = lds.x[w * CAP + q];
  }
  for (int q = tid; q < u; q += BLOCK) {
    const uint32_t v = lds.x[K * CAP + q];
    if (a.new2old) a.new2old[q] = int32_t(v);
    s_map[v] = uint16_t(q);
  }
  __syncthreads();
  // ---- Step 4
  uint16_t c[E];
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    if (q >= n) continue;
    const uint32_t t = s_tab[slot[i]];
    c[i] = t & kUsedBit ? s_map[t & ~kUsedBit] : kUnused;
    a.old2new[q] = c[i] == kUnused ? -1 : int32_t(c[i]);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const int q = i * BLOCK + tid;
    if (q < n) s_map[q] = c[i];
  }
  __syncthreads();
  for (int k0 = 0; k0 < m; k0 += UN * BLOCK) {
    int32_t v[UN];
#pragma unroll
    for (int r = 0; r < UN; ++r) {
      const int k = k0 + r * BLOCK + tid;
      v[r] = k < m ? a.idx[k] : -1;
    }
#pragma unroll
    for (int r = 0; r < UN; ++r) {
      const int k = k0 + r * BLOCK + tid;
      if (k >= m) continue;
      const uint16_t x = v[r] >= 0 && v[r] < n ? s_map[v[r]] : kUnused;
      a.out_idx[k] = x == kUnused ? -1 : int32_t(x);
    }
  }
  if (tid == 0) {
    *a.out_num = u;
    if (!a.keep_status) *a.status = s_bad ? kErrIndex : 0;
    else if (s_bad) atomicMax(a.status, kErrIndex);
  }
}

}  // namespace mrx
