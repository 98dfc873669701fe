// Device code of the row gather that more than one kernel is built from.
#pragma once

#include "common.hpp"

namespace lgp {

struct RowShape {
  uint32_t cpr;    // chunks per row
  uint32_t bytes;  // row width
  uint32_t last;   // where the last chunk starts: bytes - size of a chunk
};

// How hits beside misses are copied: group_rows, or flat_rows, which streams rows of whole lines past L2.
enum class HitWalk { kGroups, kFlat, kFlatLines };

// Both kinds of rows in one launch (see split_hits, split_misses).
struct SplitArgs {
  const char* hit_src;
  const char* miss_src;
  char* dst;
  RowShape hit_shape, miss_shape;
  PartLists lists;            // row = nullptr: entry e goes to row e
  const int32_t* counters;    // entries of the lists; nullptr: direct.window holds the entries of list 0 or 1, ids
  DirectIds direct;
  int64_t n_max;
  uint32_t hit_lanes, miss_lanes, hit_blocks, miss_blocks;     // 0 blocks: no such rows
  uint64_t hit_inv;           // of flat_rows
  int32_t hit_epw;
  uint32_t hit_narrow;        // workgroups that take hits where misses are few
  bool peers;
};

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// A row is copied in chunks of sizeof(VecT) bytes.  RAGGED: row width or addresses are no multiple of that; the
// chunks then start at any even address (global loads and stores of any width may), and the last one ends where
// the row ends, overlapping the one before it with the same bytes.  Copying such rows in the widest chunk that
// divides them instead leaves most of a lane's 16 bytes unused: cached rows of 150 bytes (238 k) took 74 us in
// 2-byte chunks and take 20.5, of 602 bytes 296 and 72, of 200 bytes (8-byte chunks) 27.5 and 23.
template <typename VecT, bool RAGGED>
struct Chunk {
  typedef VecT T;
};
template <typename VecT>
struct Chunk<VecT, true> {
  typedef VecT T __attribute__((aligned(2)));
};
template <typename VecT, bool RAGGED>
__device__ __forceinline__ uint32_t chunk_at(const RowShape& r, uint32_t col) {
  const uint32_t at = col * uint32_t(sizeof(VecT));
  return RAGGED ? (at < r.last ? at : r.last) : at;
}

// Called by one workgroup.
__device__ __forceinline__ void direct_stats(const DirectIds& dir, int64_t n) {
  if (dir.stats && threadIdx.x == 0) {
    dir.stats[dir.stats_slot] = int32_t(n > 0 ? n : 0);
    dir.stats[1 - dir.stats_slot] = 0;
  }
}

// Translate one entry of the source-row array; -1 = skip this row.
__device__ __forceinline__ int32_t direct_source(const DirectIds& dir, int32_t entry, bool in_range) {
  if (dir.num_vertices == 0 || !in_range) return in_range ? entry : -1;
  if (uint32_t(entry) >= uint64_t(dir.num_vertices)) {
    atomicOr(dir.d_err, ERR_BAD_ID);
    return -1;
  }
  return dir.remap ? dir.remap[entry] : entry;
}

// ---- rows by lane groups -----------------------------------------------------
// Reads of CPU memory are not cached on the GPU and travel as whole 128-byte lines, so
// a line requested by two different load instructions crosses the link twice.  Here a
// group of `lanes` >= chunks-per-row lanes (a power of two) owns a whole row, so one instruction requests each
// line of the row exactly once; UNROLL rows per group are in flight before the first
// store.  Rows wider than 64 chunks are walked in 64-chunk pieces.  HBM_SOURCE selects the
// variant used for cache hits on rows that straddle lines (cached loads, streaming stores).
// A workgroup pass takes consecutive entries, and so does each of its load instructions: where consecutive entries are
// neighbouring rows, the line that two of them share is requested once.
// The caller is workgroup `block` of `blocks` that share the entries.
template <typename VecT, bool RAGGED, int UNROLL, bool HBM_SOURCE>
__device__ __forceinline__ void group_rows(const char* __restrict__ src, char* __restrict__ dst, const RowShape& shape,
                                           const int32_t* __restrict__ row, const int32_t* __restrict__ srcrow,
                                           int64_t n_max, const int32_t* __restrict__ n_dev, const DirectIds& dir,
                                           uint32_t lanes, uint32_t block, uint32_t blocks) {
  // carried pointers keep their address space only if it is spelled out
  typedef __attribute__((address_space(1))) char Global;
  typedef __attribute__((address_space(1))) typename Chunk<VecT, RAGGED>::T GlobalMem;
  int64_t n = n_dev ? int64_t(*n_dev) : n_max;
  int64_t lo = 0;
  if (dir.window) {
    lo = dir.window[0] < 0 ? 0 : dir.window[0];
    n = dir.window[1];
  }
  if (n > n_max) n = n_max;
  if (block == 0) direct_stats(dir, n - lo);
  const uint32_t groups = 256u / lanes;                       // rows per load instruction of the workgroup
  const uint32_t sub = threadIdx.x & (lanes - 1);
  const int64_t pass = int64_t(groups) * UNROLL;
  // The list entries of the next pass are loaded before the rows of this one, so that a pass waits
  // for one round trip to memory (its rows), not two in a row (entries, then rows).
  int32_t next_src[UNROLL], next_row[UNROLL];
  const int64_t first = lo + int64_t(block) * pass + threadIdx.x / lanes;
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int64_t e = first + u * groups;
    next_src[u] = e < n ? (srcrow ? srcrow[e] : int32_t(e)) : 0;
    next_row[u] = e < n ? (row ? row[e] : int32_t(e)) : 0;
  }
  for (int64_t e0 = first; e0 < n; e0 += int64_t(blocks) * pass) {
    int64_t so[UNROLL], dof[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const bool ok = e0 + u * groups < n;
      const int32_t sr = direct_source(dir, next_src[u], ok);
      so[u] = sr >= 0 ? int64_t(sr) * shape.bytes : -1;
      dof[u] = int64_t(next_row[u]) * shape.bytes;
      const int64_t e = e0 + int64_t(blocks) * pass + u * groups;
      next_src[u] = e < n ? (srcrow ? srcrow[e] : int32_t(e)) : 0;
      next_row[u] = e < n ? (row ? row[e] : int32_t(e)) : 0;
    }
    // Addresses are carried from piece to piece: computed at the load they would share its registers and make it
    // wait for the entries requested above (38 -> 44 us on 400-byte rows).
    uint32_t at = chunk_at<VecT, RAGGED>(shape, sub);
    const Global* from[UNROLL];
    Global* to[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      from[u] = (const Global*)(src) + (so[u] + at);
      to[u] = (Global*)(dst) + (dof[u] + at);
    }
    for (uint32_t c0 = 0; c0 < shape.cpr; c0 += lanes) {
      const bool in_row = c0 + sub < shape.cpr;
      VecT val[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (so[u] >= 0 && in_row)
          val[u] = HBM_SOURCE ? *(const GlobalMem*)(from[u]) : __builtin_nontemporal_load((const GlobalMem*)(from[u]));
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (so[u] >= 0 && in_row) {
          if (HBM_SOURCE) __builtin_nontemporal_store(val[u], (GlobalMem*)(to[u]));
          else *(GlobalMem*)(to[u]) = val[u];
        }
      const uint32_t next = chunk_at<VecT, RAGGED>(shape, c0 + lanes + sub);
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        from[u] += next - at;
        to[u] += next - at;
      }
      at = next;
    }
  }
}

// ---- rows as flat runs of chunks ------------------------------------------------
// A wavefront takes 64 list entries and walks their rows as one flat run of chunks:
// all 64 lanes stay busy for any row width and UNROLL loads per lane are in flight
// before the first store.  Output rows are written once and not read again by this
// path, so they are stored non-temporally.
// The caller is workgroup `block` of `blocks` that share the entries.
template <typename VecT, bool RAGGED, int UNROLL, bool NT_LOAD>
__device__ __forceinline__ void flat_rows(const char* __restrict__ src, char* __restrict__ dst, const RowShape& shape,
                                          uint64_t inv_cpr, const int32_t* __restrict__ row,
                                          const int32_t* __restrict__ srcrow, int64_t n_max,
                                          const int32_t* __restrict__ n_dev, const DirectIds& dir, int epw, uint32_t block,
                                          uint32_t blocks) {
  typedef typename Chunk<VecT, RAGGED>::T Mem;
  int64_t n = n_dev ? int64_t(*n_dev) : n_max;
  int64_t lo = 0;
  if (dir.window) {                                 // entries [window[0], window[1]) only
    lo = dir.window[0] < 0 ? 0 : dir.window[0];
    n = dir.window[1];
  }
  if (n > n_max) n = n_max;
  if (block == 0) direct_stats(dir, n - lo);
  const int lane = threadIdx.x & 63;
  const int64_t wave = int64_t(block) * 4 + (threadIdx.x >> 6);
  const int64_t n_waves = int64_t(blocks) * 4;
  // epw (<= 64) list entries per wave and pass: fewer for wide rows, so that a pass moves a few tens of
  // KiB and the passes spread evenly over the waves whatever the (device-side) number of entries is
  for (int64_t e0 = lo + wave * epw; e0 < n; e0 += n_waves * epw) {
    const int64_t e = e0 + lane;
    const bool mine = lane < epw && e < n;
    const int32_t my_row = mine ? (row ? row[e] : int32_t(e)) : 0;
    const int32_t my_src = direct_source(dir, mine ? (srcrow ? srcrow[e] : int32_t(e)) : 0, mine);
    const uint32_t entries = uint32_t(n - e0 < epw ? n - e0 : epw);
    const uint32_t cpr = shape.cpr;
    const uint32_t total = entries * cpr;          // chunks in this wave's 64 rows
    for (uint32_t f0 = 0; f0 < total; f0 += 64 * UNROLL) {
      VecT val[UNROLL];
      int64_t doff[UNROLL];
      bool ok[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const uint32_t flat = f0 + u * 64 + lane;
        ok[u] = flat < total;
        const uint32_t k = ok[u] ? uint32_t((uint64_t(flat) * inv_cpr) >> 32) : 0u;   // flat / cpr
        const uint32_t col = flat - k * cpr;
        const int32_t r = __shfl(my_row, int(k), 64);
        const int32_t sr = __shfl(my_src, int(k), 64);
        ok[u] = ok[u] && sr >= 0;
        if (RAGGED) {
          const uint32_t at = chunk_at<VecT, true>(shape, col);
          doff[u] = int64_t(r) * shape.bytes + at;
          const Mem* from = reinterpret_cast<const Mem*>(src + (int64_t(sr) * shape.bytes + at));
          if (ok[u]) val[u] = NT_LOAD ? __builtin_nontemporal_load(from) : *from;
        } else {                                   // whole chunks: indexes, not bytes (1 % at 256-byte rows)
          doff[u] = int64_t(r) * cpr + col;
          const VecT* from = reinterpret_cast<const VecT*>(src);
          if (ok[u])
            val[u] = NT_LOAD ? __builtin_nontemporal_load(from + int64_t(sr) * cpr + col) : from[int64_t(sr) * cpr + col];
        }
      }
#pragma unroll
      for (int u = 0; u < UNROLL; ++u)
        if (ok[u])
          __builtin_nontemporal_store(val[u], RAGGED ? reinterpret_cast<Mem*>(dst + doff[u])
                                                     : reinterpret_cast<Mem*>(reinterpret_cast<VecT*>(dst) + doff[u]));
    }
  }
}

// ---- hits and misses in one launch --------------------------------------------
// The two lists of a partition (three for a clique member: list 2 is a second list of rows in HBM), or the caller's list of
// ids where all rows have the same source.  One after the other,
// the link idles while the hits are copied and HBM while the misses arrive; here the first miss_blocks workgroups
// take the misses and others the hits, beside them.  Calls, one after the other -> beside each other: 400-byte rows of
// 2.4 M vertices, 688 k ids, 30 / 70 / 95 / 99.5 % of the table cached 2925 -> 2844, 1208 -> 1100, 324 -> 231, 163 -> 148 us;
// 2-KiB rows, 95 % 654 -> 428 (356 k of 1.2 M); 7 k ids of 10 k vertices (512-byte rows, 20 %) 76 -> 65.
constexpr int kSplitHitUnroll = 2, kSplitMissUnroll = 4;
// Called by workgroup `block` of a.miss_blocks.
template <typename VecT, bool RAGGED>
__device__ __forceinline__ void split_misses(const SplitArgs& a, uint32_t block) {
  group_rows<VecT, RAGGED, kSplitMissUnroll, false>(a.miss_src, a.dst, a.miss_shape, a.lists.row[1], a.lists.src[1], a.n_max,
                                                    a.counters ? a.counters + 1 : nullptr, a.direct, a.miss_lanes, block,
                                                    a.miss_blocks);
}
// Called by workgroup `block` of `blocks`.
template <HitWalk W>
__device__ __forceinline__ void split_hits(const SplitArgs& a, uint32_t block, uint32_t blocks) {
  for (int l = 0; l <= (a.peers ? 2 : 0); l += 2) {
    const int32_t* const row = l ? a.lists.row[2] : a.lists.row[0];
    const int32_t* const src = l ? a.lists.src[2] : a.lists.src[0];
    const int32_t* const n = a.counters ? a.counters + l : nullptr;
    if constexpr (W == HitWalk::kGroups)
      group_rows<u32x4, true, kSplitHitUnroll, true>(a.hit_src, a.dst, a.hit_shape, row, src, a.n_max, n, a.direct, a.hit_lanes,
                                                     block, blocks);
    else
      flat_rows<u32x4, true, 4, W == HitWalk::kFlatLines>(a.hit_src, a.dst, a.hit_shape, a.hit_inv, row, src, a.n_max, n,
                                                          a.direct, a.hit_epw, block, blocks);
  }
}

}  // namespace
}  // namespace lgp
