// Graph constructor (Sec. 5, operator 4): turn the sampled results into one bipartite CSR
// block per hop in local numbering.  All hops go through two launches: index the lists + count
// the edges of every tile, then feature rows + offsets and relabelled sources.  (A launch costs
// 4-5 us; a workgroup of the second one adds up the tile counts before its own destinations
// instead of reading offsets that a launch between the two would write.)
//
// "Position of vertex u in a frontier": frontiers are ascending unique id lists, so each gets a
// bucket index -- where the ids of u >> s begin, with about one id per bucket -- and a lookup is
// one load of the bucket and, for the minority of buckets with several ids, a search in it.  Index
// and list together are a few MB, where a table with an entry per vertex made every write and
// lookup a random access to hundreds of MB (2.2 M accesses of a 111 M-vertex graph: 70 us per call,
// now 37; 630 k lookups of a 2.4 M-vertex graph 44 -> 37 us, four launches -> two).  A frontier
// that a caller has reordered is noticed while it is indexed, and its lookups take another path
// (position_any_order).  The
// extracted id list need not be ascending (the intra-batch pipeline lists in first-reach order),
// so "row of vertex v in the feature matrix" stays a table of V entries that is scattered with
// the positions and never cleared: only entries written for the current list are ever read.
//
// A launch is one row of workgroups cut into a range per list (Ranges): the lists' worst-case
// sizes differ by a factor of hundreds, and a grid wide enough for the longest in each row of a
// two-dimensional one dispatches 14 000 workgroups of which most find nothing to do.
#include "common.hpp"

#include <algorithm>

namespace lgp {
namespace {

__device__ __forceinline__ int64_t clamped(const int32_t* n_dev, int64_t cap) {
  const int64_t n = *n_dev;
  return n > cap ? cap : n;
}

constexpr int kMaxRanges = 2 * LGP_MAX_HOPS + 1;
struct Ranges {
  int32_t first[kMaxRanges + 1];   // range r = workgroups [first[r], first[r + 1])
  int32_t tile[LGP_MAX_HOPS];      // destinations a relabelling workgroup takes per pass, by hop
};
// Range of this workgroup, its index and the number of workgroups inside it.
__device__ __forceinline__ int find_range(const Ranges& rg, int n, int* index, int* count) {
  int r = 0;
  while (r + 1 < n && int(blockIdx.x) >= rg.first[r + 1]) ++r;
  *index = int(blockIdx.x) - rg.first[r];
  *count = rg.first[r + 1] - rg.first[r];
  return r;
}

__device__ __forceinline__ int64_t wave_inclusive_scan64(int64_t x) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int64_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  return x;
}

// Sum of one value per thread over a 256-thread workgroup (everyone gets the total) and the
// exclusive prefix of the calling thread.
__device__ __forceinline__ int64_t block_exclusive_scan64(int64_t x, int64_t* total) {
  __shared__ int64_t wave_sum[4];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int64_t inc = wave_inclusive_scan64(x);
  if (lane == 63) wave_sum[wave] = inc;
  __syncthreads();
  int64_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const int64_t sw = wave_sum[w];
    if (w < wave) before += sw;
    all += sw;
  }
  __syncthreads();
  *total = all;
  return before + inc - x;
}

// Bucket index of an ascending list of n ids: bucket b holds the ids with (id - first) >> shift == b and begins at
// start[b].  start[b] is set for every bucket that holds ids and for the one after it, which is where the bucket ends
// (the last one ends at n): the ids looked up are in the list, so the entries of other empty buckets are never read, and
// a list crowded into parts of the id range costs no more than one spread over it (100 k destinations x 10, 526 k ids
// in 2 % of 111 M: 265 us a call with every entry filled, 28 now; 561 k ids at the two ends 354, 33; spread over the
// range 38 either way).  Buckets split the span of the list, not the id range, so that a list in one corner has as few ids per bucket
// as any (2.75 M ids in 2 % of 250 M, 9.8 M x 5: 1490 us split by id range, 1075 by span).  There are at most V
// buckets, the size of a table.
struct Buckets {
  int32_t first, last, shift, count;
};
__device__ __forceinline__ Buckets bucket_shape(const int32_t* ids, int64_t num_vertices, int64_t n) {
  uint32_t end = n > 0 ? uint32_t(n - 1) : 0;
  asm("" : "+s"(end));                                         // a register of its own: a scalar load
  int32_t first = n > 0 ? ids[0] : 0, last = n > 0 ? ids[end] : 0;
  if (first < 0 || last < first || last >= num_vertices) {    // not ascending ids below V: any shape will do
    first = 0;
    last = int32_t(num_vertices - 1);
  }
  const uint32_t q = uint32_t(last - first) / uint32_t(n > 0 ? n : 1);
  // Half an id to one id per bucket on average; up to three vertices per id each vertex is a bucket of its own, and a
  // lookup needs no search (2 M destinations x 64 into 6.6 M of 20 M vertices: 1750 us with buckets of two, 1433 now,
  // a table with an entry per vertex 1460; 9.8 M x 5 into 2.75 M of a span of 5 M 1026, 873, 950).
  const int shift = q > 3 ? 31 - __clz(int(q)) : 0;
  return Buckets{first, last, shift, ((last - first) >> shift) + 1};
}

// Positions of N ids in the list, -1 for u < 0 (for an id that is not in the list: some value, from reads inside it).
// The searches run in step, so that the loads of all of them are in flight together.
template <int N>
__device__ __forceinline__ void positions(const int32_t* ids, int32_t n, const int32_t* start, const Buckets& b,
                                          const int32_t (&u)[N], int32_t (&lo)[N]) {
  int32_t hi[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const int32_t k = (u[q] - b.first) >> b.shift;
    const bool ok = u[q] >= b.first && k < b.count;
    lo[q] = ok ? start[k] : -1;
    hi[q] = ok && k + 1 < b.count ? start[k + 1] : n;
  }
#pragma unroll
  for (int q = 0; q < N; ++q) {
    hi[q] = uint32_t(hi[q]) < uint32_t(n) ? hi[q] : n;
    if (lo[q] < 0 || lo[q] > hi[q]) hi[q] = lo[q];            // nothing to search
  }
  for (;;) {
    int32_t at[N], mid[N];
    int more = 0;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      mid[q] = lo[q] + ((hi[q] - lo[q]) >> 1);               // == lo: nothing left to search
      more |= mid[q] ^ lo[q];
    }
    if (!__any(more)) break;
#pragma unroll
    for (int q = 0; q < N; ++q) at[q] = mid[q] != lo[q] ? ids[mid[q]] : u[q];
#pragma unroll
    for (int q = 0; q < N; ++q) {                             // closed searches keep lo: at == u, mid == lo
      const bool right = at[q] <= u[q];
      lo[q] = right ? mid[q] : lo[q];
      hi[q] = right ? hi[q] : mid[q];
    }
  }
}

// Position of one id per lane (-1 for u < 0 and for an id that is not in the list) in a list that is not ascending:
// the workgroup's ids go into a hash table in LDS and the whole list passes by once.  The work grows with workgroups
// times list, far beyond that of the bucket index, but a frontier comes out of the sampler ascending; only a caller
// who reorders it comes here.
constexpr int kJoinSlots = 512;                                // twice the ids of a workgroup: probing ends
struct JoinTable {
  int32_t id[kJoinSlots], at[kJoinSlots];
};
__device__ __forceinline__ uint32_t join_slot(int32_t u) { return (uint32_t(u) * 2654435761u) >> 23; }
__device__ __forceinline__ int32_t position_any_order(const int32_t* ids, int32_t n, JoinTable* t, int32_t u) {
  for (int k = threadIdx.x; k < kJoinSlots; k += 256) t->id[k] = t->at[k] = -1;
  __syncthreads();
  uint32_t mine = join_slot(u);
  while (u >= 0) {
    const int32_t old = atomicCAS(&t->id[mine], -1, u);
    if (old < 0 || old == u) break;
    mine = (mine + 1) % kJoinSlots;
  }
  __syncthreads();
  for (int32_t k = threadIdx.x; k < n; k += 256) {
    const int32_t v = ids[k];
    if (v < 0) continue;
    for (uint32_t s = join_slot(v); t->id[s] >= 0; s = (s + 1) % kJoinSlots)
      if (t->id[s] == v) {
        t->at[s] = k;
        break;
      }
  }
  __syncthreads();
  const int32_t pos = u >= 0 ? t->at[mine] : -1;
  __syncthreads();                                             // the table is reused by the next ids
  return pos;
}

// Range 0: positions inside the extracted id list go to table 0.  Range j = 1 .. n_hops: bucket index of frontier j, in
// table j.  Range n_hops + 1 + h: edge count of every tile of kScanTile destinations of hop h.
__global__ __launch_bounds__(256) void index_lists_kernel(BlocksArgs a, Ranges rg) {
  int index, count;
  const int r = find_range(rg, 2 * a.n_hops + 1, &index, &count);
  if (r == 0) {
    const int64_t n = clamped(a.n_gather, a.gather_cap);
    for (int64_t k = int64_t(index) * 256 + threadIdx.x; k < n; k += int64_t(count) * 256) {
      const int32_t v = a.gather_ids[k];
      if (uint32_t(v) < uint64_t(a.num_vertices)) a.table[v] = int32_t(k);
    }
    return;
  }
  if (r <= a.n_hops) {
    const int32_t* ids = a.frontier[r];
    const int64_t n = clamped(a.n_frontier + r, a.cap[r]);
    int32_t* start = a.table + int64_t(r) * a.num_vertices;
    const Buckets b = bucket_shape(ids, a.num_vertices, n);
    for (int64_t k = int64_t(index) * 256 + threadIdx.x; k < n; k += int64_t(count) * 256) {
      const int32_t v = ids[k], before = k > 0 ? ids[k - 1] : b.first - 1;
      if (v < b.first || v > b.last || before < b.first - (k == 0) || before >= v) {
        a.unordered[r] = a.call;                               // every writer stores the same value
        continue;
      }
      const int32_t mine = (v - b.first) >> b.shift, prev = k > 0 ? (before - b.first) >> b.shift : -1;
      if (mine != prev) {
        start[prev + 1] = int32_t(k);
        start[mine] = int32_t(k);
      }
    }
    return;
  }
  const int h = r - a.n_hops - 1;
  const int64_t n = clamped(a.n_frontier + h, a.cap[h]);
  const int32_t* cnt = a.cnt[h];
  for (int64_t tile = index; tile * kScanTile <= n; tile += count) {
    const int64_t base = tile * kScanTile + int64_t(threadIdx.x) * 4;
    int64_t mine = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (base + q < n) mine += cnt[base + q];
    int64_t total;
    block_exclusive_scan64(mine, &total);
    if (threadIdx.x == 0) a.tile_sums[a.tile_base[h] + tile] = total;
  }
}

// Range r < n_hops, hop h = n_hops - 1 - r (the longest first): blk_indptr[i] = cnt[0] + ... + cnt[i - 1] for i <= n
// (64-bit sums), and blk_src of hop h = positions of its samples in frontier h + 1, packed at those offsets.
// Range n_hops + k: feat_row of frontier j = n_hops - k, position of its vertex i in the extracted id list (table 0).
// A workgroup pass takes a power of two of destinations with at most kRelabelLoads samples per lane, all looked up
// at once: a hop of few destinations and a wide fan-out would otherwise be a handful of workgroups in a long chain.
constexpr int kRelabelLoads = 4;
inline int32_t relabel_tile(int32_t f) {
  int32_t tile = 256;
  while (tile * f > 256 * kRelabelLoads) tile /= 2;             // f <= 64: at least 16
  return tile;
}
__global__ __launch_bounds__(256, 8) void lookup_relabel_kernel(BlocksArgs a, Ranges rg) {
  __shared__ int64_t offset[256];
  __shared__ JoinTable join;
  int index, count;
  const int r = find_range(rg, 2 * a.n_hops + 1, &index, &count);
  if (r >= a.n_hops) {
    const int j = 2 * a.n_hops - r;
    const int32_t* ids = a.frontier[j];
    int32_t* out = a.feat_row[j];
    const int64_t n = clamped(a.n_frontier + j, a.cap[j]);
    for (int64_t i = int64_t(index) * 256 + threadIdx.x; i < n; i += int64_t(count) * 256) {
      const int32_t v = ids[i];
      out[i] = uint32_t(v) < uint64_t(a.num_vertices) ? a.table[v] : -1;   // an invalid seed has no row
    }
    return;
  }
  const int h = a.n_hops - 1 - r;
  const int32_t f = a.fanout[h];
  const uint32_t inv_f = (1u << 20) / uint32_t(f) + 1;       // exact division of t < 1024 by f <= 64
  const int32_t* cnt = a.cnt[h];
  const int32_t* next = a.frontier[h + 1];
  // The two frontier sizes lie side by side; as one access they become a vector load in front of everything else, and
  // apart they are scalar loads, hits for all workgroups but the first (kernel 25.0 -> 23.0 us at 111 M vertices).
  int j = h + 1;
  asm("" : "+s"(j));
  const int32_t n_next = int32_t(clamped(a.n_frontier + j, a.cap[j]));
  const int32_t* start = a.table + int64_t(h + 1) * a.num_vertices;
  const Buckets b = bucket_shape(next, a.num_vertices, n_next);
  const bool ascending = a.unordered[h + 1] != a.call;
  const int64_t* tile_sums = a.tile_sums + a.tile_base[h];
  int64_t* indptr = a.blk_indptr[h];
  int32_t* blk_src = a.blk_src[h];
  const uint32_t n = uint32_t(clamped(a.n_frontier + h, a.cap[h]));          // below 2^31: no sum overflows
  const uint32_t tile_dst = uint32_t(rg.tile[h]);
  // Edges of the whole tiles before this workgroup's destinations, this thread's share: the passes ascend, so each adds
  // the tiles since the one before (all of them again per pass: 1 M destinations x 5 267 us a call, 250 now, 9.8 M x 5
  // with 2.75 M sources 1089, 1026).
  int64_t whole = 0;
  uint32_t next_tile = threadIdx.x;
  for (uint32_t first = uint32_t(index) * tile_dst; first <= n; first += uint32_t(count) * tile_dst) {
    const uint32_t left = n - first;
    const int dst = int(left < tile_dst ? left : tile_dst), total = dst * f;
    const int32_t* nbr = a.nbr[h] + int64_t(first) * f;
    // the lookups are under way while the offsets they are written at are computed
    int32_t u[kRelabelLoads], pos[kRelabelLoads];
#pragma unroll
    for (int q = 0; q < kRelabelLoads; ++q) {
      const int t = int(threadIdx.x) + q * 256;
      u[q] = t < total ? nbr[t] : -1;
    }
    // edges before this workgroup's destinations: whole tiles, then the rest of the tile it lies in
    const uint32_t tile = first / kScanTile;
    for (; next_tile < tile; next_tile += 256) whole += tile_sums[next_tile];
    int64_t part = whole;
    for (uint32_t k = tile * kScanTile + threadIdx.x; k < first; k += 256) part += cnt[k];
    const uint32_t i = first + threadIdx.x;
    const int32_t c = int(threadIdx.x) < dst ? cnt[i] : 0;
    positions(next, n_next, start, b, u, pos);
    int64_t before, mine;
    block_exclusive_scan64(part, &before);
    const int64_t at = before + block_exclusive_scan64(c, &mine);
    if (threadIdx.x < tile_dst && i <= n) indptr[i] = at;    // entry n holds the edge total
    offset[threadIdx.x] = at;
    __syncthreads();
    if (!ascending)
      for (int q = 0; q < kRelabelLoads; ++q) pos[q] = position_any_order(next, n_next, &join, u[q]);
#pragma unroll
    for (int q = 0; q < kRelabelLoads; ++q) {
      const uint32_t t = threadIdx.x + q * 256;
      const uint32_t d = (t * inv_f) >> 20;
      if (u[q] >= 0) blk_src[offset[d] + (t - d * uint32_t(f))] = pos[q];   // padding fills the end of a row
    }
    __syncthreads();                                          // offset is reused by the next pass
  }
}

// Workgroups for `items` of which one workgroup pass takes `per`: at most eight per CU and list (4 / 8: 41.3 / 39.1 us
// at 111 M vertices, 35 / 36 us at 2.4 M).
inline int32_t groups_for(const DeviceInfo& di, int64_t items, int64_t per) {
  const int64_t most = int64_t(di.num_cus) * 8;
  return int32_t(std::min(most, (items + per - 1) / per));
}

}  // namespace

void launch_build_blocks(const DeviceInfo& di, const BlocksArgs& a, hipStream_t s) {
  const int L = a.n_hops;
  Ranges scatter = {}, lookup = {};
  for (int j = 0; j <= L; ++j)
    scatter.first[j + 1] = scatter.first[j] + groups_for(di, j == 0 ? a.gather_cap : a.cap[j], 256);
  for (int h = 0; h < L; ++h)        // one more tile than the destinations fill, so that indptr[n] is always written
    scatter.first[L + h + 2] = scatter.first[L + h + 1] + groups_for(di, a.cap[h] / kScanTile + 1, 1);
  for (int r = 0; r < L; ++r) {
    const int h = L - 1 - r;
    lookup.tile[h] = relabel_tile(a.fanout[h]);
    lookup.first[r + 1] = lookup.first[r] + groups_for(di, a.cap[h] / lookup.tile[h] + 1, 1);
  }
  for (int k = 0; k <= L; ++k) lookup.first[L + k + 1] = lookup.first[L + k] + groups_for(di, a.cap[L - k], 256);
  hipLaunchKernelGGL(index_lists_kernel, dim3(unsigned(scatter.first[2 * L + 1])), dim3(256), 0, s, a, scatter);
  hipLaunchKernelGGL(lookup_relabel_kernel, dim3(unsigned(lookup.first[2 * L + 1])), dim3(256), 0, s, a, lookup);
}

}  // namespace lgp
