// Graph constructor (Sec. 5, operator 4): turn the sampled results into one bipartite CSR
// block per hop in local numbering.  All hops go through two launches: index the lists + count
// the edges of every tile, then feature rows + offsets and relabelled sources.  (A launch costs
// 4-5 us; a workgroup of the second one adds up the tile counts before its own destinations
// instead of reading offsets that a launch between the two would write.)
//
// "Position of vertex u in a frontier": frontiers are ascending unique id lists, so each gets an
// index by blocks of vertices (see Entry): a lookup is one load of eight bytes, and for lists of few
// ids sometimes a search among the ids of a block.  Index and list together are a few MB, where a
// table with an entry per vertex made every write and lookup a random access to hundreds of MB.
// Calls, table -> where the ids of a bucket of vertices begin, two loads and a search a lookup -> now:
// 2.2 M accesses of a 111 M-vertex graph 70 -> 34.4 -> 34.4 us; 8192 seeds (15, 10, 5) of 2.4 M vertices
// 44 -> 41.5 -> 33.3; (25, 25) of 20 M 27.9 -> 27.0.  A frontier
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

// Index of an ascending list of n ids: block b holds the ids with (id - first) >> shift == b, and one eight-byte load says
// where they are.  Shift 5: a bit for each of the block's 32 vertices that is in the list and where its ids begin; the
// position of an id is that plus the bits below its own.  Wider blocks, of lists with fewer ids, hold one to two ids on
// average; an entry is four bytes, where its ids begin, the entry after it then says where they end, and a search finds the
// id.  With both in an entry of eight bytes the index outgrows the L2 cache earlier: calls with 0.55, 0.92, 1.2 and 1.6 M ids in
// 111 M vertices 33.8 / 54.5 / 73.0 / 96.3 us, now 31.7 / 49.9 / 66.9 / 89.5.  Half as many ids per block (twice the index) is slower up
// to about 1.5 M ids (the same four 33.5 / 52.4 / 68.6 / 89.0) and ahead beyond (250 M vertices, 2.1 M ids 132.4 / 129.7, 2.8 M
// 189.6 / 184.1).
// Only blocks that hold ids are set: the ids looked up are in the list, so the other entries are never read, and a list
// crowded into parts of the id range costs no more than one spread over it.  Blocks split the span of the list, not the
// id range, so that a list in one corner has as few ids per block as any (calls, two loads and a search -> now: 2 M
// destinations x 16 of 20 M vertices, 16 M sources 772 -> 390 us, 400 k sources in one corner 265 -> 181, at both ends 795 ->
// 181; 1 M x 5 of 111 M 339 -> 295, 85 -> 48, 243 -> 47; 100 k x 10, 1 M sources 55 -> 53, corner 33 -> 23, both ends 48 -> 48).
// A block has 32 vertices or more, so an index fits the table of one entry per vertex.
struct __attribute__((packed, aligned(4))) Entry {             // one load, also at an odd word
  uint32_t start, more;            // first position in the block; bits of its vertices, or the position after its last
};
struct Shape {
  int32_t first, last, shift;
};
constexpr int kBitsShift = 5;
constexpr uint32_t kBitsMaxGap = 64;      // vertices per id up to which a block is 32 vertices (calls are level at 16, 64, 128)
constexpr int64_t kManyIds = int64_t(1) << 21;   // from here on blocks that need a search hold half as many ids
__device__ __forceinline__ Shape index_shape(const int32_t* ids, int64_t num_vertices, int64_t n) {
  uint32_t end = n > 0 ? uint32_t(n - 1) : 0;
  asm("" : "+s"(end));                                         // a register of its own: a scalar load
  int32_t first = n > 0 ? ids[0] : 0, last = n > 0 ? ids[end] : 0;
  if (first < 0 || last < first || last >= num_vertices) {    // not ascending ids below V: any shape will do
    first = 0;
    last = int32_t(num_vertices - 1);
  }
  const uint32_t q = uint32_t(last - first) / uint32_t(n > 0 ? n : 1);
  return Shape{first, last, q < kBitsMaxGap ? kBitsShift : (n < kManyIds ? 32 : 31) - __clz(int(q))};
}

// Positions of N ids in the list, -1 for u < 0 (for an id that is not in the list: some value, from reads inside it).
// The searches run in step, so that the loads of all of them are in flight together.
template <int N>
__device__ __forceinline__ void positions(const int32_t* ids, int32_t n, const uint32_t* index, const Shape& sh,
                                          const int32_t (&u)[N], int32_t (&lo)[N]) {
  Entry e[N];
  const int entry_words = sh.shift == kBitsShift ? 1 : 0;     // as a power of two
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const bool ok = u[q] >= sh.first && u[q] <= sh.last;
    uint32_t at = ok ? uint32_t(u[q] - sh.first) >> sh.shift : 0;
    asm("" : "+v"(at));                                        // one load each, which no branch sets apart from the others
    e[q] = *reinterpret_cast<const Entry*>(index + (size_t(at) << entry_words));
    lo[q] = ok ? int32_t(e[q].start) : -1;
  }
  if (sh.shift == kBitsShift) {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int before = __popc(e[q].more & ((1u << (uint32_t(u[q] - sh.first) & 31u)) - 1u));
      if (lo[q] >= 0) lo[q] += before;
    }
    return;
  }
  int32_t hi[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    hi[q] = e[q].more < uint32_t(n) ? int32_t(e[q].more) : n;
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
    for (int q = 0; q < N; ++q) {
      uint32_t k = mid[q] != lo[q] ? mid[q] : 0;
      asm("" : "+v"(k));
      at[q] = ids[k];
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {                             // closed searches keep lo, which is mid
      const bool right = mid[q] == lo[q] || at[q] <= u[q];
      lo[q] = right ? mid[q] : lo[q];
      hi[q] = right ? hi[q] : mid[q];
    }
  }
}

__device__ __forceinline__ uint32_t wave_inclusive_scan32(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}

// Entries of the blocks whose first id is among the 64 ids from `base` on (one wave; base < n, a multiple of 64).
// Returns false in a lane that found its id out of order.
__device__ __forceinline__ bool index_ids(const int32_t* ids, int64_t n, const Shape& sh, int64_t base, uint32_t* index) {
  const int lane = threadIdx.x & 63;
  const int64_t k = base + lane;
  const bool in = k < n;
  const int32_t v = in ? ids[k] : 0;
  const int32_t before = in && k > 0 ? ids[k - 1] : -1;
  const bool valid = v >= sh.first && v <= sh.last, valid_before = before >= sh.first && before <= sh.last;
  const uint32_t o = uint32_t(v - sh.first), block = o >> sh.shift;
  const uint32_t block_before = uint32_t(before - sh.first) >> sh.shift;
  const bool leads = in && (k == 0 || block_before != block);
  const bool ordered = !in || (valid && (k == 0 || (valid_before && before < v)));
  if (sh.shift != kBitsShift) {
    if (leads && valid) {
      index[block] = uint32_t(k);
      if (k > 0 && valid_before) index[block_before + 1] = uint32_t(k);
    }
    if (k + 1 == n && valid) index[block + 1] = uint32_t(n);
    return ordered;
  }
  // The bits of a block are those of a run of lanes, and of the ids behind the wave where the last run goes on: a block has
  // at most 32 ids.  Ids differ, so the OR of their bits is their sum.
  const bool behind = lane < 32 && base + 64 + lane < n;
  const int32_t w = behind ? ids[base + 64 + lane] : 0;
  const uint32_t bit = in ? 1u << (o & 31u) : 0u;
  const uint32_t sum = wave_inclusive_scan32(bit);
  const uint64_t lead = __ballot(leads);
  const uint32_t last_block = uint32_t(__builtin_amdgcn_readlane(int(block), 63));
  const uint32_t o_w = uint32_t(w - sh.first);
  const bool goes_on = behind && o_w >> sh.shift == last_block;
  uint32_t sum_behind = 0;
  if (__any(goes_on))
    sum_behind = uint32_t(__builtin_amdgcn_readlane(int(wave_inclusive_scan32(goes_on ? 1u << (o_w & 31u) : 0u)), 63));
  const uint64_t mine = lead & (~0ull >> (63 - lane));         // the last of them is the first lane of this lane's run
  const int leader = mine ? 63 - __clzll((long long)mine) : 0;
  const uint32_t sum_before = uint32_t(__shfl(int(sum - bit), leader, 64));
  const bool ends = in && (lane == 63 || k + 1 == n || ((lead >> (lane + 1)) & 1ull));
  if (ends && mine && valid)
    *reinterpret_cast<Entry*>(index + 2 * size_t(block)) =
        Entry{uint32_t(base + leader), sum - sum_before + (lane == 63 ? sum_behind : 0u)};
  return ordered;
}

// Position of one id per lane (-1 for u < 0 and for an id that is not in the list) in a list that is not ascending:
// the workgroup's ids go into a hash table in LDS and the whole list passes by once.  The work grows with workgroups
// times list, far beyond that of the index, but a frontier comes out of the sampler ascending; only a caller
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

// Ids of the extracted list that a thread has in flight, and that a workgroup takes per pass.
constexpr int kScatterLoads = 4, kScatterTile = 256 * kScatterLoads;

// Range 0: positions inside the extracted id list go to table 0.  Range j = 1 .. n_hops: index of frontier j, in
// table j.  Range n_hops + 1 + h: edge count of every tile of kScanTile destinations of hop h.
__global__ __launch_bounds__(256) void index_lists_kernel(BlocksArgs a, Ranges rg) {
  int index, count;
  const int r = find_range(rg, 2 * a.n_hops + 1, &index, &count);
  if (r == 0) {
    const int64_t n = clamped(a.n_gather, a.gather_cap);
    for (int64_t k = int64_t(index) * kScatterTile + threadIdx.x; k < n; k += int64_t(count) * kScatterTile) {
      int32_t v[kScatterLoads];
#pragma unroll
      for (int q = 0; q < kScatterLoads; ++q) v[q] = k + q * 256 < n ? a.gather_ids[k + q * 256] : -1;
#pragma unroll
      for (int q = 0; q < kScatterLoads; ++q)
        if (uint32_t(v[q]) < uint64_t(a.num_vertices)) a.table[v[q]] = int32_t(k + q * 256);
    }
    return;
  }
  if (r <= a.n_hops) {
    const int32_t* ids = a.frontier[r];
    const int64_t n = clamped(a.n_frontier + r, a.cap[r]);
    uint32_t* entries = reinterpret_cast<uint32_t*>(a.table + int64_t(r) * a.table_stride);
    const Shape sh = index_shape(ids, a.num_vertices, n);
    for (int64_t k = int64_t(index) * 256 + (threadIdx.x & 192); k < n; k += int64_t(count) * 256)
      if (!index_ids(ids, n, sh, k, entries)) a.unordered[r] = a.call;      // every writer stores the same value
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
  const uint32_t* entries = reinterpret_cast<const uint32_t*>(a.table + int64_t(h + 1) * a.table_stride);
  const Shape sh = index_shape(next, a.num_vertices, n_next);
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
    positions(next, n_next, entries, sh, u, pos);
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

// Workgroups for `items` of which one workgroup pass takes `per`: at most `per_cu` per CU and list.  The lists' sizes are only
// known on the device, so most workgroups of a grid for the worst case find nothing to do, and 8000 of them take longer to
// start than the indexing takes: 8 / 4 / 3 / 2 per CU and list 33.1 / 30.4 / 30.2 / 30.3 us a call at 2.4 M vertices, 34.7 / 33.2
// / 33.1 / 33.1 at 111 M, 26.9 / 27.0 / 27.0 / 27.1 with 20 M.  The lookups wait for a chain of loads in each pass and need the
// wider grid: 8 / 4 per CU in both launches 27.6 / 30.1 at 20 M, 36.1 / 35.4 at 111 M, 33.9 / 29.0 at 2.4 M; one grid of eight
// workgroups per CU that shares out the tiles of all lists 28.2, 35.0 and 31.5.
inline int32_t groups_for(const DeviceInfo& di, int64_t items, int64_t per, int64_t per_cu) {
  return int32_t(std::min(int64_t(di.num_cus) * per_cu, (items + per - 1) / per));
}
constexpr int kIndexGroups = 4, kLookupGroups = 8;

}  // namespace

void launch_build_blocks(const DeviceInfo& di, const BlocksArgs& a, hipStream_t s) {
  const int L = a.n_hops;
  Ranges scatter = {}, lookup = {};
  for (int j = 0; j <= L; ++j)
    scatter.first[j + 1] = scatter.first[j] + groups_for(di, j == 0 ? a.gather_cap : a.cap[j], j == 0 ? kScatterTile : 256, kIndexGroups);
  for (int h = 0; h < L; ++h)        // one more tile than the destinations fill, so that indptr[n] is always written
    scatter.first[L + h + 2] = scatter.first[L + h + 1] + groups_for(di, a.cap[h] / kScanTile + 1, 1, kIndexGroups);
  for (int r = 0; r < L; ++r) {
    const int h = L - 1 - r;
    lookup.tile[h] = relabel_tile(a.fanout[h]);
    lookup.first[r + 1] = lookup.first[r] + groups_for(di, a.cap[h] / lookup.tile[h] + 1, 1, kLookupGroups);
  }
  for (int k = 0; k <= L; ++k) lookup.first[L + k + 1] = lookup.first[L + k] + groups_for(di, a.cap[L - k], 256, kLookupGroups);
  hipLaunchKernelGGL(index_lists_kernel, dim3(unsigned(scatter.first[2 * L + 1])), dim3(256), 0, s, a, scatter);
  hipLaunchKernelGGL(lookup_relabel_kernel, dim3(unsigned(lookup.first[2 * L + 1])), dim3(256), 0, s, a, lookup);
}

}  // namespace lgp
