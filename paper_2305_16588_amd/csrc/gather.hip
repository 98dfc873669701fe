// Feature extractor (Sec. 2.2 step 3; Sec. 5 "feature extractor") for gfx950:
// cache lookup + hit/miss partition, then one row-gather launch for both -- hits move
// HBM -> HBM, misses are read in place from CPU memory over PCIe beside them (gather_split_kernel),
// or two launches where they are timed apart or run on two streams.
//
// Two row-gather kernels share the work of calls with one kind of row.  The group kernel further down gives every row a
// group of lanes: it serves the misses, the cache fill and the hits on rows that straddle
// 128-byte lines.  The flat kernel serves hits on rows made of whole lines:
// a wavefront takes 64 list entries (one coalesced load of the row / source
// indices), then walks the 64 rows as one flat run of 16-byte chunks, so every lane
// issues 128-bit loads and stores, a row of any 16-byte-multiple width keeps all lanes
// busy, and several loads per lane are in flight before the first store.  The
// (row, source) pair a chunk belongs to is fetched from the owning lane by a
// cross-lane read, the LDS-crossbar path (ds_bpermute) -- the rows themselves never
// need to sit in LDS because a chunk is loaded and stored by the same lane.
#include "gather_dev.hpp"

#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

namespace lgp {
namespace {

__global__ void zero_counters_kernel(int32_t* counters, int n) {
  if (int(threadIdx.x) < n) counters[threadIdx.x] = 0;
}

// Each wave looks up kPartItems x 64 consecutive ids; the workgroup reserves its share of every
// list with ONE atomic per list (the global counters are the only contended words), then
// every lane writes its entries at wave-ballot ranks, so the lists stay in ascending row
// order inside a workgroup.  List 0 = hits, list 1 = misses; with NL = 3 a hit whose slot lies
// outside [local_lo, local_hi) -- another clique member's region of the cache -- goes to list 2.
// ALONE: one workgroup takes all ids, so the counters are written, not added to, and need no launch that clears them
// first.
constexpr int kPartItems = 4;
constexpr int kAloneThreads = 1024, kAloneItems = 4;
template <int NL, int THREADS, int ITEMS, bool ALONE>
__global__ __launch_bounds__(THREADS) void partition_kernel(
    const int32_t* __restrict__ ids, int64_t n_max, const int32_t* __restrict__ n_dev,
    const int32_t* __restrict__ f_remap, int64_t num_vertices, PartLists out, int32_t local_lo, int32_t local_hi,
    int32_t* __restrict__ counters, uint32_t* __restrict__ d_err, const int32_t* __restrict__ window) {
  constexpr int kWaves = THREADS / 64;
  __shared__ int wave_cnt[NL][kWaves], block_base[NL];
  int64_t n = n_dev ? int64_t(*n_dev) : n_max;
  int64_t lo = 0;
  if (window) {                                     // entries [window[0], window[1]) of ids
    lo = window[0] < 0 ? 0 : window[0];
    n = window[1];
  }
  if (n > n_max) n = n_max;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t lower = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  constexpr int kTile = THREADS * ITEMS;
  int listed = 0;                                  // ALONE, thread l: entries of list l so far
  for (int64_t base = lo + int64_t(blockIdx.x) * kTile; base < n; base += int64_t(gridDim.x) * kTile) {
    int32_t src[ITEMS], slot[ITEMS];
    uint64_t mask[NL][ITEMS];
    int cnt[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) cnt[l] = 0;
    // all ids are on their way before the first lookup, and all lookups before the first is used
    const int64_t mine = base + wave * (64 * ITEMS) + lane;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) src[j] = mine + j * 64 < n ? ids[mine + j * 64] : 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) slot[j] = uint32_t(src[j]) < uint64_t(num_vertices) ? f_remap[src[j]] : -1;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const bool active = mine + j * 64 < n;
      const bool ok = active && uint32_t(src[j]) < uint64_t(num_vertices);
      if (active && !ok) atomicOr(d_err, ERR_BAD_ID);
      int which = -1;                               // list of this entry
      if (ok) which = slot[j] < 0 ? 1 : (NL == 3 && (slot[j] < local_lo || slot[j] >= local_hi)) ? 2 : 0;
      if (which != 1) src[j] = slot[j];
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        mask[l][j] = __ballot(which == l);
        cnt[l] += __popcll(mask[l][j]);
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int l = 0; l < NL; ++l) wave_cnt[l][wave] = cnt[l];
    }
    __syncthreads();
    if (threadIdx.x < NL) {
      const int l = threadIdx.x;
      int t = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) t += wave_cnt[l][w];
      block_base[l] = ALONE ? listed : t ? atomicAdd(&counters[l], t) : 0;
      listed += t;
    }
    __syncthreads();
    int pos[NL];
#pragma unroll
    for (int l = 0; l < NL; ++l) {
      pos[l] = block_base[l];
      for (int w = 0; w < wave; ++w) pos[l] += wave_cnt[l][w];
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const int64_t i = base + wave * (64 * ITEMS) + j * 64 + lane;
      const uint64_t bit = 1ull << lane;
#pragma unroll
      for (int l = 0; l < NL; ++l) {
        if (mask[l][j] & bit) {
          const int at = pos[l] + __popcll(mask[l][j] & lower);
          out.row[l][at] = int32_t(i);
          out.src[l][at] = src[j];
        }
        pos[l] += __popcll(mask[l][j]);
      }
    }
    __syncthreads();                               // LDS is reused by the next tile
  }
  if (ALONE && threadIdx.x < NL) counters[threadIdx.x] = listed;
}

// ---- cache hits: HBM -> HBM ------------------------------------------------
// Rows as flat runs of chunks (see flat_rows).
template <typename VecT, bool RAGGED, int UNROLL, bool NT_LOAD>
__global__ __launch_bounds__(256) void gather_rows_flat_kernel(const char* __restrict__ src, char* __restrict__ dst,
                                                               RowShape shape, uint64_t inv_cpr,
                                                               const int32_t* __restrict__ row,
                                                               const int32_t* __restrict__ srcrow, int64_t n_max,
                                                               const int32_t* __restrict__ n_dev, DirectIds dir,
                                                               int epw) {
  flat_rows<VecT, RAGGED, UNROLL, NT_LOAD>(src, dst, shape, inv_cpr, row, srcrow, n_max, n_dev, dir, epw, blockIdx.x, gridDim.x);
}

// ---- cache misses and cache fill: CPU memory -> HBM over PCIe ---------------
// One lane group per row (see group_rows).  A call of more than `most` rows is left to the first `narrow` workgroups.
template <typename VecT, bool RAGGED, int G, int UNROLL, bool HBM_SOURCE>
__global__ __launch_bounds__(256) void gather_rows_group_kernel(const char* __restrict__ src, char* __restrict__ dst,
                                                                RowShape shape, const int32_t* __restrict__ row,
                                                                const int32_t* __restrict__ srcrow, int64_t n_max,
                                                                const int32_t* __restrict__ n_dev, DirectIds dir,
                                                                int64_t most, uint32_t narrow) {
  uint32_t blocks = gridDim.x;
  if (blocks > narrow) {
    const int64_t n = dir.window ? int64_t(dir.window[1]) - dir.window[0] : n_dev ? int64_t(*n_dev) : n_max;
    if (n > most) blocks = narrow;
    if (blockIdx.x >= blocks) return;
  }
  group_rows<VecT, RAGGED, UNROLL, HBM_SOURCE>(src, dst, shape, row, srcrow, n_max, n_dev, dir, G, blockIdx.x, blocks);
}

// Hits by lane groups, but rows of 2 KiB and more by the flat walk, as in a launch of their own; with six workgroups per CU
// while the link is the last to finish, and with two where there are 200 hits and more to a miss.  Lane groups / flat with two / with six, at 95, 99, 99.5 and 99.99 % cached: 257 k rows of 1792 bytes 350 / 380 / 330,
// 200 / 218 / 204, 193 / 204 / 200, 178 / 191 / 195 us a call, of 2048 396 / 434 / 379, 231 / 233 / 222, 225 / 214 / 215, 209 / 198 / 205, of 4096
// 778 / 849 / 752, 451 / 450 / 431, 437 / 414 / 415, 405 / 390 / 407; 278 k of 3080 718 / 785 / 689, 450 / 449 / 434, 439 / 419 / 422,
// 417 / 373 / 405 (one launch after the other 954, 495, 438, 388).  Beside a hop (launch_hop_and_rows) lane groups are ahead or
// level: all rows cached and 4096 seeds of 400 k vertices, 2048 bytes 125 / 152 / 147, 4096 211 / 236 / 227.
constexpr int64_t kFlatHitBytes = 2048, kNarrowHitsPerMiss = 200;
template <typename VecT, bool RAGGED, HitWalk W>
__global__ __launch_bounds__(256) void gather_split_kernel(SplitArgs a) {
  if (blockIdx.x < a.miss_blocks) split_misses<VecT, RAGGED>(a, blockIdx.x);
  else {
    const uint32_t block = blockIdx.x - a.miss_blocks;
    uint32_t blocks = a.hit_blocks;
    if (W != HitWalk::kGroups && blocks > a.hit_narrow) {
      const int64_t hits = int64_t(a.counters[0]) + (a.peers ? a.counters[2] : 0);
      if (int64_t(a.counters[1]) * kNarrowHitsPerMiss <= hits) blocks = a.hit_narrow;
    }
    if (block < blocks) split_hits<W>(a, block, blocks);
  }
}

inline unsigned blocks_for(int64_t work_blocks, int64_t limit) {
  int64_t b = work_blocks < limit ? work_blocks : limit;
  return unsigned(b < 1 ? 1 : b);
}

// Where a gather kernel is launched: on stream s, and -- when a and b are given -- with its own start
// and stop times recorded into those two events (hipExtLaunchKernelGGL), which costs no extra packets
// on the stream, unlike a pair of hipEventRecord calls around the launch.
struct Where {
  hipStream_t s;
  hipEvent_t a, b;
  int64_t hbm_blocks;   // most workgroups an HBM-bound gather may use
  int64_t items;        // entries to size the grid for (<= n_max: a window covers part of the array)
};

template <typename K, typename... Args>
void launch_on(const Where& w, K kernel, unsigned blocks, Args... args) {
  if (w.a && w.b) hipExtLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, w.s, w.a, w.b, 0, args...);
  else hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256), 0, w.s, args...);
}

inline uint64_t inverse(uint32_t cpr) { return (uint64_t(1) << 32) / cpr + 1; }   // exact for flat < 64 * cpr, cpr <= 4096
inline int entries_per_wave(const RowShape& r, bool wide) {
  int epw = 64;
  while (epw > 4 && int64_t(epw) * r.bytes > (wide ? 8192 : 32768)) epw >>= 1;
  return epw;
}

constexpr uint32_t kWideChunks = 160;   // ragged cached rows of more chunks go through the flat kernel (see by_lane_group)

template <typename VecT, bool RAGGED>
void launch_flat(const DeviceInfo& di, const char* src, char* dst, const RowShape& shape, const int32_t* row,
                 const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, const DirectIds& dir, const Where& s) {
  const int64_t row_bytes = shape.bytes;
  const uint64_t inv = inverse(shape.cpr);
  // Three workgroups (12 waves) per CU: the flat walk keeps 4 x 16 bytes per lane in flight, and more
  // waves than that only add concurrent streams for the memory system to interleave -- measured hit
  // gather at 8 / 4 / 3 / 2 workgroups per CU: 51.3 / 48.9 / 48.3 / 49.0 us on 505 k 256-byte rows,
  // 163.1 / 157.4 / 155.3 / 156.5 us on 855 k 512-byte rows, 335.7 / 315.3 / 310.4 / 307.2 us on 379 k
  // 2-KiB rows.  A narrower gather also leaves room for a sampler running beside it on another stream.
  // A wave takes at most 32 KiB of rows per pass (64 rows of up to 512 bytes, 16 rows of 2 KiB): the number
  // of entries is only known on the device, and with 128 KiB passes a launch of 233 k 2-KiB rows left most
  // waves with one pass and a few with two (216.6 -> 195.7 us; 379 k such rows: 311.5 -> 263.8 us).
  // Wide ragged rows: two workgroups and 8-KiB passes, so that a wave's rows end sooner and the line two rows share is
  // still in L2 when its other part arrives (3080 bytes, 187 k rows: 248 -> 225 us, 4100 bytes, 175 k: 295 -> 281; but
  // 264 bytes, 584 k rows: 61 -> 68).
  const bool wide = RAGGED && shape.cpr > kWideChunks;
  const int epw = entries_per_wave(shape, wide);
  const unsigned blocks = blocks_for((s.items + 4 * epw - 1) / (4 * epw),
                                     std::min<int64_t>(s.hbm_blocks, int64_t(di.num_cus) * (wide ? 2 : 3)));
  // Rows made of whole 128-byte lines are read once: stream them past L2 (+2.5 % at 512-B and 2-KiB
  // rows).  Rows that straddle lines share their boundary lines between consecutive load
  // instructions, and L2 has to merge those (non-temporal loads cost 7 % on 400-B rows).
  if (row_bytes % 128 == 0)
    launch_on(s, gather_rows_flat_kernel<VecT, RAGGED, 4, true>, blocks, src, dst, shape, inv, row, srcrow, n_max, n_dev, dir, epw);
  else
    launch_on(s, gather_rows_flat_kernel<VecT, RAGGED, 4, false>, blocks, src, dst, shape, inv, row, srcrow, n_max, n_dev, dir, epw);
}

template <typename VecT, bool RAGGED, int G>
void launch_group_g(const DeviceInfo& di, const char* src, char* dst, const RowShape& shape, const int32_t* row,
                    const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, const DirectIds& dir, const Where& s) {
  constexpr int U = 4;
  // PCIe needs far fewer waves than HBM to stay saturated (bandwidth x latency is ~150 KB): one
  // workgroup per four CUs holds ~1 MB of reads in flight, and measured rates FALL with wider grids
  // (400-B rows 44.9 -> 44.0 GB/s, 2-KiB rows 57.5 -> 55.7 GB/s from 64 to 512 workgroups), because the
  // excess requests only queue up in front of the link.
  const unsigned blocks = blocks_for((s.items + (256 / G) * U - 1) / ((256 / G) * U), std::max(1, di.num_cus / 4));
  launch_on(s, gather_rows_group_kernel<VecT, RAGGED, G, U, false>, blocks, src, dst, shape, row, srcrow, n_max, n_dev, dir,
            n_max, blocks);
}

// Cache hits whose rows straddle 128-byte lines (e.g. 400-byte rows): one lane group per row, one
// row per group in flight.  Every line of a row is then requested by a single load instruction,
// which beats the flat walk by ~5 % on such rows; rows made of whole lines stay with the flat kernel.
template <typename VecT, bool RAGGED, int G>
void launch_group_hbm_g(const DeviceInfo& di, const char* src, char* dst, const RowShape& shape, const int32_t* row,
                        const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, const DirectIds& dir,
                        const Where& s) {
  // One row per group in flight needs more waves than the flat walk: 8 workgroups per CU (2 / 3 / 4 / 6 / 8: 512 k rows of 400
  // bytes 138.7 / 107.6 / 95.6 / 90.7 / 91.4 us), but 6 for a call whose rows leave little of the 256-MB last-level cache,
  // unless so many lanes of a group have no chunk that 8 workgroups keep no more requests in flight than 6 full ones.
  // 6 / 8 with 300 k, 500 k, 1 M and 2 M rows of 20 M vertices: 250 bytes 31.2 / 29.7, 52.3 / 49.4, 109 / 114, 221 / 246, 352 bytes 40.1 / 38.5,
  // 77.0 / 71.8, 140 / 144, 278 / 292, 400 bytes of 2.4 M 42.9 / 42.5, 80.6 / 72.0, 152 / 155, 280 / 312, 700 bytes 81.3 / 78.1, 141 / 151, 280 /
  // 306, 562 / 617; with few busy lanes 66 bytes 14.2 / 13.2, 21.9 / 20.4, 43.1 / 40.3, 85.8 / 82.1, 150 bytes 24.9 / 23.0, 40.3 / 37.0, 79.1 /
  // 71.2, 164 / 154, 520 bytes 66.9 / 67.0, 116 / 104, 234 / 214, 464 / 425.  Two rows in flight are level or slower below 150 bytes
  // and on rows of multiples of 4.
  const bool few = G <= 16 ? shape.cpr * 8 <= G * 5 : shape.cpr * 16 <= G * 9;
  const int64_t most = few ? n_max : (int64_t(224) << 20) / shape.bytes;
  const unsigned blocks = blocks_for((s.items + 256 / G - 1) / (256 / G), std::min<int64_t>(s.hbm_blocks, int64_t(di.num_cus) * 8));
  launch_on(s, gather_rows_group_kernel<VecT, RAGGED, G, 1, true>, blocks, src, dst, shape, row, srcrow, n_max, n_dev, dir, most,
            uint32_t(di.num_cus) * 6);
}

template <typename VecT, bool RAGGED>
void launch_group_hbm(const DeviceInfo& di, const char* src, char* dst, const RowShape& shape, const int32_t* row,
                      const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, const DirectIds& dir, const Where& s) {
  if (shape.cpr <= 4) launch_group_hbm_g<VecT, RAGGED, 4>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if (shape.cpr <= 8) launch_group_hbm_g<VecT, RAGGED, 8>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if (shape.cpr <= 16) launch_group_hbm_g<VecT, RAGGED, 16>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if (!RAGGED || shape.cpr <= 32) launch_group_hbm_g<VecT, RAGGED, 32>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if constexpr (RAGGED) launch_group_hbm_g<VecT, RAGGED, 64>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
}

// Which cached rows take the group kernel; the others, and all rows of whole lines, take the flat one.
// Aligned chunks: rows of up to 32.  Ragged rows end inside a line and inside a chunk; where the flat walk cuts a line
// between two store instructions, both parts can reach memory (872 bytes, 465 k rows: 408 MiB written for 387), and
// one lane group per row avoids it -- 488 k rows of 872 bytes flat / group 188 / 163 us, 1352 bytes (220 k) 120 / 111,
// 2056 (204 k) 197 / 177, 2312 (199 k) 199 / 184, 2568 (161 chunks, 195 k) 212 / 199; but from there the narrow flat walk
// is ahead (2568 bytes 189, 3080 bytes 225 against 241), while on 91 k rows of 2312 bytes it is behind (76 against 71).
// With 17 to 21 chunks a group of 32 leaves too many lanes idle: 264 bytes (584 k rows) flat / group 61 / 74 us, 328
// bytes 72 / 81, 344 (22 chunks) 81-85 / 82, 376 (24) 79 / 79, 408 (26) 88 / 79, 456 (29) 100 / 83.
// In aligned chunks of 8 bytes these rows took 68 (264 bytes), 77 (328), 99 (456), 168 (872), 117 (1352), 203 (2056)
// and 201 us (2568).
template <bool RAGGED>
bool by_lane_group(const RowShape& r) {
  if (r.bytes % 128 == 0) return false;
  if (!RAGGED) return r.cpr <= 32;
  return r.cpr <= 16 || (r.cpr > 21 && r.cpr <= kWideChunks);
}

template <typename VecT, bool RAGGED>
void launch_group(const DeviceInfo& di, const char* src, char* dst, const RowShape& shape, const int32_t* row,
                  const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, const DirectIds& dir, const Where& s) {
  if (shape.cpr <= 4) launch_group_g<VecT, RAGGED, 4>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if (shape.cpr <= 8) launch_group_g<VecT, RAGGED, 8>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if (shape.cpr <= 16) launch_group_g<VecT, RAGGED, 16>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else if (shape.cpr <= 32) launch_group_g<VecT, RAGGED, 32>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
  else launch_group_g<VecT, RAGGED, 64>(di, src, dst, shape, row, srcrow, n_max, n_dev, dir, s);
}

// The widest chunk that fits the row; RAGGED (see Chunk) where rows or addresses are no multiple of it.  Over PCIe
// a chunk that straddles two lines requests one of them a second time, so there a row that divides into at most
// 32 aligned chunks of 4 or 8 bytes -- one load instruction of a 32-lane group -- keeps them (200-byte rows: 240 us
// ragged, 233 aligned; 100-byte rows 181 / 179; but 50-byte rows of 2-byte chunks 150 ragged, 154 aligned, and
// rows of more chunks 302 / 329 at 300 bytes, 509 / 1060 at 602).  align: addresses and row width, OR-ed.
int64_t chunk_width(uintptr_t align, int64_t row_bytes, bool streaming) {
  const int64_t whole = (align & 15) == 0 ? 16 : (align & 7) == 0 ? 8 : (align & 3) == 0 ? 4 : 2;
  if (streaming && whole >= 4 && row_bytes / whole <= 32) return whole;
  return row_bytes >= 16 ? 16 : row_bytes >= 8 ? 8 : row_bytes >= 4 ? 4 : 2;
}
RowShape row_shape(int64_t row_bytes, int64_t width) {
  return RowShape{uint32_t((row_bytes + width - 1) / width), uint32_t(row_bytes), uint32_t(row_bytes - width)};
}
// Lanes of the group that owns a row: the power of two that covers its chunks, 4 to 64.
uint32_t group_lanes(const RowShape& r) {
  uint32_t g = 4;
  while (g < r.cpr && g < 64) g *= 2;
  return g;
}

}  // namespace

void launch_partition(const DeviceInfo& di, const int32_t* ids, int64_t n_max, const int32_t* n_dev,
                      const int32_t* f_remap, int64_t num_vertices, const PartLists& out, int n_lists,
                      int32_t local_lo, int32_t local_hi, int32_t* counters, uint32_t* d_err, hipStream_t s,
                      const int32_t* window, int64_t grid_items, bool zeroed) {
  const bool three = n_lists == 3;
  const int64_t items = (window && grid_items > 0 && grid_items < n_max) ? grid_items : n_max;
  auto launch = [&](auto two_lists, auto three_lists, int64_t blocks, int threads) {
    hipLaunchKernelGGL(three ? three_lists : two_lists, dim3(unsigned(blocks)), dim3(unsigned(threads)), 0, s, ids, n_max,
                       n_dev, f_remap, num_vertices, out, three ? local_lo : 0, three ? local_hi : 0, counters, d_err,
                       window);
  };
  // One workgroup for up to 4096 ids: a launch less (calls on 500 to 4096 ids 14.4 -> 11.2 us).  Beyond that its lookups
  // take longer than the launch: 10 k ids of 2 M vertices 20.9 us with one workgroup of ten ids per thread, 14.3 with many.
  if (items <= kAloneThreads * kAloneItems) {
    launch(&partition_kernel<2, kAloneThreads, kAloneItems, true>, &partition_kernel<3, kAloneThreads, kAloneItems, true>, 1,
           kAloneThreads);
    return;
  }
  if (!zeroed) hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, s, counters, three ? 3 : 2);
  int64_t blocks = (items + 256 * kPartItems - 1) / (256 * kPartItems);
  const int64_t full = int64_t(di.num_cus) * 8;
  if (blocks > full) blocks = full;
  launch(&partition_kernel<2, 256, kPartItems, false>, &partition_kernel<3, 256, kPartItems, false>, blocks, 256);
}

void launch_gather_rows(const DeviceInfo& di, const void* src, void* dst, int64_t row_bytes, const int32_t* row,
                        const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, bool streaming, hipStream_t stream,
                        const DirectIds& dir, hipEvent_t ev_start, hipEvent_t ev_stop, bool beside_pcie,
                        int64_t grid_items) {
  if (n_max <= 0) return;
  // An HBM-bound gather is capped at 8 workgroups per CU (each kernel narrows that further).  One that runs beside a
  // PCIe-bound kernel is throttled by the PCIe reads queued ahead of it whatever its width, and
  // in turn delays them; two workgroups per CU keep it out of the link's way (measured on 400-byte
  // rows, 506 k hits beside 253 k misses: the miss gather takes 2.40 ms beside a full-width hit
  // gather, 2.24 ms beside a narrow one, and the step 2.49 ms instead of 2.66 ms).
  const Where s{stream, ev_start, ev_stop, int64_t(di.num_cus) * (beside_pcie ? 2 : 8),
                (grid_items > 0 && grid_items < n_max) ? grid_items : n_max};
  const uintptr_t align = uintptr_t(src) | uintptr_t(dst) | uintptr_t(row_bytes);
  const int64_t width = chunk_width(align, row_bytes, streaming);
  const RowShape shape = row_shape(row_bytes, width);
  const char* from = static_cast<const char*>(src);
  char* to = static_cast<char*>(dst);
  auto rows = [&](auto vec, auto ragged) {
    typedef decltype(vec) VecT;
    constexpr bool kRagged = decltype(ragged)::value;
    if (streaming) launch_group<VecT, kRagged>(di, from, to, shape, row, srcrow, n_max, n_dev, dir, s);
    else if (by_lane_group<kRagged>(shape))
      launch_group_hbm<VecT, kRagged>(di, from, to, shape, row, srcrow, n_max, n_dev, dir, s);
    else launch_flat<VecT, kRagged>(di, from, to, shape, row, srcrow, n_max, n_dev, dir, s);
  };
  auto width_of = [&](auto vec) {
    if ((align & uintptr_t(width - 1)) == 0) rows(vec, std::false_type{});
    else rows(vec, std::true_type{});
  };
  if (width == 16) width_of(u32x4{});
  else if (width == 8) width_of(u32x2{});
  else if (width == 4) width_of(uint32_t{});
  else rows(uint16_t{}, std::false_type{});
}

int split_args(const DeviceInfo& di, const RowSources& r, const void* hit_src, const void* miss_src, void* dst,
               int64_t row_bytes, SplitArgs* out) {
  if (row_bytes < 16) return 0;
  const uintptr_t align = uintptr_t(miss_src) | uintptr_t(dst) | uintptr_t(row_bytes);
  const int64_t width = chunk_width(align, row_bytes, true);
  SplitArgs a = {};
  a.hit_src = static_cast<const char*>(hit_src);
  a.miss_src = static_cast<const char*>(miss_src);
  a.dst = static_cast<char*>(dst);
  a.hit_shape = row_shape(row_bytes, 16);
  a.miss_shape = row_shape(row_bytes, width);
  a.lists = r.lists;
  a.counters = r.counters;
  a.direct = r.direct;
  a.n_max = r.n_max;
  a.hit_lanes = group_lanes(a.hit_shape);
  a.miss_lanes = group_lanes(a.miss_shape);
  a.peers = r.peers;
  const int64_t items = (r.grid_items > 0 && r.grid_items < r.n_max) ? r.grid_items : r.n_max;
  const int64_t miss_pass = 256 / a.miss_lanes * kSplitMissUnroll, hit_pass = 256 / a.hit_lanes * kSplitHitUnroll;
  // Misses keep the width that suits the link; hits take six workgroups per CU with two rows per group in flight.  At 2 / 4 /
  // 6 / 8 per CU: 512-byte rows, 688 k of 2.4 M ids with 95 % of the table cached 291 / 252 / 233 / 227 us a call, 30 % cached and
  // 400-byte rows 2841 / 2843 / 2850 / 2845, 99.5 % cached 167 / 150 / 148 / 156.
  if (r.misses) a.miss_blocks = blocks_for((items + miss_pass - 1) / miss_pass, std::max(1, di.num_cus / 4));
  if (r.hits) a.hit_blocks = blocks_for((items + hit_pass - 1) / hit_pass, int64_t(di.num_cus) * 6);
  *out = a;
  return int(width);
}

bool launch_gather_split(const DeviceInfo& di, const RowSources& r, const void* hit_src, const void* miss_src, void* dst,
                         int64_t row_bytes, hipStream_t s) {
  SplitArgs a;
  const int width = split_args(di, r, hit_src, miss_src, dst, row_bytes, &a);
  if (width == 0) return false;
  const bool lines = row_bytes % 128 == 0, flat = width == 16 && row_bytes >= kFlatHitBytes;
  if (flat) {
    a.hit_inv = inverse(a.hit_shape.cpr);
    a.hit_epw = entries_per_wave(a.hit_shape, !lines && a.hit_shape.cpr > kWideChunks);
    a.hit_narrow = uint32_t(di.num_cus) * 2;
    const int64_t items = (r.grid_items > 0 && r.grid_items < r.n_max) ? r.grid_items : r.n_max;
    a.hit_blocks = blocks_for((items + 4 * a.hit_epw - 1) / (4 * a.hit_epw), int64_t(di.num_cus) * 6);
  }
  const dim3 grid{a.miss_blocks + a.hit_blocks}, block{256};
  if (flat && lines) hipLaunchKernelGGL((gather_split_kernel<u32x4, true, HitWalk::kFlatLines>), grid, block, 0, s, a);
  else if (flat) hipLaunchKernelGGL((gather_split_kernel<u32x4, true, HitWalk::kFlat>), grid, block, 0, s, a);
  else if (width == 16) hipLaunchKernelGGL((gather_split_kernel<u32x4, true, HitWalk::kGroups>), grid, block, 0, s, a);
  else if (width == 8) hipLaunchKernelGGL((gather_split_kernel<u32x2, false, HitWalk::kGroups>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gather_split_kernel<uint32_t, false, HitWalk::kGroups>), grid, block, 0, s, a);
  return true;
}

}  // namespace lgp
