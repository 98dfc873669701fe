// Internal declarations shared by the translation units of liblegion_prep.
// Host-side launchers only; kernels live in the .hip files.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <functional>
#include <string>
#include <vector>

#include "legion_prep.h"

namespace lgp {

// Device-side error bits (sticky, OR-ed into ctx->d_err).
enum : uint32_t { ERR_BAD_ID = 1u, ERR_OVERRUN = 2u };

// Vertex v is bit (v << spread_shift) of a dedup map, and marking it means setting that bit.
//   shift 0      one bit per vertex, set with an atomic OR.  Scattered atomics run at about 26 G/s on this
//                chip whatever their scope or target, so they bound the sampler of a large graph.
//   shift 3..5   a byte, half-word or word per vertex, set with a plain store of 1 (every writer of the entry
//                stores the same value).  Scattered stores run at 78-162 G/s and do not serialise on hot
//                lines, but the compaction has 8-32 times as many bytes to scan.
// Measured for three-hop calls of 8192 seeds (15, 10, 5): at 2.4 M vertices the last hop's kernel takes 25 us
// with bytes and 54 us with atomics (the best sparser bitmap, 4 bits per vertex); a whole call bits -> bytes
// 79 -> 49 us at 3 M vertices, 74 -> 64 at 6 M, 74 -> 77 at 12 M, 74 -> 94 at 25 M: bytes up to 2^23 vertices.
// Words instead of bytes on the smallest graphs keep neighbours' marks on different lines (10 k vertices:
// 2 us of a 33-us call).
// Calls of few seeds pay the larger scan too, and are still faster than with atomics on spread bits and two launches per
// compaction: 64 seeds (15, 10, 5) take 28.9 -> 21.8 us at 300 k vertices (words) and 700 k (half-words), 28.9
// -> 22.4 at 2.4 M and 28.8 -> 25.5 at 8 M (bytes); 16 seeds (10, 5) 20.6 -> 15.7 at 1 M, 20.9 -> 16.1 at 8 M.
constexpr int64_t kWordMapMaxVertices = int64_t(1) << 19;
constexpr int64_t kHalfMapMaxVertices = int64_t(1) << 20;
constexpr int64_t kByteMapMaxVertices = int64_t(1) << 23;
// Up to twice as many vertices the layout is chosen per call of the sampler (both maps are clear between calls; the pipeline
// inside a batch always marks bits): a compaction has 1 to 2.4 us more to scan, and many marks earn that back.  Bits -> bytes,
// 8192 seeds (15, 10, 5), and expected marks per vertex (expected_marks with the graph's own degrees): 8.5 M vertices of power-law
// degrees, mean 25, 91 -> 60 us, 0.18; 12 M, mean 12, 43.9 -> 42.3 and with the last frontier, which scans two maps at once, 46.0 ->
// 46.0, 0.053; 12 M of which a quarter own 40 edges per vertex 32.9 -> 38.1 and 34.8 -> 41.3, 0.017; 9 M of which 2 % own them 23.4 ->
// 24.4, below 0.001.  Of 480 calls on such graphs none that lies beyond the line is slower in bytes.  The mean degree alone cannot
// tell: by it the last two lie beyond the second (0.60, 0.78; 0.48).
constexpr int64_t kEitherMapMaxVertices = int64_t(1) << 24;
constexpr double kByteMarksPerVertex = 0.04;
inline int mark_shift(int64_t num_vertices) {
  return num_vertices <= kWordMapMaxVertices ? 5 : num_vertices <= kHalfMapMaxVertices ? 4
         : num_vertices <= kByteMapMaxVertices ? 3 : 0;
}

// How the compaction splits a map: `groups` workgroups of kCompactThreads threads, each thread taking
// words_per_thread 64-bit words in each of `passes` passes.  Two workgroups fit a CU, so 512 of them run at
// once; a larger map gets wider threads, then (beyond 2^28 bits) several passes.  (Up to 1024 narrower workgroups
// instead: 9.4 -> 11.1 us at 111 M vertices with 480 k marks, 12.9 -> 13.1 at 250 M with 506 k.)
constexpr int kCompactThreads = 1024;
constexpr int64_t kCompactMaxGroups = 512;
constexpr int kMaxPasses = 8;             // 2^31 bits / (512 groups * 1024 threads * 8 words * 64 bits)
struct MapGeom {
  int words_per_thread = 2;
  int passes = 1;
  int64_t groups = 1;
  int64_t words() const { return groups * passes * words_per_thread * kCompactThreads; }   // allocated, >= the map
};
inline MapGeom map_geometry(int64_t num_vertices, int shift) {
  const int64_t need = ((num_vertices << shift) + 63) / 64;
  MapGeom g;
  auto groups = [&] { const int64_t share = int64_t(g.passes) * g.words_per_thread * kCompactThreads; return (need + share - 1) / share; };
  while (g.words_per_thread < 8 && groups() > kCompactMaxGroups) g.words_per_thread *= 2;
  while (groups() > kCompactMaxGroups) ++g.passes;
  g.groups = groups();
  return g;
}

constexpr int32_t kDefaultPolls = 1 << 12;   // about 4 ms of polling before a share is counted by the one who waits

// The two dedup maps of a context and the status words of the compaction kernel (one per workgroup).  Both maps
// are clear between calls; every hop kernel clears the status words for the compaction that follows it.
struct DedupMaps {
  uint64_t* frontier = nullptr;
  uint64_t* gather = nullptr;
  uint64_t* status = nullptr;
  MapGeom geom;
  int32_t polls = kDefaultPolls;
};

// Binned marks, for large graphs.  A sample is not marked in a map but appended to a segment of its workgroup and its bin
// (2^shift consecutive vertices), at a place that a counter in LDS hands out: a plain store, where an atomic on a bit runs at
// 26 G/s.  The workgroup of a bin then sets the bits in LDS (bins.hip), so the map in HBM is neither read nor cleared.  Samples
// beyond a segment's room are marked in the frontier map, and the bin is flagged: right, but dearer than marks alone (columns_spread).
constexpr int kBinThreads = 1024;     // of a workgroup of either kernel
constexpr int kBinWriters = 512;      // most workgroups of a hop: two per CU
constexpr int kBinWords = 128;        // words of a segment
constexpr int kHeadWords = 16;        // of them in its head
constexpr int kMaxBins = 256;         // a workgroup each, one per CU
constexpr int kStatusCopies = 8;      // of the status words: one channel of memory does not answer all workgroups at once
constexpr int kBinStatusWords = 2 * kStatusCopies * kMaxBins;      // of 32 bits: for the list of a hop, and for the union
// Which calls: a hop saves about 25 us per million samples against atomics, and less against bytes; a list from bins costs 1 to 3 us
// more than the compaction of a map of up to 2^26 bits and less than that of one of more than 2^27.  So from expected_marks on, and a
// little more where every bin's workgroup has many seeds to look through.  Calls of lgp_sample_khop, map -> bins, and thousands of
// expected marks: 12 M vertices of power-law degrees, 8192 seeds (15, 10, 5) 42.4 -> 40.6 us, 634; 16000 (10, 10) 27.8 -> 27.6, 317; 8000
// (25, 10) 24.3 -> 25.9, 207.  16.5 M 63.9 -> 51.5, 1518; 38.4 -> 30.8, 582; 30.0 -> 27.0, 398; 4096 (15, 10) 23.3 -> 24.4, 173.  40 M
// 32000 (10, 10) 46.4 -> 36.7, 709; 31.3 -> 28.7, 355; 25.5 -> 27.4, 233; 64 (15, 10, 5) 25 -> 32 whatever the size.  111 M 61.6 -> 48.5,
// 713; 36.5 -> 33.4, 343; 31.5 -> 30.2, 225.  140 M 67.5 -> 50.7, 663; 41.3 -> 36.7, 327; 35.5 -> 31.9, 213; 64 (15, 10, 5) 33.9 -> 35.6, 5.
// 250 M 83.1 -> 55.5, 802; 48.3 -> 36.7, 372; 41.8 -> 33.3, 245; 45.2 -> 36.4, 6.  Degrees of 12 everywhere: 12 M, 8192 (15, 10, 5) 211 ->
// 175, 5778; 111 M 308 -> 195, 5972.  Fewer than 144 bins hold so many ids each that bytes are ahead (8.5 M vertices, 130 bins, 16000 (10,
// 10) 31.0 -> 33.3, 8192 (15, 10, 5) 59.1 -> 57.0), as they are on small graphs (2.4 M, 44.1 -> 49.9), and with 120000 seeds (10, 5) of
// 16.5 M vertices, degrees of 12 and the last frontier (230 -> 237; 250 M and power-law degrees 137 -> 97).
constexpr int64_t kBinMinVertices = int64_t(9) << 20, kBinMaxVertices = int64_t(1) << 28;
constexpr double kBinMarksPerSeed = 4.0;
inline int32_t bin_max_seeds(int64_t num_vertices) { return num_vertices <= int64_t(1) << 24 ? 1 << 16 : 1 << 17; }
inline double bin_marks(int64_t num_vertices) {
  return num_vertices <= int64_t(1) << 24 ? 510e3 : num_vertices <= int64_t(1) << 26 ? 400e3
         : num_vertices <= int64_t(1) << 27 ? 200e3 : num_vertices <= int64_t(5) << 25 ? 60e3 : 0.0;
}
// Most workgroups of a hop.  Half as many segments to read and their heads fuller, against half as many waves to hide the loads: with
// up to six samples per vertex a wave takes ten vertices and more at once, and one workgroup per CU is enough.  Calls at two -> one:
// 8192 seeds (15, 10, f) of 111 M vertices, f = 2 47.4 -> 45.4 us, 3 46.3 -> 44.5, 5 46.8 -> 45.5, 6 48.5 -> 47.1, 8 48.5 -> 49.0, 12 51.3
// -> 52.8; 32000 (15, 10, 5) 103 -> 95.5, of 12 M 141 -> 127; (10, 6) 39.1 -> 38.8, (10, 7) 40.6 -> 40.7, (10, 16) 48.3 -> 53.0.
inline int32_t bin_writers(int32_t fanout) { return fanout <= 6 ? kBinWriters / 2 : kBinWriters; }
// And, where bytes are the other way (up to 2^24 vertices), only while segments hold what a hop promises: samples beyond their room are
// marked with atomics in a map of bits, which the lists then read and clear as well.  A hop that promises more than kBinFill times
// its room takes all workgroups, and a call with a hop of more than kBinFill times the room of those marks bytes.  Calls, bytes -> one
// workgroup per CU -> two, and the promise over the room of two: uniform degrees, 9.5 M vertices 16384 seeds (10, 10, 5) 284 -> 282 -> 240
// us, 0.79; 20000 (15, 10, 5) 376 -> 426 -> 321, 1.11; 32000 529 -> 671 -> 539, 1.65; 65536 890 -> 1170 -> 1032, 2.8; 12 M 65536 (25, 10)
// 438 -> 406, 1.28; 16384 (15, 10, 10) 636 -> 700, 1.84; 16.5 M 65536 (15, 25) 739 -> 632, 1.46.  Where popularity is skewed hops are
// smaller than promised: 9.5 M of mean degree 40, 32000 (15, 10, 5) 226 -> 180 -> 192, 1.24; 65536 329 -> 332 -> 292, 2.2; 12 M of 60 289 ->
// 252 -> 265, 1.36.  Against bits no promise is too large (33 M, 131072 (15, 10, 5), 4.4 times the room: 3824 -> 3300).
constexpr double kBinFill = 1.5;
// Against bytes one hop alone is no gain either: every bin's workgroup looks through all seeds, and there are more than 8000 of them
// before one hop has enough samples.  Bytes -> bins, 65536 seeds: 9.5 M vertices of degree 12 (25) 25.8 -> 29.4 us, (64) 28.8 -> 34.1;
// 16.5 M (12) 26.6 -> 27.4; 12 M of power-law degrees, mean 40, (40) 32.6 -> 39.0; 9.5 M of degree 64 (40) 76.4 -> 89.1, 32000 seeds 44.0 ->
// 47.5.  Faster were those that take all of each row, (64) there 84.6 -> 70.9.  Against bits that holds for one sample per seed only, from
// kBinSeedsOfOne seeds on: 168 M vertices, 131072 seeds (1) 26.7 -> 32.7, (2) 32.1 -> 33.6, (4) 42.5 -> 36.4; 65536 (1) 19.7 -> 21.9, (3) 25.6 ->
// 21.8; 250 M 28.6 -> 32.6, 34.1 -> 33.2, 44.8 -> 35.6, 21.8 -> 22.8, 27.3 -> 22.0.
constexpr int32_t kBinSeedsOfOne = 1 << 16;
// And only graphs whose column ids are spread: where a call's samples crowd into few bins, few workgroups make its list and most samples
// are marked in the map after all.  Degrees of 12, map -> bins, 8192 (15, 10, 5) and 8000 (25, 10): all columns within half of
// the ids 12 M vertices 199 -> 179 us and 41 -> 38, 111 M 310 -> 218 and 68 -> 39; a third 160 -> 206, 39 -> 42 and 311 -> 260,
// 68 -> 44; an eighth 97 -> 243, 39 -> 62 and 329 -> 379, 74 -> 65; a 64th 83 -> 267, 49 -> 132 and 413 -> 805, 129 -> 247.
// Columns within 4096 ids of their rows crowd where seeds do: seeds spread 147 -> 186, 37 -> 48 and 196 -> 217, 48 -> 60; a run of
// ids 52 -> 194, 33 -> 138 and 157 -> 226, 134 -> 163; one column in 16 so and the others spread, a run of ids 216 -> 160, 45 -> 45
// and 315 -> 214, 83 -> 68; one in 32 214 -> 156, 43 -> 40 and 316 -> 202, 80 -> 61.  So for any number of bins, w of them may take
// one column in 20 and twice their part: of the bins themselves, and of those around each column's row.
constexpr double kCrowdedColumns = 0.05, kCrowdedBins = 2.0;
inline bool columns_spread(const uint32_t* counts, int32_t bins) {
  uint32_t by_bin[kMaxBins];
  std::copy(counts, counts + kMaxBins, by_bin);
  std::sort(by_bin, by_bin + kMaxBins, std::greater<uint32_t>());
  double total = 0, fullest = 0, near = 0;
  for (uint32_t n : by_bin) total += double(n);
  if (total == 0) return false;            // no edges, so there will be no samples
  for (int32_t w = 0; w < bins; ++w) {
    fullest += double(by_bin[w]);
    near += double(counts[kMaxBins + w]);
    if (fullest > total * (kCrowdedColumns + kCrowdedBins * double(w + 1) / double(bins))) return false;
    if (near > total * (kCrowdedColumns + kCrowdedBins * double(2 * w + 1) / double(bins))) return false;
  }
  return true;
}
inline int bin_shift(int64_t num_vertices) {
  int shift = 16;
  while ((num_vertices - 1) >> shift >= kMaxBins) ++shift;
  return shift;
}
struct BinMaps {                      // all null while the context holds no segments (hold_segments)
  // Segments [bin][workgroup of the hop]; word 0 of a segment is its count, which may be larger than its room.
  uint32_t* heads = nullptr;          // the first kHeadWords words of each, which are always read
  uint32_t* tails = nullptr;          // the others
  uint32_t* spilled = nullptr;        // [bin]: the frontier map has taken something; all zero between calls.  And [kMaxBins], below
  int32_t* first = nullptr;           // [hop][kMaxBins + 1]: where the ids of each bin begin in frontier `hop`
  // The number of this call, a value of its own.  spilled[kMaxBins] is that of the last call that met a vertex without a row, or with
  // one that makes no sense: its seeds are looked at one by one.  The context's error word does not say so: kernels of a gather on
  // another stream set it and lgp_check on that stream clears it while this call runs.
  uint32_t call = 0;
  int32_t shift = 0, bins = 0;        // bins == 0: this context marks maps in every call
};

struct DeviceInfo {
  int device = 0;
  int num_cus = 256;
  int spread_shift = 0;
};

// Row table: one 64-bit entry per vertex, resident in HBM, so that finding a vertex's adjacency
// costs one load whether or not the row is cached.
//   bit 63      1 = the row's column ids are in the topology cache, 0 = in CPU memory
//   bits 62..24 offset of the row's first column id inside that array (39 bits)
//   bits 23..0  degree; kRowDegOverflow means "too large to pack: use the CPU-resident CSR"
constexpr uint64_t kRowCachedBit = 1ull << 63;
constexpr uint32_t kRowDegOverflow = 0xFFFFFFu;
constexpr int kRowStartShift = 24;
constexpr uint64_t kRowStartMask = (1ull << 39) - 1;

// Pointers every sampling kernel needs.
struct TopoView {
  const uint64_t* row_tab;   // row table (HBM)
  const void* h_indptr;      // CPU-resident CSR (GPU-addressable); offsets only read for overflow rows
  const int32_t* h_indices;
  const int32_t* t_indices;  // cached column ids (HBM)
  int32_t indptr_bytes;
  int64_t num_vertices;
  bool over_pcie;            // h_indices lies in CPU memory, and not all rows are cached
};

// ---- sampler.hip ----------------------------------------------------------
// What the first hop of the intra-batch pipeline does beside: listed[0 .. n_seeds) = the seeds, seg[0] = 0, seg[1] = n_seeds, and
// zeroed[0 .. n_zeroed) = 0 (at most 256), the counters of the groups behind the seeds.  A launch ahead of the pipeline for that, one
// behind it that cleared the map and copied the bounds, and one per partition that zeroed its counters were small ones of 4 to 5 us:
// calls with them -> without, 8192 seeds (15, 10, 5) of 2.4 M vertices, 400-byte rows, all cached 143.7 -> 138, (10) 23.9 -> 19.2;
// (25, 10) of 10 M, 256-byte rows 64.7 -> 60.0; 4000 (10, 10, 5) of 1 M, 256-byte rows, 90 % cached 113.5 -> 103.6.
struct FirstGroup {
  int32_t* listed = nullptr;
  int32_t* seg = nullptr;
  int32_t* zeroed = nullptr;
  int32_t n_zeroed = 0;
};
// Expand frontier[0 .. *n_frontier) with fan-out f at hop `hop`; the array has room for `cap` ids.  Writes nbr / cnt
// (either may be null), marks every sampled neighbour in `mark_bits` (bit v << di.spread_shift),
// adds cnt to topo_hot[v] if topo_hot is given.  With self_bits given (first hop) the
// frontier is the seed list: exactly `cap` ids, *n_frontier is written (= cap) instead of
// read, and every valid seed is marked in self_bits (and listed as `first` says).  status[0 .. n_status) is cleared for the compaction
// that follows.
void launch_sample_hop(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier,
                       int64_t cap, int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt,
                       uint32_t* mark_bits, uint32_t* self_bits, uint32_t* topo_hot, uint32_t* d_err, uint64_t* status,
                       int64_t n_status, hipStream_t s, const FirstGroup& first = FirstGroup{});

// The same for binned marks: no hotness, and seeds are not marked; what finds no room is marked in mark_bits.  status[0 ..
// kBinStatusWords) of 32 bits is cleared.  At most `writers` workgroups; returns their number, which is that of the segments of a bin.
int32_t launch_sample_hop_binned(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier,
                                 int64_t cap, int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt,
                                 const BinMaps& m, int32_t writers, uint32_t* mark_bits, uint32_t* d_err, uint64_t* status, hipStream_t s);

// Pre-sampling: staged[0 .. n_edges) = h_indices[0 .. n_edges), from CPU memory to HBM.  The two addresses are equal modulo 16.
void launch_stage_topology(const int32_t* h_indices, int32_t* staged, int64_t n_edges, hipStream_t s);

// ---- compact.hip ----------------------------------------------------------
struct CompactArgs {
  uint64_t* bits;
  uint64_t* other;
  uint64_t* status;
  int32_t* out;       // list of the marks in `bits`, nullptr = not wanted
  int64_t out_cap;
  int32_t* n_out;
  int32_t* out2;      // second list
  int64_t out2_cap;
  int32_t* n_out2;
  int32_t* seg;
  int32_t* stats;     // last listing: stats[stats_slot] = its length, the other one of the two = 0; may be null
  int32_t stats_slot;
  uint32_t* d_err;
  int32_t shift, passes;
  int32_t polls;      // looks at a status word before the share is counted instead
};
// Frontier map -> ascending id list out[0 .. *n_out); its marks are added to the gather map, the frontier map is
// cleared.  Every compaction follows a launch_sample_hop on the same stream, which clears the status words.
void launch_compact(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                    uint32_t* d_err, hipStream_t s);
// Gather map -> ascending id list; the gather map is cleared.
void launch_compact_gather(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                           uint32_t* d_err, hipStream_t s);
// Both of the above in one pass: out = the frontier map's ids, all = the ids of either map; both maps are cleared.
void launch_compact_both(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                         int32_t* all, int64_t all_cap, int32_t* n_all, uint32_t* d_err, hipStream_t s);
// Compaction for the intra-batch pipeline: like launch_compact, and in addition the vertices not yet in the gather
// map -- the ones this hop reached first -- are appended, ascending, to listed[seg[0] ..], and seg[1] = seg[0] +
// their number (seg: device int32 pair).  With out == nullptr no frontier list is written; n_listed, if given, also
// receives seg[1].  last: no hop follows; both maps are cleared, and stats, if given, receives {0, 0} but for seg[1] at stats_slot.
void launch_compact_new(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                        int32_t* listed, int64_t listed_cap, int32_t* seg, int32_t* n_listed, bool last, int32_t* stats,
                        int32_t stats_slot, uint32_t* d_err, hipStream_t s);
// Pre-sampling: bump[id] += 1 for every id of the gather map, which is cleared; acc[0] += sizes[0] + ... (the
// frontier sizes of the batch).
void launch_bump(const DeviceInfo& di, const DedupMaps& m, uint32_t* bump, const int32_t* sizes, int32_t n_sizes,
                 unsigned long long* acc, hipStream_t s);

// ---- bins.hip -------------------------------------------------------------
// What the samples of one binned hop are turned into.  With n_list: their ascending list, and in list_first (optional) where the ids
// of each bin begin in it.  With n_all: the ascending union of them, the seeds and frontiers 1 .. inner, whose bins begin where
// `first` says.  Every launch follows a launch_sample_hop_binned on the same stream, which clears the status words.
struct BinArgs {
  BinMaps maps;
  int32_t writers;          // segments of a bin
  uint64_t* spill;          // the frontier map
  uint32_t* status;         // kBinStatusWords
  int32_t polls;
  uint32_t* d_err;
  int32_t* list;
  int64_t list_cap;
  int32_t *n_list, *list_first;
  int32_t* all;
  int64_t all_cap;
  int32_t* n_all;
  const int32_t* seeds;
  int32_t n_seeds, inner;
  const int32_t* frontier[LGP_MAX_HOPS];
  const int32_t* first;
  TopoView tv;
};
void launch_list_bins(const BinArgs& a, hipStream_t s);

// ---- gather.hip -----------------------------------------------------------
// Look up every id in the feature remap and append (row, slot) to the hit list (list 0) or
// (row, id) to the miss list (list 1).  With n_lists = 3, hits whose slot lies outside
// [local_lo, local_hi) go to list 2 instead: rows cached by another member of a clique.
// counters[l] = entries of list l, l < n_lists (zeroed here, unless the caller says that they are zero).
struct PartLists {
  int32_t* row[3];
  int32_t* src[3];
};
void launch_partition(const DeviceInfo& di, const int32_t* ids, int64_t n_max, const int32_t* n_dev,
                      const int32_t* f_remap, int64_t num_vertices, const PartLists& out, int n_lists,
                      int32_t local_lo, int32_t local_hi, int32_t* counters, uint32_t* d_err, hipStream_t s,
                      const int32_t* window = nullptr, int64_t grid_items = 0, bool zeroed = false);
// "Direct" launches skip the partition: when every row is cached (or none is) the source-row
// array is the caller's id list itself.
struct DirectIds {
  const int32_t* remap;   // id -> cache slot (everything cached); nullptr = the id is the source row (nothing cached)
  int64_t num_vertices;   // > 0: entries are vertex ids, validate them; 0: entries are trusted list entries
  int32_t* stats;         // {n_hit, n_miss} to fill in, or nullptr
  int32_t stats_slot;     // which of the two gets the row count
  uint32_t* d_err;
  const int32_t* window;  // device {begin, end}: only these entries of the array are gathered (nullptr = all)
};

// dst[row[e], :] = src[srcrow[e], :] for e < *n_dev (or n_max if n_dev is null); rows are
// row_bytes wide; `row` and `srcrow` may each be null (= e).  streaming = source is read once over
// PCIe (non-temporal loads, one lane group per row).
// With ev_start and ev_stop given (and n_max > 0) the kernel's own start and stop times are recorded
// into them.  beside_pcie: this HBM-bound gather runs at the same time as a PCIe-bound one.  With
// dir.window given, entries [window[0], window[1]) are gathered (their output rows keep their absolute
// numbers) and grid_items is the most entries the window can hold, for sizing the grid.
void launch_gather_rows(const DeviceInfo& di, const void* src, void* dst, int64_t row_bytes, const int32_t* row,
                        const int32_t* srcrow, int64_t n_max, const int32_t* n_dev, bool streaming, hipStream_t s,
                        const DirectIds& dir = DirectIds{nullptr, 0, nullptr, 0, nullptr, nullptr},
                        hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr, bool beside_pcie = false,
                        int64_t grid_items = 0);

// Rows to copy from their two sources side by side.  With counters: the lists of a partition, counters as launch_partition
// left them (lists[2] with peers; rows of lists[1] are misses).  Without: the caller's list of ids is lists.src[0] (hits) or
// lists.src[1] (misses), and direct.window says which entries.
struct RowSources {
  PartLists lists;
  const int32_t* counters;
  DirectIds direct;
  int64_t n_max, grid_items;   // as for launch_gather_rows
  bool hits, misses, peers;
};
// One launch for both, hits from hit_src and misses from miss_src in CPU memory.  False, and nothing is launched, for rows
// below 16 bytes.
bool launch_gather_split(const DeviceInfo& di, const RowSources& r, const void* hit_src, const void* miss_src, void* dst,
                         int64_t row_bytes, hipStream_t s);
// Arguments of the device code for that; returns the width of a miss's chunks, 0 for rows below 16 bytes.
struct SplitArgs;
int split_args(const DeviceInfo& di, const RowSources& r, const void* hit_src, const void* miss_src, void* dst,
               int64_t row_bytes, SplitArgs* out);

// ---- extract.hip ----------------------------------------------------------
// A sampling hop (arguments as launch_sample_hop) and, beside it in the same launch, the rows r; not for rows below 16 bytes.
void launch_hop_and_rows(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier, int64_t cap,
                         int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt, uint32_t* mark_bits,
                         uint32_t* self_bits, uint32_t* d_err, uint64_t* status, int64_t n_status, const RowSources& r,
                         const void* hit_src, const void* miss_src, void* dst, int64_t row_bytes, hipStream_t s,
                         const FirstGroup& first = FirstGroup{});
// stats[0 .. 2) = column sums of the n_seg x 3 matrix seg_counters, first two columns.
void launch_sum_counters(const int32_t* seg_counters, int32_t n_seg, int32_t* stats, hipStream_t s);
// Clears words 64-bit words of a map.
void launch_clear_map(const DeviceInfo& di, uint64_t* map, int64_t words, hipStream_t s);

// ---- blocks.hip -----------------------------------------------------------
constexpr int kScanTile = 1024;   // elements per workgroup of the counts -> offsets scan
// Everything one graph-constructor call reads and writes.  cap[h] = 0 marks a frontier that
// is empty in the worst case: its lists are not touched, its hop still gets blk_indptr[h][0] = 0.
struct BlocksArgs {
  int32_t n_hops;
  int64_t num_vertices;
  const int32_t* frontier[LGP_MAX_HOPS + 1];   // [0] = the seeds
  const int32_t* n_frontier;                   // device int32[n_hops + 1]
  int64_t cap[LGP_MAX_HOPS + 1];
  const int32_t* gather_ids;
  const int32_t* n_gather;
  int64_t gather_cap;
  const int32_t* nbr[LGP_MAX_HOPS];
  const int32_t* cnt[LGP_MAX_HOPS];
  int32_t fanout[LGP_MAX_HOPS];
  int64_t* blk_indptr[LGP_MAX_HOPS];
  int32_t* blk_src[LGP_MAX_HOPS];
  int32_t* feat_row[LGP_MAX_HOPS + 1];
  int32_t* table;                              // n_hops + 1 tables of table_stride entries each (at least num_vertices, even)
  int64_t table_stride;
  int64_t* tile_sums;                          // hop h owns cap[h] / kScanTile + 1 entries from tile_base[h]
  int64_t tile_base[LGP_MAX_HOPS];
  uint32_t* unordered;                         // [j] == call: frontier j is not ascending (n_hops + 1 words)
  uint32_t call;                               // number of this call (a value of its own, so that nothing is cleared)
};
void launch_build_blocks(const DeviceInfo& di, const BlocksArgs& a, hipStream_t s);

// ---- cache.hip ------------------------------------------------------------
struct CachePlan {
  int64_t n_topo = 0, topo_edges = 0, n_feat = 0;
  uint64_t topo_bytes = 0, feat_bytes = 0;
};
// Rank vertices by (hotness descending, id ascending) into order[V].  Synchronous parts
// use `s`.  Returns hipSuccess or the failing HIP status.
hipError_t rank_by_hotness(const uint32_t* hot, int64_t num_vertices, int32_t* order, hipStream_t s);
// deg[v] = indptr[v + 1] - indptr[v], streamed from CPU memory.
void launch_degrees(const DeviceInfo& di, const void* h_indptr, int32_t indptr_bytes, int64_t num_vertices,
                    int32_t* deg, hipStream_t s);
// Inclusive scan of the Eq. 3 cost (deg * 4 + 8) along `order`; cost_scan has V entries.
hipError_t scan_topo_cost(const int32_t* deg, const int32_t* order, int64_t num_vertices, uint64_t* cost_scan,
                          hipStream_t s);
// result[0] = number of entries of the ascending array scan[0..n) that are <= budget,
// result[1] = scan[that - 1] (0 if none).  Device-side binary search.
void launch_prefix_within_budget(const uint64_t* scan, int64_t n, uint64_t budget, uint64_t* result, hipStream_t s);
// t_indptr[r] = edges before rank r, r = 0 .. n_topo (derived from the cost scan).
void launch_topo_offsets(const DeviceInfo& di, const uint64_t* cost_scan, int64_t n_topo, int64_t* t_indptr,
                         hipStream_t s);
// Copy the adjacency of order[0 .. n_topo) from CPU memory into the cached CSR.
void launch_fill_topo(const DeviceInfo& di, const void* h_indptr, int32_t indptr_bytes, const int32_t* h_indices,
                      const int32_t* order, int64_t n_topo, const int64_t* t_indptr, int32_t* t_indices,
                      hipStream_t s);
// Inclusive scan of hot[order[r]] along a ranking (64-bit sums); hot_scan has V entries.
hipError_t scan_hotness(const uint32_t* hot, const int32_t* order, int64_t num_vertices, uint64_t* hot_scan,
                        hipStream_t s);
// One thread per candidate plan: boundary of Eq. 3 by binary search in the cost scan, Eq. 6 by
// division, sums from the hotness scans, exact 128-bit comparison key; *best = first smallest key.
void launch_alpha_search(const uint64_t* cost_scan, const uint64_t* hot_t_scan, const uint64_t* hot_f_scan,
                         int64_t num_vertices, uint64_t row_bytes, const uint64_t* m_topo, uint64_t total_budget,
                         uint64_t n_tsum, uint64_t per_row, int32_t n_alpha, lgp_plan_point* points, int32_t* best,
                         hipStream_t s);
void launch_fill_i32(const DeviceInfo& di, int32_t* p, int64_t n, int32_t value, hipStream_t s);
// out = in reordered by ascending Philox key of the position (one permutation per epoch).  Synchronises `s`.
hipError_t shuffle_by_key(const DeviceInfo& di, const int32_t* in, int32_t* out, int64_t n, uint64_t seed,
                          uint32_t epoch, hipStream_t s);
// Algorithm 1 for k_g hotness rows: column sums, ranking, arg-max owner, per-GPU queues.  counts
// (device uint64[k_g]) receives the queue lengths.  Synchronises `s`.
hipError_t cslp_rank(const DeviceInfo& di, int32_t k_g, int64_t num_vertices, const uint32_t* hot, uint64_t* acc,
                     int32_t* order, int32_t* owner, int32_t* queues, unsigned long long* counts, hipStream_t s);
// row_tab[v] = (not cached, CPU offset, degree) for every vertex, streamed from the CPU-resident offsets.
// counts[k] += vertices of degree k, counts[LGP_MAX_FANOUT] += those of that degree and more.
void launch_count_degrees(const DeviceInfo& di, const uint64_t* row_tab, int64_t num_vertices, uint32_t* counts, hipStream_t s);
// counts[bin] += columns of the bin, counts[kMaxBins + d] += columns that lie d bins from their row, of kColumnSamples column ids.
constexpr int64_t kColumnSamples = 1 << 16;
void launch_count_columns(const DeviceInfo& di, const uint64_t* row_tab, const int32_t* indices, int64_t num_vertices,
                          int64_t num_edges, int shift, uint32_t* counts, hipStream_t s);
void launch_init_row_table(const DeviceInfo& di, const void* h_indptr, int32_t indptr_bytes, int64_t num_vertices,
                           uint64_t* row_tab, hipStream_t s);
// row_tab[order[r]] = (cached, t_indptr[r], degree) for r < n_topo (rows too long to pack keep their CPU entry).
void launch_set_cached_rows(const DeviceInfo& di, const int32_t* order, int64_t n_topo, const int64_t* t_indptr,
                            uint64_t* row_tab, hipStream_t s);
// p[k] = k for k < n.
void launch_iota_i32(const DeviceInfo& di, int32_t* p, int64_t n, hipStream_t s);
// remap[order[r]] = r for r < n.
void launch_scatter_rank(const DeviceInfo& di, const int32_t* order, int64_t n, int32_t* remap, hipStream_t s);

}  // namespace lgp
