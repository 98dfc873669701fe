// Device code of a sampling hop that more than one kernel is built from.
#pragma once

#include "common.hpp"
#include "philox_dev.hpp"

namespace lgp {
namespace {

// Mark vertex u in a dedup map (see mark_shift): a plain store where it has an entry of its own, else one bit.
template <int SHIFT>
__device__ __forceinline__ void mark_vertex(uint32_t* map, int32_t u) {
  if (SHIFT == 3)
    __hip_atomic_store(reinterpret_cast<uint8_t*>(map) + u, uint8_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  else if (SHIFT == 4)
    __hip_atomic_store(reinterpret_cast<uint16_t*>(map) + u, uint16_t(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  else if (SHIFT == 5)
    __hip_atomic_store(map + u, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
  else
    atomicOr(&map[uint32_t(u) >> 5], 1u << (uint32_t(u) & 31u));
}

// Floyd's subset algorithm for all slots of a wave at once.  Slot i draws t[i] in 0 .. j[i] = d - f + i and takes t[i], or
// j[i] if t[i] is taken already.  After slot k both outcomes leave t[k] among the taken, so slot i has to move to j[i] if and
// only if t[i] == t[k] for some k < i, or t[i] == j[m] for the one slot m = t[i] - (d - f) < i and slot m has moved.  The
// first needs no order; the second follows a chain of ever smaller slots, one ballot per step, and hardly ever takes two.
// Returns whether the calling lane's slot moves; `first` = lane of slot 0, every lane of the wave calls this.
__device__ __forceinline__ bool floyd_moves(bool big, int32_t t, int32_t d, int32_t f, int slot, int first) {
  bool taken = false;
  int32_t x = t;
  for (int r = 1; r < f; ++r) {
    x = __builtin_amdgcn_update_dpp(x, x, 0x138, 0xf, 0xf, false);   // wave_shr:1, now the t of r lanes before
    taken |= slot >= r && x == t;
  }
  taken = taken && big;
  const int32_t m = t - (d - f);
  const bool after = big && m >= 0 && m < slot;
  uint64_t moved = __ballot(taken);
  if (__any(after)) {
    for (;;) {
      const uint64_t next = __ballot(taken || (after && ((moved >> (first + m)) & 1ull)));
      if (next == moved) break;
      moved = next;
    }
  }
  return (moved >> (threadIdx.x & 63)) & 1ull;
}

// One hop: see launch_sample_hop.
struct HopArgs {
  TopoView tv;
  const int32_t* frontier;
  int32_t* n_frontier;
  int64_t cap;
  int32_t f, lanes, hop;   // fan-out, lanes of a vertex (hop_lanes)
  uint32_t k0, k1;
  int32_t* nbr;
  int32_t* cnt;
  uint32_t* mark_bits;
  uint32_t* self_bits;
  uint32_t* topo_hot;
  uint32_t* d_err;
  uint64_t* status;
  int32_t n_status;
  BinMaps bins;            // of a binned hop
  int32_t* listed;         // first hop of the intra-batch pipeline: the seeds are listed there as given, and
  int32_t* seg;            // seg[0], seg[1] are the bounds of that group,
  int32_t* zeroed;         // and the n_zeroed counters of the groups behind it are cleared
  int32_t n_zeroed;
};

// Append vertex u to this workgroup's segment of its bin; used = entries of those segments, by bin (LDS).
constexpr int kBinned = -1;               // in the place of a map's shift
__device__ __forceinline__ void append_to_bin(const HopArgs& a, uint32_t* used, uint32_t block, uint32_t blocks, int32_t u) {
  const uint32_t bin = uint32_t(u) >> a.bins.shift, at = atomicAdd(&used[bin], 1u) + 1u, segment = bin * blocks + block;
  if (at < uint32_t(kHeadWords)) {
    a.bins.heads[segment * uint32_t(kHeadWords) + at] = uint32_t(u);
  } else if (at < uint32_t(kBinWords)) {
    a.bins.tails[segment * uint32_t(kBinWords - kHeadWords) + at - kHeadWords] = uint32_t(u);
  } else {
    mark_vertex<0>(a.mark_bits, u);
    if (at == uint32_t(kBinWords)) a.bins.spilled[bin] = 1;      // the workgroup's first: not all samples store to one address
  }
}

// Marks bound this kernel (last hop of 190 k vertices x 5 at 2.4 M vertices: 23 us with its 950 k byte marks, 11 without;
// 490 k atomic marks of a map of 250 M: 24 and 9; appended to segments instead they take 13); what is left is loads and issue slots, so lanes are packed without gaps (but see
// hop_lanes).  Against a power of two of lanes per vertex and a chain of fanout - 1 broadcasts for Floyd's test, calls on
// 2.4 M vertices from 8192 seeds: fan-outs 17, 17 28.2 -> 25.1 us, 64 17.5 -> 15.4, 9, 9 21.2 -> 20.2, 15, 10, 5 with blocks
// and gather 190 -> 186; 25 or 3, 3, 3 and graphs with atomic marks are level.
// The caller is workgroup `block` of `blocks` that share the frontier.
template <int SHIFT, int WAVES = 4>
__device__ __forceinline__ void sample_hop(const HopArgs& a, uint32_t block, uint32_t blocks, uint32_t* used = nullptr) {
  const uint64_t* __restrict__ row_tab = a.tv.row_tab;
  const int32_t* __restrict__ h_indices = a.tv.h_indices;
  const int32_t* __restrict__ frontier = a.frontier;
  int32_t* __restrict__ nbr = a.nbr;
  int32_t* __restrict__ cnt = a.cnt;
  uint32_t* __restrict__ mark_bits = a.mark_bits;
  uint32_t* __restrict__ self_bits = a.self_bits;
  const int32_t f = a.f, lanes = a.lanes;
  // self_bits != nullptr: this is the first hop; the frontier is the caller's seed list of `cap`
  // ids, whose size is published here and whose members are marked in the gather set.
  const bool seeds = SHIFT == kBinned ? a.hop == 0 : self_bits != nullptr;
  if (seeds && block == 0 && threadIdx.x == 0) {
    *a.n_frontier = int32_t(a.cap);
    if (a.seg) {
      a.seg[0] = 0;
      a.seg[1] = int32_t(a.cap);
    }
  }
  if (block == 0) {
    for (int k = threadIdx.x; k < a.n_status; k += WAVES * 64) a.status[k] = 0;
    if (int(threadIdx.x) < a.n_zeroed) a.zeroed[threadIdx.x] = 0;
  }
  const int per_wave = 64 / lanes;                // vertices per wave pass
  const int lane = threadIdx.x & 63;
  const int sub = lane / lanes, slot = lane - sub * lanes;   // vertex of this lane in the pass, sample slot (below f)
  // Three loads depend on one another (frontier id -> row-table entry -> column id).  The id is loaded two passes ahead
  // and the row-table entry one pass ahead, so that a pass waits for its column ids only (two hops of 17 from 8192 seeds
  // of 2.4 M vertices 25.8 -> 25.1 us, one hop of 64 16.0 -> 15.4).
  const int64_t wave = int64_t(block) * WAVES + (threadIdx.x >> 6);
  const int64_t stride = int64_t(blocks) * WAVES * per_wave;
  const uint64_t nv = uint64_t(a.tv.num_vertices);
  auto id_at = [&](int64_t g, int64_t end) { return sub < per_wave && g < end ? frontier[g] : -1; };
  auto row_of = [&](int32_t v) { return uint32_t(v) < nv ? row_tab[v] : 0; };
  int64_t g0 = wave * per_wave;
  // The first two ids are loaded with the frontier's size still on its way: the frontier has room for `cap` (calls replayed from
  // a graph, 111 M vertices, 64 seeds (15, 10, 5) 24.1 -> 23.4 us; 2.4 M, 8192 (25, 10) 24.8 -> 24.4).
  int32_t v_next = id_at(g0 + sub, a.cap), v_after = id_at(g0 + stride + sub, a.cap);
  int64_t n = seeds ? a.cap : int64_t(*a.n_frontier);
  if (n > a.cap) n = a.cap;                           // never trust a count beyond the buffer
  if (g0 + sub >= n) v_next = -1;
  if (g0 + stride + sub >= n) v_after = -1;
  uint64_t e_next = row_of(v_next);
  for (; g0 < n; g0 += stride) {
    const int64_t g = g0 + sub;
    const bool active = sub < per_wave && g < n;
    const int32_t v = v_next;
    const uint64_t e = e_next;
    v_next = v_after;
    v_after = id_at(g + 2 * stride, n);
    e_next = row_of(v_next);
    bool bad = active && uint32_t(v) >= nv;
    int64_t s = 0, d64 = 0;
    const int32_t* colbase = h_indices;
    if (active && !bad) {
      const uint32_t d24 = uint32_t(e) & kRowDegOverflow;
      if (d24 != kRowDegOverflow) {
        s = int64_t((e >> kRowStartShift) & kRowStartMask);
        d64 = d24;
        if (e & kRowCachedBit) colbase = a.tv.t_indices;
      } else if (a.tv.indptr_bytes == 8) {         // degree does not fit the entry: CPU-resident CSR
        s = static_cast<const int64_t*>(a.tv.h_indptr)[v];
        d64 = static_cast<const int64_t*>(a.tv.h_indptr)[int64_t(v) + 1] - s;
      } else {
        s = static_cast<const int32_t*>(a.tv.h_indptr)[v];
        d64 = static_cast<const int32_t*>(a.tv.h_indptr)[int64_t(v) + 1] - s;
      }
      if (d64 < 0 || d64 > 0x7fffffff) { bad = true; d64 = 0; }
    }
    if (bad) {
      if (slot == 0) atomicOr(a.d_err, ERR_BAD_ID);
      if (SHIFT == kBinned) a.bins.spilled[kMaxBins] = a.bins.call;
      d64 = 0;
    }
    const int32_t d = int32_t(d64);
    const bool big = active && d > f;
    int32_t p = slot;                              // position inside the row
    if (__any(big)) {
      const int32_t j = d - f + slot;
      const int32_t t = int32_t(
          __umul64hi(philox_draw64(a.k0, a.k1, uint32_t(v), uint32_t(a.hop), uint32_t(slot)), uint64_t(uint32_t(j)) + 1));
      const bool moves = floyd_moves(big && slot < f, t, d, f, slot, lane - slot);
      if (big) p = moves ? j : t;
    }
    if (active && slot < f) {
      int32_t u = -1;
      if (big || slot < d) {
        u = colbase[s + p];
        if (uint32_t(u) >= nv) {
          atomicOr(a.d_err, ERR_BAD_ID);
          u = -1;
        } else if (SHIFT == kBinned) {
          append_to_bin(a, used, block, blocks, u);
        } else {
          mark_vertex<SHIFT>(mark_bits, u);
        }
      }
      if (nbr) nbr[g * f + slot] = u;
      if (slot == 0) {
        if (SHIFT != kBinned && self_bits) {
          if (!bad) mark_vertex<SHIFT>(self_bits, v);
          if (a.listed) a.listed[g] = v;
        }
        const int32_t c = d < f ? d : f;
        if (cnt) cnt[g] = c;
        if (a.topo_hot && c > 0) atomicAdd(&a.topo_hot[v], uint32_t(c));
      }
    }
  }
}

// Lanes of a vertex: as many as samples, but a power of two of them where rows cross PCIe.  The link bounds the hop there, and
// lanes packed without gaps cost it up to 4 %.  Calls, packed / power of two: 4096 seeds of 8 M vertices 9, 9 169.5 / 162.4 us,
// 11, 11 185.9 / 180.7, 5, 5 116.6 / 113.5, 20, 20 236.3 / 237.0; 8192 seeds (15, 10, 5) of 2.4 M 931 / 915, with half of the
// topology cached 504 / 499 (where the cached half serves most rows 275.7 / 276.9).
inline int32_t hop_lanes(const TopoView& tv, int32_t f) {
  if (!tv.over_pcie) return f;
  int32_t lanes = 1;
  while (lanes < f) lanes *= 2;
  return lanes;
}

// Workgroups for a hop over at most `cap` vertices.
// Six workgroups (24 waves) per CU: more waves do not make scattered marks faster.  Calls at 4 / 6 / 8 per CU: 2.4 M
// vertices, half of the topology over PCIe 279.9 / 276.3 / 276.4 us; marking bits, as the pipeline inside a batch and calls of few
// samples do (calls like these two are binned), 111 M vertices 67.7 / 64.8 / 67.0, 250 M 63.3 / 61.7 / 63.4; sampling server step at 2.4 M 194.6 / 189.9 / 192.6.  Sampling a batch beside the extraction of the one before, 2.4 M
// vertices, at 4 / 6: half of the topology and 30 % of the features cached 1869 / 1870 us a step, half and 90 % 574 / 575,
// everything 148.7 / 145.0.
inline uint32_t hop_blocks(const DeviceInfo& di, int64_t cap, int32_t lanes) {
  const int64_t per_block = 4 * (64 / lanes), full = int64_t(di.num_cus) * 6;       // vertices of a workgroup pass
  const int64_t blocks = (cap + per_block - 1) / per_block;
  return uint32_t(blocks > full ? full : blocks < 1 ? 1 : blocks);
}

}  // namespace
}  // namespace lgp
