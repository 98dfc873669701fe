// Neighbour sampler (Sec. 2.2 step 2; Sec. 5 "neighbor sampler") for gfx950.
//
// A wave takes 64 / fanout frontier vertices, `fanout` lanes each; a lane is a sample
// slot.  One load of the HBM row table gives the row's offset and degree and says
// whether its column ids sit in the HBM topology cache or in the CPU-resident CSR (read
// in place over PCIe), so an uncached vertex costs one PCIe round trip, not two.  All slots draw their
// Philox number at once, and Floyd's sequential "already taken?" test becomes one that needs
// no order (floyd_moves).  The kernel is bound by dependent loads and, on large graphs, by the bitmap
// atomics, not by issue slots, so the grid is capped at six workgroups per CU (see launch_one).
#include "common.hpp"
#include "philox_dev.hpp"

#include <type_traits>

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

// Marks bound this kernel (last hop of 190 k vertices x 5 at 2.4 M vertices: 23 us with its 950 k byte marks, 11 without;
// 490 k atomic marks at 250 M: 24 and 9); what is left is loads and issue slots, so lanes are packed without gaps.  Against
// a power of two of lanes per vertex and a chain of fanout - 1 broadcasts for Floyd's test, calls on 2.4 M vertices from
// 8192 seeds: fan-outs 17, 17 28.2 -> 25.1 us, 64 17.5 -> 15.4, 9, 9 21.2 -> 20.2, 15, 10, 5 with blocks and gather
// 190 -> 186; 25 or 3, 3, 3 and graphs with atomic marks are level.
template <typename IdxT, int SHIFT>
__global__ __launch_bounds__(256) void sample_hop_kernel(
    const uint64_t* __restrict__ row_tab, const IdxT* __restrict__ h_indptr, const int32_t* __restrict__ h_indices,
    const int32_t* __restrict__ t_indices, int64_t num_vertices,
    const int32_t* __restrict__ frontier, int32_t* __restrict__ n_frontier, int64_t cap, int32_t f, int32_t hop,
    uint32_t k0, uint32_t k1, int32_t* __restrict__ nbr, int32_t* __restrict__ cnt, uint32_t* __restrict__ mark_bits,
    uint32_t* __restrict__ self_bits, uint32_t* __restrict__ topo_hot, uint32_t* __restrict__ d_err,
    uint64_t* __restrict__ status, int n_status, const int32_t* __restrict__ staged,
    const uint64_t* __restrict__ use_staged) {
  // self_bits != nullptr: this is the first hop; the frontier is the caller's seed list of `cap`
  // ids, whose size is published here and whose members are marked in the gather set.
  if (self_bits && blockIdx.x == 0 && threadIdx.x == 0) *n_frontier = int32_t(cap);
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < n_status; k += 256) status[k] = 0;
  if (use_staged && *use_staged) h_indices = staged;
  int64_t n = self_bits ? cap : int64_t(*n_frontier);
  if (n > cap) n = cap;                           // never trust a count beyond the buffer
  const int per_wave = 64 / f;                    // vertices per wave pass
  const int lane = threadIdx.x & 63;
  const int sub = lane / f, slot = lane - sub * f;   // vertex of this lane in the pass, sample slot
  // Three loads depend on one another (frontier id -> row-table entry -> column id).  The id is loaded two passes ahead
  // and the row-table entry one pass ahead, so that a pass waits for its column ids only (two hops of 17 from 8192 seeds
  // of 2.4 M vertices 25.8 -> 25.1 us, one hop of 64 16.0 -> 15.4).
  const int64_t wave = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int64_t stride = int64_t(gridDim.x) * 4 * per_wave;
  const uint64_t nv = uint64_t(num_vertices);
  auto id_at = [&](int64_t g) { return sub < per_wave && g < n ? frontier[g] : -1; };
  auto row_of = [&](int32_t v) { return uint32_t(v) < nv ? row_tab[v] : 0; };
  int64_t g0 = wave * per_wave;
  int32_t v_next = id_at(g0 + sub), v_after = id_at(g0 + stride + sub);
  uint64_t e_next = row_of(v_next);
  for (; g0 < n; g0 += stride) {
    const int64_t g = g0 + sub;
    const bool active = sub < per_wave && g < n;
    const int32_t v = v_next;
    const uint64_t e = e_next;
    v_next = v_after;
    v_after = id_at(g + 2 * stride);
    e_next = row_of(v_next);
    bool bad = active && uint32_t(v) >= nv;
    int64_t s = 0, d64 = 0;
    const int32_t* colbase = h_indices;
    if (active && !bad) {
      const uint32_t d24 = uint32_t(e) & kRowDegOverflow;
      if (d24 != kRowDegOverflow) {
        s = int64_t((e >> kRowStartShift) & kRowStartMask);
        d64 = d24;
        if (e & kRowCachedBit) colbase = t_indices;
      } else {                                     // degree does not fit the entry: CPU-resident CSR
        s = int64_t(h_indptr[v]);
        d64 = int64_t(h_indptr[int64_t(v) + 1]) - s;
      }
      if (d64 < 0 || d64 > 0x7fffffff) { bad = true; d64 = 0; }
    }
    if (bad) {
      if (slot == 0) atomicOr(d_err, ERR_BAD_ID);
      d64 = 0;
    }
    const int32_t d = int32_t(d64);
    const bool big = active && d > f;
    int32_t p = slot;                              // position inside the row
    if (__any(big)) {
      const int32_t j = d - f + slot;
      const int32_t t = int32_t(
          __umul64hi(philox_draw64(k0, k1, uint32_t(v), uint32_t(hop), uint32_t(slot)), uint64_t(uint32_t(j)) + 1));
      const bool moves = floyd_moves(big, t, d, f, slot, lane - slot);
      if (big) p = moves ? j : t;
    }
    if (active) {
      int32_t u = -1;
      if (big || slot < d) {
        u = colbase[s + p];
        if (uint32_t(u) >= nv) {
          atomicOr(d_err, ERR_BAD_ID);
          u = -1;
        } else {
          mark_vertex<SHIFT>(mark_bits, u);
        }
      }
      if (nbr) nbr[g0 * f + lane] = u;
      if (slot == 0) {
        if (self_bits && !bad) mark_vertex<SHIFT>(self_bits, v);
        const int32_t c = d < f ? d : f;
        if (cnt) cnt[g] = c;
        if (topo_hot && c > 0) atomicAdd(&topo_hot[v], uint32_t(c));
      }
    }
  }
}

// Pre-sampling reads rows of a few column ids at random places of CPU memory, a 128-byte line of the link each (340 M
// lines/s = 43.5 GB/s when every line stands alone), and comes back to the same rows batch after batch; all column ids in
// order cross the link at 57 GB/s, once.  The first batch tells how many rows a batch reads, so the choice is made here on
// the device, without the host waiting for the count.  16 batches of 8192 seeds (15, 10, 5) on 2.4 M vertices and 62 M edges:
// 0.79 ms a batch over PCIe, 4.4 ms for the copy and 0.08 ms a batch from HBM; the call with the vectors' copy to the host
// 15.8 -> 8.5 ms, 8 batches of 4555 seeds (11, 11, 11) on 0.87 M vertices and 30 M edges 5.6 -> 3.7.
// 64 workgroups keep the link full (57.5 GB/s; 55.5 at 1024).
constexpr int kStageGroups = 64;
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void stage_topology_kernel(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                                             int64_t n, const unsigned long long* __restrict__ rows,
                                                             int64_t remaining, uint64_t* __restrict__ use_staged) {
  constexpr uint64_t kIdsPerLine = 128 / sizeof(int32_t);
  if (*rows * uint64_t(remaining) <= uint64_t(n) / kIdsPerLine) return;
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x, threads = int64_t(gridDim.x) * 256;
  if (t == 0) *use_staged = 1;
  // whole 16-byte chunks from the first aligned id on; fewer than four ids are left over at either end
  const int64_t head = int64_t((0 - (uintptr_t(src) >> 2)) & 3) < n ? int64_t((0 - (uintptr_t(src) >> 2)) & 3) : n;
  const int64_t chunks = (n - head) / 4, tail = head + chunks * 4;
  if (t < head) dst[t] = src[t];
  if (t < n - tail) dst[tail + t] = src[tail + t];
  const i32x4* from = reinterpret_cast<const i32x4*>(src + head);
  i32x4* to = reinterpret_cast<i32x4*>(dst + head);
  constexpr int U = 4;
  for (int64_t k = t; k < chunks; k += threads * U) {
    i32x4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u * threads < chunks) v[u] = __builtin_nontemporal_load(from + k + u * threads);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u * threads < chunks) to[k + u * threads] = v[u];
  }
}

template <typename IdxT, int SHIFT>
void launch_one(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier,
                int64_t cap, int32_t f, int32_t hop, uint64_t seed, int32_t* nbr, int32_t* cnt, uint32_t* mark_bits,
                uint32_t* self_bits, uint32_t* topo_hot, uint32_t* d_err, uint64_t* status, int64_t n_status, hipStream_t s) {
  const int64_t per_block = 4 * (64 / f);         // vertices of a workgroup pass
  int64_t blocks = (cap + per_block - 1) / per_block;
  // Six workgroups (24 waves) per CU: the kernel is bound by scattered marks and dependent loads, not by issue slots.
  // Calls at 4 / 6 / 8 per CU: 2.4 M vertices, half of the topology over PCIe 279.9 / 276.3 / 276.4 us, 111 M vertices
  // 67.7 / 64.8 / 67.0, 250 M 63.3 / 61.7 / 63.4; sampling server step at 2.4 M 194.6 / 189.9 / 192.6.  Sampling a batch
  // beside the extraction of the one before, 2.4 M vertices, at 4 / 6: half of the topology and 30 % of the features
  // cached 1869 / 1870 us a step, half and 90 % 574 / 575, everything 148.7 / 145.0.
  const int64_t full = int64_t(di.num_cus) * 6;
  if (blocks > full) blocks = full;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL((sample_hop_kernel<IdxT, SHIFT>), dim3(unsigned(blocks)), dim3(256), 0, s,
                     tv.row_tab, static_cast<const IdxT*>(tv.h_indptr), tv.h_indices, tv.t_indices,
                     tv.num_vertices, frontier, n_frontier, cap, f, hop, uint32_t(seed), uint32_t(seed >> 32), nbr,
                     cnt, mark_bits, self_bits, topo_hot, d_err, status, int(n_status), tv.staged, tv.use_staged);
}

}  // namespace

void launch_stage_topology(const int32_t* h_indices, int32_t* staged, int64_t n_edges, const unsigned long long* rows,
                           int64_t remaining, uint64_t* use_staged, hipStream_t s) {
  hipLaunchKernelGGL(stage_topology_kernel, dim3(kStageGroups), dim3(256), 0, s, h_indices, staged, n_edges, rows,
                     remaining, use_staged);
}

void launch_sample_hop(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier,
                       int64_t cap, int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt,
                       uint32_t* mark_bits, uint32_t* self_bits, uint32_t* topo_hot, uint32_t* d_err, uint64_t* status, int64_t n_status, hipStream_t s) {
  auto launch = [&](auto idx, auto shift) {
    launch_one<decltype(idx), decltype(shift)::value>(di, tv, frontier, n_frontier, cap, fanout, hop, rng_seed, nbr, cnt,
                                                      mark_bits, self_bits, topo_hot, d_err, status, n_status, s);
  };
  auto with_marks = [&](auto shift) {
    if (tv.indptr_bytes == 8) launch(int64_t{}, shift);
    else launch(int32_t{}, shift);
  };
  switch (di.spread_shift) {
    case 0: with_marks(std::integral_constant<int, 0>{}); break;
    case 3: with_marks(std::integral_constant<int, 3>{}); break;
    case 4: with_marks(std::integral_constant<int, 4>{}); break;
    default: with_marks(std::integral_constant<int, 5>{}); break;
  }
}

}  // namespace lgp
