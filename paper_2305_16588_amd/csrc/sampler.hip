// Neighbour sampler (Sec. 2.2 step 2; Sec. 5 "neighbor sampler") for gfx950.
//
// A wave takes 64 / fanout frontier vertices, `fanout` lanes each (see hop_lanes); a lane is a sample
// slot.  One load of the HBM row table gives the row's offset and degree and says
// whether its column ids sit in the HBM topology cache or in the CPU-resident CSR (read
// in place over PCIe), so an uncached vertex costs one PCIe round trip, not two.  All slots draw their
// Philox number at once, and Floyd's sequential "already taken?" test becomes one that needs
// no order (floyd_moves).  What bounds the kernel stands at sample_hop, the width of its grid at
// hop_blocks.
#include "sampler_dev.hpp"

#include <algorithm>

namespace lgp {
namespace {

template <int SHIFT>
__global__ __launch_bounds__(256) void sample_hop_kernel(HopArgs a) {
  sample_hop<SHIFT>(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(kBinThreads, 8) void sample_hop_binned_kernel(HopArgs a) {
  __shared__ uint32_t used[kMaxBins];
  if (threadIdx.x < kMaxBins) used[threadIdx.x] = 0;
  __syncthreads();
  sample_hop<kBinned, kBinThreads / 64>(a, blockIdx.x, gridDim.x, used);
  __syncthreads();
  if (int(threadIdx.x) < a.bins.bins)
    a.bins.heads[(threadIdx.x * gridDim.x + blockIdx.x) * uint32_t(kHeadWords)] = used[threadIdx.x];
}

// Pre-sampling reads rows of a few column ids at random places of CPU memory, a 128-byte line of the link each (340 M
// lines/s = 43.5 GB/s when every line stands alone), and comes back to the same rows batch after batch; all column ids in
// order cross the link at 57 GB/s, once.  16 batches of 8192 seeds (15, 10, 5) on 2.4 M vertices and 62 M edges:
// 0.79 ms a batch over PCIe, 4.4 ms for the copy and 0.08 ms a batch from HBM; the call with the vectors' copy to the host
// 16.1 -> 6.8 ms, 8 batches of 4555 seeds (11, 11, 11) on 0.87 M vertices and 30 M edges 5.6 -> 3.2.
// 64 workgroups keep the link full (57.5 GB/s; 55.5 at 1024).
constexpr int kStageGroups = 64;
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
__global__ __launch_bounds__(256) void stage_topology_kernel(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                                             int64_t n) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x, threads = int64_t(gridDim.x) * 256;
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

}  // namespace

void launch_stage_topology(const int32_t* h_indices, int32_t* staged, int64_t n_edges, hipStream_t s) {
  hipLaunchKernelGGL(stage_topology_kernel, dim3(kStageGroups), dim3(256), 0, s, h_indices, staged, n_edges);
}

void launch_sample_hop(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier,
                       int64_t cap, int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt,
                       uint32_t* mark_bits, uint32_t* self_bits, uint32_t* topo_hot, uint32_t* d_err, uint64_t* status,
                       int64_t n_status, hipStream_t s, const FirstGroup& first) {
  HopArgs a{tv,  frontier, n_frontier, cap,       fanout,   hop_lanes(tv, fanout), hop,    uint32_t(rng_seed), uint32_t(rng_seed >> 32),
                  nbr, cnt,      mark_bits,  self_bits, topo_hot, d_err,                 status, int32_t(n_status)};
  a.listed = first.listed;
  a.seg = first.seg;
  a.zeroed = first.zeroed;
  a.n_zeroed = first.n_zeroed;
  const dim3 grid{hop_blocks(di, cap, a.lanes)}, block{256};
  switch (di.spread_shift) {
    case 0: hipLaunchKernelGGL((sample_hop_kernel<0>), grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL((sample_hop_kernel<3>), grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL((sample_hop_kernel<4>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((sample_hop_kernel<5>), grid, block, 0, s, a); break;
  }
}

int32_t launch_sample_hop_binned(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier,
                                 int64_t cap, int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt,
                                 const BinMaps& m, int32_t writers, uint32_t* mark_bits, uint32_t* d_err, uint64_t* status, hipStream_t s) {
  const HopArgs a{tv,  frontier, n_frontier, cap,     fanout,  hop_lanes(tv, fanout), hop,    uint32_t(rng_seed), uint32_t(rng_seed >> 32),
                  nbr, cnt,      mark_bits,  nullptr, nullptr, d_err,                 status, kBinStatusWords / 2, m};
  const int64_t per_block = kBinThreads / 64 * (64 / a.lanes), blocks = (cap + per_block - 1) / per_block;
  writers = int32_t(std::max<int64_t>(1, std::min<int64_t>(blocks, writers)));
  hipLaunchKernelGGL(sample_hop_binned_kernel, dim3(unsigned(writers)), dim3(unsigned(kBinThreads)), 0, s, a);
  return writers;
}

}  // namespace lgp
