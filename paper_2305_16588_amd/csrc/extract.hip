// The pipeline inside one mini-batch (Sec. 5): while a hop is sampled, the rows of the vertices that the hop before it
// reached are extracted beside it, in the same launch.  On two streams every group of rows cost an event and a wait
// between them (10-25 us each).  8192 seeds (15, 10, 5) on 2.4 M vertices, 400-byte rows, all cached: 181 -> 146 us a call (sampling
// takes 60 of that and extraction 80 by themselves: both are bound by requests to HBM); 64 seeds (15, 10) 76 -> 24; 8000 seeds
// (15, 10) on 1 M vertices in CPU memory, a fifth cached 871 -> 839; 128-byte rows of which 95 % are cached 196 -> 168.
#include "gather_dev.hpp"
#include "sampler_dev.hpp"

#include <type_traits>

namespace lgp {
namespace {

// Misses first: they need the link for the whole time; then the hop, whose chains of loads are the longest, then the hits.
// Hits as wide as beside misses only: at 2 / 3 / 4 / 6 workgroups per CU the first call above takes 175 / 159 / 151 / 145 us; hop
// and hits in turn 148.
template <int SHIFT, typename VecT, bool RAGGED>
__global__ __launch_bounds__(256) void hop_and_rows_kernel(HopArgs h, SplitArgs a, uint32_t hop_groups) {
  if (blockIdx.x < a.miss_blocks) split_misses<VecT, RAGGED>(a, blockIdx.x);
  else if (blockIdx.x < a.miss_blocks + hop_groups) sample_hop<SHIFT>(h, blockIdx.x - a.miss_blocks, hop_groups);
  else split_hits<HitWalk::kGroups>(a, blockIdx.x - a.miss_blocks - hop_groups, a.hit_blocks);
}

__global__ __launch_bounds__(64) void sum_counters_kernel(const int32_t* __restrict__ seg_counters, int32_t n_seg,
                                                          int32_t* __restrict__ stats) {
  if (threadIdx.x >= 2) return;
  int32_t sum = 0;
  for (int32_t k = 0; k < n_seg; ++k) sum += seg_counters[3 * k + threadIdx.x];
  stats[threadIdx.x] = sum;
}

__global__ __launch_bounds__(256) void clear_map_kernel(uint64_t* __restrict__ map, int64_t words) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  for (int64_t k = t * 2; k < words; k += int64_t(gridDim.x) * 512)       // a map has a multiple of 2048 words
    *reinterpret_cast<ulonglong2*>(map + k) = make_ulonglong2(0, 0);
}

}  // namespace

void launch_hop_and_rows(const DeviceInfo& di, const TopoView& tv, const int32_t* frontier, int32_t* n_frontier, int64_t cap,
                         int32_t fanout, int32_t hop, uint64_t rng_seed, int32_t* nbr, int32_t* cnt, uint32_t* mark_bits,
                         uint32_t* self_bits, uint32_t* d_err, uint64_t* status, int64_t n_status, const RowSources& r,
                         const void* hit_src, const void* miss_src, void* dst, int64_t row_bytes, hipStream_t s,
                         const FirstGroup& first) {
  HopArgs h{tv,  frontier, n_frontier, cap,       fanout,  hop_lanes(tv, fanout), hop,    uint32_t(rng_seed), uint32_t(rng_seed >> 32),
                  nbr, cnt,      mark_bits,  self_bits, nullptr, d_err,                 status, int32_t(n_status)};
  h.listed = first.listed;
  h.seg = first.seg;
  h.zeroed = first.zeroed;
  h.n_zeroed = first.n_zeroed;
  SplitArgs a;
  const int width = split_args(di, r, hit_src, miss_src, dst, row_bytes, &a);
  const uint32_t hop_groups = hop_blocks(di, cap, h.lanes);
  const dim3 grid{a.miss_blocks + hop_groups + a.hit_blocks}, block{256};
  auto launch = [&](auto shift, auto vec, auto ragged) {
    hipLaunchKernelGGL((hop_and_rows_kernel<decltype(shift)::value, decltype(vec), decltype(ragged)::value>), grid, block, 0, s,
                       h, a, hop_groups);
  };
  auto with_marks = [&](auto shift) {
    if (width == 16) launch(shift, u32x4{}, std::true_type{});
    else if (width == 8) launch(shift, u32x2{}, std::false_type{});
    else launch(shift, uint32_t{}, std::false_type{});
  };
  switch (di.spread_shift) {
    case 0: with_marks(std::integral_constant<int, 0>{}); break;
    case 3: with_marks(std::integral_constant<int, 3>{}); break;
    case 4: with_marks(std::integral_constant<int, 4>{}); break;
    default: with_marks(std::integral_constant<int, 5>{}); break;
  }
}

void launch_sum_counters(const int32_t* seg_counters, int32_t n_seg, int32_t* stats, hipStream_t s) {
  hipLaunchKernelGGL(sum_counters_kernel, dim3(1), dim3(64), 0, s, seg_counters, n_seg, stats);
}

void launch_clear_map(const DeviceInfo& di, uint64_t* map, int64_t words, hipStream_t s) {
  int64_t blocks = (words + 511) / 512;
  if (blocks > di.num_cus * 8) blocks = di.num_cus * 8;
  hipLaunchKernelGGL(clear_map_kernel, dim3(unsigned(blocks)), dim3(256), 0, s, map, words);
}

}  // namespace lgp
