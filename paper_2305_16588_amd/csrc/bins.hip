// Dedup of a large graph's samples without a map in HBM (see BinMaps).  The hop has sorted its samples by ranges of vertices
// (bins) into segments of one workgroup each; here a workgroup takes one bin, sets a bit per sample in LDS, counts the bits,
// learns from the workgroups before it where its ids begin, and writes them at their ranks.  Each sample is one read of four
// bytes, and nothing has to be cleared for the next call.
//
// What bounds it: a chain of latencies (segments, LDS, status words of the bins before, ids), not bytes.  Segment heads are at
// fixed places, so that counts and ids arrive in one round trip; the count of a bin comes out of the atomics that set its bits, so
// that it is published before the words are ranked; status words are read from one of eight copies, so that not all workgroups
// ask one channel of memory (8192 seeds (15, 10, 5) of 12 M vertices, 184 bins: one copy 60.2 us a call, two 58.6, eight 57.1,
// sixteen 57.0).  Kernel times, map -> bins: 250 M vertices, 8192 seeds (25, 10), hops 6.6 -> 7.2 and 24.4 -> 13.6 us, lists
// 13.3 -> 7.4 and 13.4 -> 11.0; 111 M, (15, 10, 5), hops 4.8 -> 6.0, 10.5 -> 9.3 and 23.0 -> 11.7, lists 6.6 -> 5.3, 7.6 -> 6.8
// and 8.4 -> 9.9.
// Built and left: ids gathered in a list in LDS and ranked through their group's words (union 11.4 us at 111 M, and the list has
// an end).
//
// Waiting works as in compact.hip: a workgroup publishes its count before it looks for the others', and one that has looked for a
// long time without an answer counts that bin itself, so no wait depends on when another workgroup is scheduled.  The segments are
// only read, so a recount sees what the owner saw; marks that did not fit a segment (spilled, in the map in HBM) are cleared by the
// owner after its status has reached memory, and the status is looked at again after they were read.
#include "common.hpp"

#include <algorithm>

namespace lgp {
namespace {

constexpr int kWaves = kBinThreads / 64;
constexpr uint32_t kPublished = 1u << 31;                   // a bin has at most 2^20 ids
constexpr int kHeads = kBinWriters / (kBinThreads / 4);     // segment heads of a thread: four lanes take one, 16 bytes each

// Sum of the lanes up to the calling one.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return x;
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
  return uint32_t(__builtin_amdgcn_readlane(int(wave_inclusive_scan(x)), 63));
}
template <typename T>
__device__ __forceinline__ T agent_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kHeldSeeds = 8 * kBinThreads;                 // seeds that are loaded ahead
constexpr int kInner = 2;                                   // inner frontiers of which a thread's first id is loaded ahead
typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));

template <int B>
struct Lds {
  // The bits: 1 << B of them.  A thread ranks a span of up to 256; spans of 256 lie in halves, the first halves of all of them
  // before the second halves, so that a wave reads either without gaps.
  static constexpr int kSpan = B >= 18 ? 256 : 1 << (B - 10);   // 17: all threads take part (256 bits each: 17 M 44.7 -> 42.8 us a call)
  uint4 bits[1 << (B - 7)];
  uint32_t wave_count[64], wave_ahead[kWaves];
  uint64_t late[kMaxBins / 64];
  uint32_t again, total, late_any;
};

// What is listed: the samples (kList), their union with the seeds and the inner frontiers (kUnion), or first one, then the other.
enum Mode { kList = 1, kUnion = 2, kBoth = 3 };

template <int B>
struct Lister {
  static constexpr int kSpan = Lds<B>::kSpan, kSpans = (1 << B) / kSpan, kPasses = kSpans / kBinThreads;   // spans of a thread
  static constexpr int kWords = kSpan / 64;
  static_assert(kWords >= 1 && kPasses * kWaves <= 64, "one lane per wave and pass");
  const BinArgs a;                                           // by value: by reference the compiler keeps the arguments in scratch memory
  Lds<B>& m;
  uint32_t fresh;                                            // bits set by this thread and not yet counted
  uint64_t word[kPasses][kWords];                            // the bits of this thread's spans
  uint32_t rank[kPasses];                                    // ids of the bin before them
  const int t = threadIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

  __device__ __forceinline__ void clear() const {
    for (int k = t; k < 1 << (B - 7); k += kBinThreads) m.bits[k] = make_uint4(0, 0, 0, 0);
  }
  __device__ __forceinline__ void set(uint32_t x) {
    const uint32_t o = x & ((1u << B) - 1u);
    const uint32_t chunk = kSpan == 256 ? (o >> 8) + ((o >> 7) & 1u) * uint32_t(kSpans) : o >> 7;
    const uint32_t old = atomicOr(reinterpret_cast<uint32_t*>(&m.bits[chunk]) + ((o >> 5) & 3u), 1u << (o & 31u));
    fresh += 1u - ((old >> (o & 31u)) & 1u);
  }
  // Whether a seed is a member of the bin; one whose offsets make no sense is no member of the batch (the hop has reported it).
  __device__ __forceinline__ bool seed_counts(uint32_t bin, int32_t v) const {
    if (uint32_t(v) >> B != bin || v >= a.tv.num_vertices) return false;
    if ((uint32_t(a.tv.row_tab[v]) & kRowDegOverflow) != kRowDegOverflow) return true;
    const int64_t d = a.tv.indptr_bytes == 8
        ? static_cast<const int64_t*>(a.tv.h_indptr)[int64_t(v) + 1] - static_cast<const int64_t*>(a.tv.h_indptr)[v]
        : int64_t(static_cast<const int32_t*>(a.tv.h_indptr)[int64_t(v) + 1]) - static_cast<const int32_t*>(a.tv.h_indptr)[v];
    return d >= 0 && d <= 0x7fffffff;
  }
  // Sample words k, k + 1, .. of a lane's four that the segment's count says are there.
  __device__ __forceinline__ void set_four(const uint4& v, uint32_t k, uint32_t used) {
    if (k <= used && k != 0) set(v.x);                       // word 0 is the count
    if (k + 1 <= used) set(v.y);
    if (k + 2 <= used) set(v.z);
    if (k + 3 <= used) set(v.w);
  }
  __device__ __forceinline__ uint32_t segment(uint32_t bin, int l) const {      // four lanes take a segment
    return bin * uint32_t(a.writers) + uint32_t(t >> 2) + uint32_t(l) * (kBinThreads / 4);
  }
  __device__ __forceinline__ void load_heads(uint32_t bin, uint4 (&v)[kHeads]) const {
#pragma unroll
    for (int l = 0; l < kHeads; ++l) {
      v[l] = make_uint4(0, 0, 0, 0);
      if ((t >> 2) + l * (kBinThreads / 4) < a.writers)
        v[l] = reinterpret_cast<const uint4*>(a.maps.heads)[segment(bin, l) * (kHeadWords / 4) + (t & 3)];
    }
  }
  __device__ __forceinline__ void set_samples(uint32_t bin, const uint4 (&v)[kHeads], bool spilled) {
    const uint32_t k = uint32_t(t & 3) * 4;
    uint32_t used[kHeads];
#pragma unroll
    for (int l = 0; l < kHeads; ++l) {
      used[l] = uint32_t(__builtin_amdgcn_update_dpp(0, int(v[l].x), 0x00, 0xf, 0xf, false));   // of the quad's first lane
      set_four(v[l], k, used[l]);
    }
#pragma unroll
    for (int l = 0; l < kHeads; ++l) {                       // tails are rare
      if (used[l] >= uint32_t(kBinWords)) used[l] = kBinWords - 1;
#pragma unroll 1
      for (uint32_t o = kHeadWords; o <= used[l]; o += kHeadWords)
        set_four(reinterpret_cast<const uint4*>(a.maps.tails)[segment(bin, l) * ((kBinWords - kHeadWords) / 4) +
                                                              (o - kHeadWords) / 4 + (t & 3)],
                 o + k, used[l]);
    }
    if (!spilled) return;
    const uint64_t* marks = a.spill + (size_t(bin) << (B - 6));
#pragma unroll 1
    for (int j = t; j < 1 << (B - 6); j += kBinThreads) {
#pragma unroll 1
      for (uint64_t x = agent_load(marks + j); x; x &= x - 1) set(uint32_t(j) * 64u + uint32_t(__ffsll((unsigned long long)x) - 1));
    }
  }
  __device__ __forceinline__ void set_seed(uint32_t bin, int32_t v) {
    if (uint32_t(v) >> B == bin && v < a.tv.num_vertices) set(uint32_t(v));
  }
  __device__ __forceinline__ void set_seeds(uint32_t bin, i32x4_any v) {
    set_seed(bin, v.x);
    set_seed(bin, v.y);
    set_seed(bin, v.z);
    set_seed(bin, v.w);
  }
  // The seeds from number `from` (a multiple of four) on, and the bin's share of the inner frontiers but for the first `held` ids of
  // kInner of them.
  __device__ __forceinline__ void set_earlier(uint32_t bin, int32_t from, int32_t held, bool odd_rows) {
    if (!odd_rows) {
      constexpr int kLoads = 4;
#pragma unroll 1
      for (; from + 3 < a.n_seeds; from += 4 * kLoads * kBinThreads) {
        i32x4_any v[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
          const int32_t i = from + 4 * (t + u * kBinThreads);
          v[u] = -1;
          if (i + 3 < a.n_seeds) v[u] = *reinterpret_cast<const i32x4_any*>(a.seeds + i);
        }
#pragma unroll
        for (int u = 0; u < kLoads; ++u) set_seeds(bin, v[u]);
      }
      from = a.n_seeds / 4 * 4;
    }
#pragma unroll 1
    for (int32_t i = from + t; i < a.n_seeds; i += kBinThreads)
      if (seed_counts(bin, a.seeds[i])) set(uint32_t(a.seeds[i]));
#pragma unroll                                               // an index that is no constant would put the arguments in scratch memory
    for (int h = 1; h < LGP_MAX_HOPS; ++h) {
      if (h > a.inner) break;
      const int32_t* first = a.first + h * (kMaxBins + 1) + bin;
      const int32_t end = first[1];
#pragma unroll 1
      for (int32_t i = first[0] + (h <= kInner ? held : 0) + t; i < end; i += kBinThreads) set(uint32_t(a.frontier[h][i]));
    }
  }
  // Takes this thread's words and ranks them; returns the number of ids.
  __device__ __forceinline__ uint32_t count() {
    uint32_t c[kPasses], up_to[kPasses];
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const int g = p * kBinThreads + t;
      if constexpr (kSpan >= 128) {
        const uint4 x = m.bits[g];
        word[p][0] = x.x | uint64_t(x.y) << 32;
        word[p][1] = x.z | uint64_t(x.w) << 32;
        if constexpr (kSpan == 256) {
          const uint4 y = m.bits[g + kSpans];
          word[p][2] = y.x | uint64_t(y.y) << 32;
          word[p][3] = y.z | uint64_t(y.w) << 32;
        }
      } else {
        word[p][0] = reinterpret_cast<const uint64_t*>(m.bits)[g];
      }
      c[p] = 0;
#pragma unroll
      for (int w = 0; w < kWords; ++w) c[p] += uint32_t(__popcll(word[p][w]));
      up_to[p] = wave_inclusive_scan(c[p]);
      if (lane == 63) m.wave_count[p * kWaves + wave] = up_to[p];
    }
    __syncthreads();
    const uint32_t own = lane < kPasses * kWaves ? m.wave_count[lane] : 0, sums = wave_inclusive_scan(own);
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const uint32_t ahead = uint32_t(__builtin_amdgcn_readlane(int(sums - own), __builtin_amdgcn_readfirstlane(p * kWaves + wave)));
      rank[p] = ahead + up_to[p] - c[p];
    }
    return uint32_t(__builtin_amdgcn_readlane(int(sums), 63));
  }
  // Ids of all bins before this one, once it has published its own; early: what the status of bin t was when last looked at.
  __device__ __forceinline__ uint32_t place(uint32_t bin, const uint32_t* status, uint32_t early, bool with_earlier) {
    uint32_t ahead = early & ~kPublished;
    bool late = uint32_t(t) < bin && !(early & kPublished);
#pragma unroll 1
    for (int it = 0; late && it < a.polls; ++it) {
      const uint32_t s = agent_load(&status[t]);
      if (s & kPublished) {
        ahead = s & ~kPublished;
        late = false;
      } else {
        __builtin_amdgcn_s_sleep(2);
      }
    }
    if (t < kStatusCopies) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // published before any spilled mark is cleared
    const uint64_t mask = __ballot(late);
    const uint32_t sum = wave_sum(ahead);
    if (lane == 0) {
      if (wave < kMaxBins / 64) m.late[wave] = mask;
      if (mask) m.late_any = 1;
      m.wave_ahead[wave] = sum;
    }
    __syncthreads();
    ahead = wave_sum(lane < kWaves ? m.wave_ahead[lane] : 0);
    if (__builtin_expect(m.late_any, 0)) {
#pragma unroll 1
      for (uint32_t k = 0; k <= bin; ++k) {                  // the bins whose counts are late, and then this one again
        if (k < bin && !((m.late[k >> 6] >> (k & 63u)) & 1ull)) continue;
        uint4 v[kHeads];
        load_heads(k, v);
        const bool spilled = agent_load(&a.maps.spilled[k]) != 0;
        __syncthreads();
        clear();
        __syncthreads();
        set_samples(k, v, spilled);
        if (with_earlier) set_earlier(k, 0, 0, true);
        __syncthreads();
        const uint32_t counted = count();
        if (t == 0) m.again = agent_load(&status[k]);
        __syncthreads();
        if (k < bin) ahead += (m.again & kPublished) ? m.again & ~kPublished : counted;
      }
      fresh = 0;
    }
    return ahead;
  }
  // Writes the bin's ids, once their bits are set.
  __device__ __forceinline__ void write(uint32_t bin, bool with_earlier, uint32_t* status, int32_t* out, int64_t out_cap,
                                        int32_t* n_out, int32_t* first) {
    const uint32_t own = wave_sum(fresh), cap = uint32_t(out_cap);
    fresh = 0;
    if (lane == 0 && own) atomicAdd(&m.total, own);
    __syncthreads();                                         // all bits are set
    const uint32_t n = m.total;
    if (t < kStatusCopies) __hip_atomic_store(&status[t * kMaxBins + bin], n | kPublished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    count();                                                 // while the status words travel
    const uint32_t* const others = status + bin % kStatusCopies * kMaxBins;
    const uint32_t early = uint32_t(t) < bin ? agent_load(&others[t]) : 0;
    const uint32_t at = place(bin, others, early, with_earlier), end = at + n;
#pragma unroll
    for (int p = 0; p < kPasses; ++p) {
      const uint32_t id0 = (bin << B) + uint32_t(p * kBinThreads + t) * uint32_t(kSpan);
      uint32_t k = at + rank[p];
#pragma unroll
      for (int w = 0; w < kWords; ++w) {
#pragma unroll 1
        for (uint64_t x = word[p][w]; x; x &= x - 1, ++k)
          if (k < cap) out[k] = int32_t(id0 + uint32_t(w) * 64u + uint32_t(__ffsll((unsigned long long)x) - 1));
      }
    }
    if (t != 0) return;
    if (first) first[bin] = int32_t(at < cap ? at : cap);
    if (bin + 1 != gridDim.x) return;
    if (first) first[bin + 1] = int32_t(end < cap ? end : cap);
    *n_out = int32_t(end < cap ? end : cap);
    if (end > cap) atomicOr(a.d_err, ERR_OVERRUN);
  }
};

template <int B, int M>
__global__ __launch_bounds__(kBinThreads) void list_bins_kernel(BinArgs a) {
  __shared__ Lds<B> lds;
  Lister<B> l{a, lds};
  const uint32_t bin = blockIdx.x;
  const int t = l.t;
  if (t == 0) lds.total = lds.late_any = 0;
  l.fresh = 0;
  // All loads are under way before the first one is waited for, but for those of ids whose place is loaded.
  uint4 heads[kHeads];
  constexpr int kSeedLoads = kHeldSeeds / (4 * kBinThreads);
  i32x4_any seeds[kSeedLoads];
  int32_t inner[kInner], held_seeds = 0;
  bool odd_rows = false;
  l.load_heads(bin, heads);
  const bool spilled = agent_load(&a.maps.spilled[bin]) != 0;
  if (M & kUnion) {
    odd_rows = a.maps.spilled[kMaxBins] == a.maps.call;    // set by the hops, so all threads see the same
    const int32_t whole = odd_rows ? 0 : (a.n_seeds < kHeldSeeds ? a.n_seeds : kHeldSeeds) / 4;
    held_seeds = whole * 4;
#pragma unroll
    for (int k = 0; k < kSeedLoads; ++k) {
      seeds[k] = -1;
      if (t + k * kBinThreads < whole) seeds[k] = reinterpret_cast<const i32x4_any*>(a.seeds)[t + k * kBinThreads];
    }
#pragma unroll
    for (int h = 0; h < kInner; ++h) {
      inner[h] = -1;
      if (h >= a.inner) continue;
      const int32_t* first = a.first + (h + 1) * (kMaxBins + 1) + bin;
      const int32_t i = first[0] + t;
      if (i < first[1]) inner[h] = a.frontier[h + 1][i];
    }
  }
  l.clear();
  __syncthreads();
  l.set_samples(bin, heads, spilled);
  if (M & kList) {
    l.write(bin, false, a.status, a.list, a.list_cap, a.n_list, a.list_first);
    if (M == kBoth) __syncthreads();                         // the count of the samples has been read
  }
  if (M & kUnion) {
#pragma unroll
    for (int k = 0; k < kSeedLoads; ++k) l.set_seeds(bin, seeds[k]);
#pragma unroll
    for (int h = 0; h < kInner; ++h)
      if (inner[h] >= 0) l.set(uint32_t(inner[h]));
    l.set_earlier(bin, held_seeds, kBinThreads, odd_rows);
    l.write(bin, true, a.status + kStatusCopies * kMaxBins, a.all, a.all_cap, a.n_all, nullptr);
  }
  if (!spilled) return;
  uint64_t* marks = a.spill + (size_t(bin) << (B - 6));
  for (int k = t; k < 1 << (B - 6); k += kBinThreads) marks[k] = 0;
  if (t == 0) a.maps.spilled[bin] = 0;
}

template <int M>
void launch_mode(const BinArgs& a, hipStream_t s) {
  const dim3 grid{unsigned(a.maps.bins)}, block{unsigned(kBinThreads)};
  switch (a.maps.shift) {
    case 16: hipLaunchKernelGGL((list_bins_kernel<16, M>), grid, block, 0, s, a); break;
    case 17: hipLaunchKernelGGL((list_bins_kernel<17, M>), grid, block, 0, s, a); break;
    case 18: hipLaunchKernelGGL((list_bins_kernel<18, M>), grid, block, 0, s, a); break;
    case 19: hipLaunchKernelGGL((list_bins_kernel<19, M>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((list_bins_kernel<20, M>), grid, block, 0, s, a); break;
  }
}

}  // namespace

void launch_list_bins(const BinArgs& a, hipStream_t s) {
  BinArgs b = a;
  b.list_cap = std::min<int64_t>(a.list_cap, INT32_MAX);     // as for a compaction: a list holds fewer than 2^31 ids
  b.all_cap = std::min<int64_t>(a.all_cap, INT32_MAX);
  if (!a.n_all) launch_mode<kList>(b, s);
  else if (!a.n_list) launch_mode<kUnion>(b, s);
  else launch_mode<kBoth>(b, s);
}

}  // namespace lgp
