// Frontier / gather-set dedup (implied by Sec. 4.2.2: each vertex of a mini-batch's
// sample result counts once).  The sampler marks every sampled vertex in a dedup map; this
// file turns the map into the ascending list of marked vertices, which is the sorted-unique
// order without any sort, in one launch per map.
//
// A workgroup owns a contiguous share of the map.  It loads its words once, counts their
// marks, publishes the count in a status word, adds up the counts of all workgroups before
// it (one thread per predecessor, all waits at once, no chain), and writes its ids, clearing
// the map on the way.  A dependent launch costs 3-4.5 us however little it does, which is
// what a counting launch ahead of this one would add, and the map would be read twice.
// Kernel time per compaction, counting launch + writing launch -> this kernel: 2.4 M vertices
// (2.4-MB map) 4.8 + 5.7 -> 5.4 us; 111 M (13.9 MB) 4.1 + 7.8 -> 6.8-8.8 us; 250 M (31 MB)
// 6.2 + 12.0 -> 12.9-13.5 us.  Loading and counting take 4.2 / 6.6 / 8.5 us of that.
//
// Waiting: a workgroup publishes before it waits, so workgroups that run make progress
// together.  One that has polled a predecessor for a long time without an answer (it may be
// queued behind other work on the chip) counts that share itself, looking for the status
// between a few words and the next, so no wait depends on when another workgroup is scheduled.
// The recount is sound because a workgroup clears its words only after its status has reached
// memory: if the status is still missing after the words were read, they were read untouched.
#include "common.hpp"

#include <algorithm>

namespace lgp {
namespace {

constexpr int kWaves = kCompactThreads / 64;
constexpr uint64_t kPublished = 1ull << 63;     // status word: published | second count << 32 | first count
constexpr int kMaxSubs = kMaxPasses * 4;         // sub-passes of two words in a share of 8 * passes words per thread

// What a compaction produces besides the ascending list of the marks in `bits`.
enum Mode {
  kList,      // `other`, if given, receives the marks (OR)
  kListUnion, // second list: marks of `bits` or `other`; both maps are cleared
  kListNew,   // second list, appended at seg[0]: marks not yet in `other`; `other` receives the marks (OR)
  kListLast   // the same, but both maps are cleared
};

struct Words {
  uint64_t a, b;
};

// Inclusive scan over the lanes of a wave with data-parallel-primitive moves: six vector adds.  (Cross-lane reads
// through LDS would make the compaction bound by them: 32 waves per CU times a dozen reads per sum cost 3 us.)
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

// Marks of one word that go to the second list.
template <Mode M>
__device__ __forceinline__ uint64_t second(uint64_t x, uint64_t y) {
  return M == kListUnion ? (x | y) : M == kListNew || M == kListLast ? (x & ~y) : 0ull;
}

// Marks of one word, both lists' counts in one register (low and high half).
template <Mode M>
__device__ __forceinline__ uint32_t count_of(uint64_t x, uint64_t y) {
  uint32_t c = uint32_t(__popcll(x));
  if (M != kList) c |= uint32_t(__popcll(second<M>(x, y))) << 16;
  return c;
}
__device__ __forceinline__ uint64_t widen(uint32_t c) { return uint64_t(c & 0xffffu) | (uint64_t(c >> 16) << 32); }

// Counts of one workgroup's share: its status if that appears, else its words, counted by this one thread (see the note
// on waiting above).
template <Mode M>
__device__ __forceinline__ uint64_t wait_for(const uint64_t* status, const uint64_t* bits, const uint64_t* other,
                                             int64_t first, int64_t words, int polls) {
#pragma unroll 1
  for (int it = 0; it < polls; ++it) {
    const uint64_t s = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (s & kPublished) return s & ~kPublished;
    __builtin_amdgcn_s_sleep(2);
  }
  constexpr int kBatch = M == kList ? 8 : 4;                // loads in flight; a share is a multiple of 2048 words
  uint64_t c = 0;
#pragma unroll 1
  for (int64_t k = first; k < first + words; k += kBatch) {
    uint64_t x[kBatch], y[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      x[j] = __hip_atomic_load(bits + k + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      y[j] = M == kList ? 0ull : __hip_atomic_load(other + k + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) c += widen(count_of<M>(x[j], y[j]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the words are read before the status is looked at
    const uint64_t s = __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (s & kPublished) return s & ~kPublished;
  }
  return c;
}

// The word (pair) at 32-bit word index k of a map of at most 2^25 words, so that an address is one register.
__device__ __forceinline__ uint64_t* word_at(uint64_t* map, uint32_t k) {
  return reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(map) + k * 8u);
}
__device__ __forceinline__ Words load2(uint64_t* map, uint32_t k) {
  const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(word_at(map, k));
  return Words{v.x, v.y};
}

// One workgroup's share of the map is W * passes words per thread, taken in sub-passes of S words per thread;
// a thread's S words are consecutive, so one scan per wave and sub-pass places its ids.  With REREAD = false (one
// pass) the words stay in registers between counting and writing; beyond 8 words per thread they are read again.
//
// Writing goes through a list of the non-zero words in LDS (the word, its place in the map, where its ids go), and
// the list is then shared out evenly: marks are sparse in a large map (0.2 % of the bits at 250 M vertices), so a
// walk of every thread over its own words leaves most lanes idle in every step.  The list is also what hides the
// wait for the workgroups before this one: it is built between publishing and waiting.
template <Mode M, int W, bool REREAD>
__global__ __launch_bounds__(kCompactThreads, 8) void compact_kernel(CompactArgs a) {
  constexpr int S = M == kList && W >= 4 ? 4 : 2;
  constexpr int NS = W / S;
  constexpr int kEntries = S * kCompactThreads;
  constexpr bool kDual = M != kList, kNew = M == kListNew || M == kListLast, kClear = M == kListUnion || M == kListLast;
  // counts per wave and sub-pass: at most 64 * S * 64 <= 16384 marks per list, both lists in one word
  __shared__ uint32_t wave_count[REREAD ? kMaxSubs : NS][kWaves];
  __shared__ uint32_t wave_total[kWaves], wave_total2[kWaves], wave_before[kWaves], wave_before2[kWaves];
  __shared__ int list_size[REREAD ? kMaxSubs : NS];
  __shared__ uint64_t ent_x[kEntries], ent_y[kDual ? kEntries : 1];
  __shared__ uint32_t ent_loc[kEntries], ent_loc2[kDual ? kEntries : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int passes = REREAD ? a.passes : 1;
  const uint32_t share = uint32_t(passes) * W * kCompactThreads;      // words of a workgroup
  const uint32_t word0 = blockIdx.x * share;
  if (int(threadIdx.x) < passes * NS) list_size[threadIdx.x] = 0;
  uint64_t x[NS][S], y[NS][S];
  uint32_t c = 0, c2 = 0;
  for (int p = 0; p < passes; ++p) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
      for (int j = 0; j < S; j += 2) {
        const uint32_t k = word0 + uint32_t((p * NS + s) * kEntries) + threadIdx.x * S + j;
        const Words v = load2(a.bits, k);
        x[s][j] = v.a;
        x[s][j + 1] = v.b;
        if (kDual) {
          const Words u = load2(a.other, k);
          y[s][j] = u.a;
          y[s][j + 1] = u.b;
        }
      }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      uint32_t cs = 0;
#pragma unroll
      for (int j = 0; j < S; ++j) cs += count_of<M>(x[s][j], kDual ? y[s][j] : 0);
      cs = wave_sum(cs);
      if (lane == 0) wave_count[p * NS + s][wave] = cs;
      c += cs & 0xffffu;
      c2 += cs >> 16;
    }
  }
  if (lane == 0) {
    wave_total[wave] = c;
    if (kDual) wave_total2[wave] = c2;
  }
  __syncthreads();
  const uint64_t mine = uint64_t(wave_sum(lane < kWaves ? wave_total[lane] : 0)) |
                        (kDual ? uint64_t(wave_sum(lane < kWaves ? wave_total2[lane] : 0)) << 32 : 0);
  if (threadIdx.x == 0)
    __hip_atomic_store(&a.status[blockIdx.x], mine | kPublished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  const uint32_t base2 = kNew ? uint32_t(a.seg[0]) : 0;
  const uint32_t cap = uint32_t(a.out ? a.out_cap : 0), cap2 = uint32_t(a.out2_cap);      // below 2^31 (capacity())
  uint32_t pos = 0, pos2 = 0;                 // where the ids of the sub-pass begin
  for (int p = 0; p < passes; ++p) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int sub = p * NS + s;
      const uint32_t at = uint32_t(sub * kEntries) + threadIdx.x * S;   // first word of this thread in the share
      if (REREAD) {
#pragma unroll
        for (int j = 0; j < S; j += 2) {
          const Words v = load2(a.bits, word0 + at + j);
          x[s][j] = v.a;
          x[s][j + 1] = v.b;
          if (kDual) {
            const Words u = load2(a.other, word0 + at + j);
            y[s][j] = u.a;
            y[s][j + 1] = u.b;
          }
        }
      }
      if (sub > 0) __syncthreads();           // the list of the sub-pass before this one has been used up
      // ---- list of the non-zero words; places are relative to the sub-pass
      const uint32_t per_wave = lane < kWaves ? wave_count[sub][lane] : 0;
      const uint32_t ahead = lane < wave ? per_wave : 0;                // wave < kWaves: lanes without a count add 0
      uint32_t mine_sub = 0;
#pragma unroll
      for (int j = 0; j < S; ++j) mine_sub += count_of<M>(x[s][j], kDual ? y[s][j] : 0);
      const uint32_t excl = wave_inclusive_scan(mine_sub) - mine_sub;
      uint32_t o = wave_sum(ahead & 0xffffu) + (excl & 0xffffu), o2 = kDual ? wave_sum(ahead >> 16) + (excl >> 16) : 0;
      uint64_t filled[S];
      int n_wave = 0;
#pragma unroll
      for (int j = 0; j < S; ++j) {
        filled[j] = __ballot((x[s][j] | (kClear ? y[s][j] : 0)) != 0);
        n_wave += __popcll(filled[j]);
      }
      int slot = 0;
      if (lane == 0 && n_wave) slot = atomicAdd(&list_size[sub], n_wave);
      slot = __builtin_amdgcn_readfirstlane(slot);
#pragma unroll
      for (int j = 0; j < S; ++j) {
        if ((filled[j] >> lane) & 1ull) {
          const int e = slot + __popcll(filled[j] & ((1ull << lane) - 1));
          ent_x[e] = x[s][j];
          ent_loc[e] = o | ((threadIdx.x * S + j) << 19);               // o < 2^18, word < 2^12
          if (kDual) {
            ent_y[e] = y[s][j];
            ent_loc2[e] = o2;
          }
        }
        slot += __popcll(filled[j]);
        const uint32_t cj = count_of<M>(x[s][j], kDual ? y[s][j] : 0);
        o += cj & 0xffffu;
        o2 += cj >> 16;
      }
      if (sub == 0) {                          // where this workgroup's ids begin
        uint64_t before = 0;
#pragma unroll 1
        for (int k = threadIdx.x; k < int(blockIdx.x); k += kCompactThreads)
          before += wait_for<M>(&a.status[k], a.bits, a.other, int64_t(k) * share, int64_t(share),
                                a.polls);
        const uint32_t b1 = wave_sum(uint32_t(before)), b2 = kDual ? wave_sum(uint32_t(before >> 32)) : 0;
        if (lane == 0) {
          wave_before[wave] = b1;
          if (kDual) wave_before2[wave] = b2;
        }
        if (threadIdx.x == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // published before any word is cleared
      }
      __syncthreads();
      if (sub == 0) {
        pos = wave_sum(lane < kWaves ? wave_before[lane] : 0);
        pos2 = base2 + (kDual ? wave_sum(lane < kWaves ? wave_before2[lane] : 0) : 0);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
          const int64_t total = int64_t(pos) + int64_t(uint32_t(mine));
          if (a.n_out) {
            *a.n_out = int32_t(total <= a.out_cap ? total : a.out_cap);
            if (total > a.out_cap) atomicOr(a.d_err, ERR_OVERRUN);
          }
          if (kDual) {
            int64_t end = int64_t(pos2) + int64_t(mine >> 32);
            if (end > a.out2_cap) {
              atomicOr(a.d_err, ERR_OVERRUN);
              end = a.out2_cap;
            }
            if (kNew) a.seg[1] = int32_t(end);
            if (M == kListLast && a.stats) {
              a.stats[a.stats_slot] = int32_t(end);
              a.stats[1 - a.stats_slot] = 0;
            }
            if (a.n_out2) *a.n_out2 = int32_t(end);
          }
        }
      }
      // ---- ids of the listed words
      const int n_list = list_size[sub];
      for (int e = threadIdx.x; e < n_list; e += kCompactThreads) {
        const uint64_t xw = ent_x[e];
        const uint32_t loc = ent_loc[e];
        const uint32_t wi = word0 + uint32_t(sub * kEntries) + (loc >> 19);
        uint64_t yw = kDual ? ent_y[e] : 0;
        if (M == kList && a.other) yw = *word_at(a.other, wi);
        if (xw) *word_at(a.bits, wi) = 0;
        const uint64_t sw = second<M>(xw, yw);
        uint32_t at1 = pos + (loc & 0x7ffffu), at2 = kDual ? pos2 + ent_loc2[e] : 0;
        const uint32_t id0 = wi * 64u;                     // map bits: at most 2^31
#pragma unroll 1
        for (uint64_t todo = xw | sw; todo; todo &= todo - 1) {
          const int b = __ffsll((unsigned long long)todo) - 1;
          const int32_t id = int32_t((id0 + uint32_t(b)) >> a.shift);
          if (!kDual || ((xw >> b) & 1ull)) {
            if (at1 < cap) a.out[at1] = id;
            ++at1;
          }
          if (kDual && ((sw >> b) & 1ull)) {
            if (at2 < cap2) a.out2[at2] = id;
            ++at2;
          }
        }
        if (kClear) {
          if (yw) *word_at(a.other, wi) = 0;
        } else if (kDual || a.other) {
          *word_at(a.other, wi) = yw | xw;
        }
      }
      pos += wave_sum(per_wave & 0xffffu);
      if (kDual) pos2 += wave_sum(per_wave >> 16);
    }
  }
}

// Pre-sampling's last step: bump[id] += 1 for every mark, clear the map, add the batch's frontier sizes to *acc.
// An id belongs to one thread, so the counter needs no atomic (520 k marks at 2.4 M vertices: 22.3 us with one).
__global__ __launch_bounds__(256) void bump_kernel(uint64_t* __restrict__ bits, int64_t n_words, int shift,
                                                   uint32_t* __restrict__ bump, const int32_t* __restrict__ sizes,
                                                   int32_t n_sizes, unsigned long long* __restrict__ acc) {
  const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (t == 0) {
    unsigned long long sum = 0;
    for (int32_t h = 0; h < n_sizes; ++h) sum += (unsigned long long)(sizes[h]);
    acc[0] += sum;                                // one writer, stream-ordered
  }
  for (int64_t k = t * 2; k < n_words; k += int64_t(gridDim.x) * 512) {
    const Words x = load2(bits, uint32_t(k));
    if (!(x.a | x.b)) continue;
    *reinterpret_cast<ulonglong2*>(word_at(bits, uint32_t(k))) = make_ulonglong2(0, 0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      for (uint64_t todo = h ? x.b : x.a; todo; todo &= todo - 1)
        bump[((k + h) * 64 + __ffsll((unsigned long long)todo) - 1) >> shift] += 1u;
    }
  }
}

template <Mode M>
void launch_mode(const MapGeom& g, CompactArgs a, hipStream_t s) {
  const dim3 grid{unsigned(g.groups)}, block{unsigned(kCompactThreads)};
  a.passes = g.passes;
  if (g.passes > 1 || (M != kList && g.words_per_thread == 8))   // 8 words of two maps do not fit the registers
    hipLaunchKernelGGL((compact_kernel<M, 8, true>), grid, block, 0, s, a);
  else if (g.words_per_thread == 8) hipLaunchKernelGGL((compact_kernel<kList, 8, false>), grid, block, 0, s, a);
  else if (g.words_per_thread == 4) hipLaunchKernelGGL((compact_kernel<M, 4, false>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((compact_kernel<M, 2, false>), grid, block, 0, s, a);
}

// A list holds fewer than 2^31 ids, and the kernel compares an id's place with the capacity in 32 bits; a caller may
// state any capacity at or above the worst case.
int64_t capacity(int64_t cap) { return std::min<int64_t>(cap, INT32_MAX); }

CompactArgs base_args(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                      uint32_t* d_err) {
  CompactArgs a = {};
  a.bits = m.frontier;
  a.other = m.gather;
  a.status = m.status;
  a.polls = m.polls;
  a.out = out;
  a.out_cap = capacity(out_cap);
  a.n_out = n_out;
  a.d_err = d_err;
  a.shift = di.spread_shift;
  return a;
}

}  // namespace

void launch_compact(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                    uint32_t* d_err, hipStream_t s) {
  launch_mode<kList>(m.geom, base_args(di, m, out, out_cap, n_out, d_err), s);
}

void launch_compact_gather(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                           uint32_t* d_err, hipStream_t s) {
  CompactArgs a = base_args(di, m, out, out_cap, n_out, d_err);
  a.bits = m.gather;
  a.other = nullptr;
  launch_mode<kList>(m.geom, a, s);
}

void launch_compact_both(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                         int32_t* all, int64_t all_cap, int32_t* n_all, uint32_t* d_err, hipStream_t s) {
  CompactArgs a = base_args(di, m, out, out_cap, n_out, d_err);
  a.out2 = all;
  a.out2_cap = capacity(all_cap);
  a.n_out2 = n_all;
  launch_mode<kListUnion>(m.geom, a, s);
}

void launch_compact_new(const DeviceInfo& di, const DedupMaps& m, int32_t* out, int64_t out_cap, int32_t* n_out,
                        int32_t* listed, int64_t listed_cap, int32_t* seg, int32_t* n_listed, bool last, int32_t* stats,
                        int32_t stats_slot, uint32_t* d_err, hipStream_t s) {
  CompactArgs a = base_args(di, m, out, out_cap, n_out, d_err);
  a.out2 = listed;
  a.out2_cap = capacity(listed_cap);
  a.n_out2 = n_listed;
  a.seg = seg;
  a.stats = stats;
  a.stats_slot = stats_slot;
  if (last) launch_mode<kListLast>(m.geom, a, s);
  else launch_mode<kListNew>(m.geom, a, s);
}

void launch_bump(const DeviceInfo& di, const DedupMaps& m, uint32_t* bump, const int32_t* sizes, int32_t n_sizes,
                 unsigned long long* acc, hipStream_t s) {
  int64_t blocks = (m.geom.words() + 511) / 512;
  if (blocks > di.num_cus * 8) blocks = di.num_cus * 8;
  hipLaunchKernelGGL(bump_kernel, dim3(unsigned(blocks)), dim3(256), 0, s, m.gather, m.geom.words(), di.spread_shift,
                     bump, sizes, n_sizes, acc);
}

}  // namespace lgp
