// Steps before and after the main all-reduce stage, for gfx950: per-super-group statistics
// (Section 3.1), their combination over workers with the bf16 exchange format (Sections 3.1,
// 3.5), the bit allocation with tied thresholds (Section 3.2, Appendix A), the reorder into
// increasing width order (Section 3.5), the means the main stage subtracts in that order
// (Section 3.1) and the final restore (Section 3.4, last paragraph).  All of them stream each entry once; the allocation
// works on 4 bytes per super-group.
#include <type_traits>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dq_bounds.h"
#include "dq_device.h"

namespace {

constexpr int kSG = 256;
constexpr int kThreads = 256;

__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }
__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ T gld(const void *p) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T *>((uintptr_t)p);
}
template <typename T>
__device__ __forceinline__ void gst(void *p, T v) {
  *reinterpret_cast<__attribute__((address_space(1))) T *>((uintptr_t)p) = v;
}

// fp32 -> bf16 pattern, round to nearest, ties to even (finite inputs)
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t b = f2u(f);
  return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}

// ---------------------------------------------------------------------------------------
// Statistics.  One wave takes 4 super-groups: lane l owns group l (16 entries,
// 32 or 64 consecutive bytes), sums them left to right in fp32 (squares by fma), and the 16
// lanes of a row are combined pairwise (partner distance 1, 2, 4, 8).  It is bound by memory.  A wave has one tile and then makes room
// for the next block's, so that some tiles are always being requested: 500,000 super-groups in bf16 42 us, in fp32 83, where a grid of
// what the GPU holds at once, its waves going round the tiles, took 51 and 93; 51,200 in bf16 6.0 -> 5.75.  (Two and four tiles
// per wave requested together: 44 and 45 us.)
template <typename LT>
struct Entries {
  u32x4 w[sizeof(LT) == 4 ? 4 : 2];  // a lane's 16 entries, raw
};
template <typename LT>
__device__ __forceinline__ Entries<LT> load_entries(const void *x, uint64_t first) {
  const uint8_t *p = static_cast<const uint8_t *>(x) + first * sizeof(LT);
  Entries<LT> e;
#pragma unroll
  for (int i = 0; i < (sizeof(LT) == 4 ? 4 : 2); ++i) e.w[i] = gld<u32x4>(p + 16 * i);
  return e;
}
// In the row's first lane: its 16 lanes' sum, lane pairs first, then pairs of pairs, then the lanes 4 and 8 further on.
__device__ __forceinline__ float row_sum(float x) {
  auto from = [&](auto ctrl) { return u2f((uint32_t)__builtin_amdgcn_update_dpp(0, (int)f2u(x), decltype(ctrl)::value, 0xF, 0xF, true)); };
  x += from(std::integral_constant<int, 0xB1>());   // quad_perm 1,0,3,2
  x += from(std::integral_constant<int, 0x4E>());   // quad_perm 2,3,0,1
  x += from(std::integral_constant<int, 0x12C>());  // row_ror 12
  x += from(std::integral_constant<int, 0x128>());  // row_ror 8
  return x;
}
// Sum and sum of squares over the row's super-group, in the row's first lane.
template <typename LT>
__device__ __forceinline__ void row_sums(const Entries<LT> &e, float &s, float &f) {
  float v[16];
  if constexpr (sizeof(LT) == 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[4 * i] = u2f(e.w[i].x); v[4 * i + 1] = u2f(e.w[i].y); v[4 * i + 2] = u2f(e.w[i].z); v[4 * i + 3] = u2f(e.w[i].w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t w[4] = {e.w[i].x, e.w[i].y, e.w[i].z, e.w[i].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[8 * i + 2 * j] = u2f(w[j] << 16);
        v[8 * i + 2 * j + 1] = u2f(w[j] & 0xFFFF0000u);
      }
    }
  }
  s = 0.0f;
  f = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    s += v[k];
    f = __builtin_fmaf(v[k], v[k], f);
  }
  s = row_sum(s);
  f = row_sum(f);
}

template <typename LT>
__global__ void __launch_bounds__(kThreads) k_stats(const void *x, uint64_t n_sg, float *mu, float *F) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t t = (uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const uint64_t sg = t * 4 + (lane >> 4);
  float s, f;
  row_sums<LT>(load_entries<LT>(x, min(sg, n_sg - 1) * kSG + (lane & 15u) * 16), s, f);  // idle rows redo the last SG, store nothing
  if ((lane & 15u) == 0 && sg < n_sg) {
    gst<float>(mu + sg, s * (1.0f / kSG));
    gst<float>(F + sg, f);
  }
}

// k_stats of every worker and k_combine in one pass: a simulated all-reduce, which holds all workers' tensors, has no use for
// the single workers' statistics.  One launch instead of n + 1.
struct WorkerTensors {
  const void *x[dq::kMostTensors];
};
template <typename LT>
__global__ void __launch_bounds__(kThreads) k_stats_all(WorkerTensors W, uint32_t n, uint64_t n_sg, float *mu, float *F, const void **grads) {
  if (grads && blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < 2 * n; i += kThreads) grads[i] = W.x[i < n ? i : i - n];
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t wave = (uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const uint64_t n_waves = (uint64_t)gridDim.x * (kThreads / 64);
  const uint64_t n_tiles = (n_sg + 3) / 4;
  for (uint64_t t = wave; t < n_tiles; t += n_waves) {
    const uint64_t sg = min(t * 4 + (lane >> 4), n_sg - 1), first = sg * kSG + (lane & 15u) * 16;
    float sm = 0.0f, sf = 0.0f;
    Entries<LT> e = load_entries<LT>(W.x[0], first);
    for (uint32_t w = 0; w < n; ++w) {
      Entries<LT> next = e;
      if (w + 1 < n) next = load_entries<LT>(W.x[w + 1], first);
      float s, f;
      row_sums<LT>(e, s, f);
      sm = sm + u2f(bf16_rne(s * (1.0f / kSG)) << 16);
      sf = sf + u2f(bf16_rne(f) << 16);
      e = next;
    }
    if ((lane & 15u) == 0 && t * 4 + (lane >> 4) < n_sg) {
      gst<float>(mu + sg, sm / (float)n);
      gst<float>(F + sg, sf);
    }
  }
}

// The same where that leaves a worker's tile after the other's trip to memory: a wave takes every `slots`-th worker's, and their numbers meet in LDS, where
// they are summed in the order of the ranks.  What bounds it are launch and trips.  Taken by more than four workers up to so many waves per CU that memory
// would be what bounds it, 11 in bf16 and 7 in fp32 (the kernel alone in a graph, us, one wave per tile -> 2, 4, 8, 16): bf16, 32 workers' 64 super-groups 8.0 ->
// 5.7, 4.0, 3.1, 3.0; 8 of 1,000 3.1 -> 2.7, 2.4, 2.3; 18 of 2,000 5.3 -> 4.1, 3.4, 3.4, 3.5; 64 of 4,000 22.7 -> 20.2, 20.6, 22.0, 21.3; 18 of 6,000 9.8 ->
// 10.0, 10.1; 4 of 3,000 2.4 -> 2.5, 2.5; fp32, 12 of 3,000 6.8 -> 6.1, 5.6, 5.5; 12 of 4,000 8.6 -> 9.2, 9.5.  30 workers' all-reduce of 210 31.2 -> 26.1.
constexpr uint32_t kMostSlots = 16;  // waves for one tile
template <typename LT>
__global__ void __launch_bounds__(64 * kMostSlots) k_stats_split(WorkerTensors W, uint32_t n, uint32_t slots, uint32_t tiles, uint64_t n_sg, float *mu,
                                                                 float *F, const void **grads) {
  extern __shared__ float2 part[];  // tile of the block, worker, super-group
  if (grads && blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < 2 * n; i += blockDim.x) grads[i] = W.x[i < n ? i : i - n];
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t tile = wave / slots, slot = wave - tile * slots;
  const uint64_t t0 = (uint64_t)blockIdx.x * tiles, first = min((t0 + tile) * 4 + (lane >> 4), n_sg - 1) * kSG + (lane & 15u) * 16;
  Entries<LT> e = load_entries<LT>(W.x[slot], first);
  for (uint32_t w = slot; w < n; w += slots) {
    Entries<LT> next = e;
    if (w + slots < n) next = load_entries<LT>(W.x[w + slots], first);
    float s, f;
    row_sums<LT>(e, s, f);
    if ((lane & 15u) == 0) part[(tile * n + w) * 4 + (lane >> 4)] = float2{u2f(bf16_rne(s * (1.0f / kSG)) << 16), u2f(bf16_rne(f) << 16)};
    e = next;
  }
  __syncthreads();
  const uint64_t sg = t0 * 4 + threadIdx.x;
  if (threadIdx.x >= 4 * tiles || sg >= n_sg) return;
  const float2 *p = part + (threadIdx.x >> 2) * n * 4 + (threadIdx.x & 3u);
  float sm = 0.0f, sf = 0.0f;
#pragma unroll 8
  for (uint32_t w = 0; w < n; ++w) {
    sm = sm + p[4 * w].x;
    sf = sf + p[4 * w].y;
  }
  gst<float>(mu + sg, sm / (float)n);
  gst<float>(F + sg, sf);
}

// Combination over workers: contributions rounded to bf16 (what is exchanged), summed in rank
// order in fp32; the mean of the means by one division.  A thread per super-group, eight workers' numbers requested at a time: what
// bounds it are the trips to memory (8 workers, 51,200 super-groups: 3.2 us with one, 4.8 with one per worker).
__global__ void __launch_bounds__(kThreads) k_combine(const float *mu_all, const float *F_all, uint32_t n, uint64_t J,
                                                      uint64_t count, float *mu, float *F) {
  const uint64_t j = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= count) return;  // of a worker's J
  float sm = 0.0f, sf = 0.0f;
  for (uint32_t i = 0; i < n; i += 8) {
    float m[8], f[8];
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) {
      const uint64_t at = (uint64_t)min(i + k, n - 1) * J + j;
      m[k] = gld<float>(mu_all + at);
      f[k] = gld<float>(F_all + at);
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k)
      if (i + k < n) {
        sm = sm + u2f(bf16_rne(m[k]) << 16);
        sf = sf + u2f(bf16_rne(f[k]) << 16);
      }
  }
  gst<float>(mu + j, sm / (float)n);
  gst<float>(F + j, sf);
}

// ---------------------------------------------------------------------------------------
// Allocation: a search is one block of 1024 threads (of which a bucket has one, or one for each of its rows of 1024 super-groups).  In buckets of at most
// 64 rows the threads hold all norms in registers, four neighbours each, so every global access
// is coalesced; larger ones are read again in every pass.  Values are handled as int32 bit patterns: non-negative floats order like their
// patterns, and the difference of two patterns below 2^31 has the sign of the comparison,
// F >= theta  <=>  bits(F) - bits(theta) >= 0.  Negative values and NaN count as +0; places past
// the bucket's end hold -1, which is below every threshold.
constexpr int kAllocThreads = 1024;
constexpr int kAllocWaves = kAllocThreads / 64;
constexpr int kRegs = 64;
constexpr uint32_t kBins = 2048;  // 2 per thread

__device__ __forceinline__ int32_t pattern_of(float f) { return f > 0.0f ? (int32_t)f2u(f) : 0; }

// class 0, 1, 2, 3 = 2, 4, 8, 16 bits; 4 = no super-group.  Section 3.2's tied thresholds:
// p8 = pattern of T_{4,8}, p4 = pattern of T_{2,4} = T_{4,8} * 17/512, p16 = pattern of
// T_{8,16} = T_{4,8} * 2^17/257 (0x7FFFFFFF, above every value, when 16 bits are not allowed).
__device__ __forceinline__ uint32_t class_of(int32_t v, int32_t p4, int32_t p8, int32_t p16) {
  return v < 0 ? 4u : (v >= p16 ? 3u : (v >= p8 ? 2u : (v >= p4 ? 1u : 0u)));
}
constexpr int32_t kNever = 0x7FFFFFFF;
__device__ __forceinline__ int32_t p4_from(uint32_t pattern) { return (int32_t)f2u(u2f(pattern) * (17.0f / 512.0f)); }
__device__ __forceinline__ int32_t p16_from(uint32_t pattern, bool allow16) {
  return allow16 ? (int32_t)f2u(u2f(pattern) * (131072.0f / 257.0f)) : kNever;
}

// Widths and positions once the threshold is known (counts[5b..5b+4] as the search left them):
// grid (ceil(J / 1024), buckets), a block ranks its own 1024 super-groups: position = the row's first place of the
// class + members in earlier waves + members in lower lanes.  The search left each row's four first places where the
// row's own positions go (read here before they are overwritten); the last row, which may be shorter than that, counts
// back from the classes' ends.  (A block that counted the rows before its own took 12.5 us for 51,200 super-groups.)
struct Placed {
  uint32_t k, at;  // class (4: beyond the bucket), position
};
__device__ __forceinline__ Placed place_row(const float *F, uint32_t J, bool allow16, const uint32_t *cnt, const uint32_t *places, uint32_t row,
                                            bool last, uint32_t (*mine_w)[4]) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t j = row * kAllocThreads + tid;
  const float f = gld<float>(F + min(j, J - 1));
  uint32_t at_row[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) at_row[c] = last ? gld<uint32_t>(cnt + c) : gld<uint32_t>(places + (uint64_t)row * kAllocThreads + c);
  const uint32_t pattern = gld<uint32_t>(cnt + 4);
  const int32_t p8 = (int32_t)pattern, p4 = p4_from(pattern), p16 = p16_from(pattern, allow16);
  const uint32_t k = j < J ? class_of(pattern_of(f), p4, p8, p16) : 4u;
  const uint64_t b[4] = {__ballot(k == 0), __ballot(k == 1), __ballot(k == 2), __ballot(k == 3)};
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) mine_w[wave][i] = (uint32_t)__builtin_popcountll(b[i]);
  }
  __syncthreads();
  if (k == 4) return Placed{4u, 0u};
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kAllocWaves; ++w) {
    before += (uint32_t)w < wave ? mine_w[w][k] : 0u;
    all += mine_w[w][k];
  }
  uint32_t at = k == 0 ? at_row[0] : (k == 1 ? at_row[1] : (k == 2 ? at_row[2] : at_row[3]));
  if (last) {  // at_row holds the classes' sizes: the class's end less what this row adds to it
    at = at_row[0] - all;
    if (k > 0) at += at_row[1];
    if (k > 1) at += at_row[2];
    if (k > 2) at += at_row[3];
  }
  const uint64_t mine = k == 0 ? b[0] : (k == 1 ? b[1] : (k == 2 ? b[2] : b[3]));
  return Placed{k, at + before + __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u))};
}

__global__ void __launch_bounds__(kAllocThreads) k_alloc_positions(const float *F_all, uint32_t J, bool allow16,
                                                                   const uint32_t *counts_all, uint8_t *widths_all,
                                                                   uint32_t *pos_all) {
  __shared__ uint32_t mine_w[kAllocWaves][4];
  const uint64_t first = (uint64_t)blockIdx.y * J;
  const uint32_t j = blockIdx.x * kAllocThreads + threadIdx.x;
  const Placed x = place_row(F_all + first, J, allow16, counts_all + 5ull * blockIdx.y, pos_all + first, blockIdx.x, blockIdx.x + 1 == gridDim.x, mine_w);
  if (x.k < 4) {
    gst<uint8_t>(widths_all + first + j, (uint8_t)(2u << x.k));
    gst<uint32_t>(pos_all + first + j, x.at);
  }
}

// The search for buckets of at most 64 rows of 1024, the norms' patterns in registers: register 4g + q of thread t holds
// norm 4096 g + 4 t + q.  Every pass skips the groups of 4096 that the bucket does not have.
//
// Wanted: the smallest fp32 pattern in [1, +inf] whose allocation fits (the host has checked 2J <= budget).  With
// c8, c4, c16 = norms at or above T_{4,8} and its tied thresholds, cost = 2J + 4 c8 + 2 c4 + 8 c16 never increases with
// the threshold, so a bracket (lo does not fit or is 0, hi fits) is narrowed.  The first level is a histogram of the top 11 bits of all norms: its
// suffix counts give at the bins' boundaries a lower and an upper bound of the cost (c8 is exact there, c4 and c16 lie between the counts of two
// bins), which leave 1 to 3 bins of 2^20 patterns.  The next two look at the places where the cost falls: a norm v costs 4 bits less beyond the threshold v,
// 2 less beyond the last threshold T whose tied one is at most v, 8 less beyond the last whose other tied one is.  One histogram of those places,
// weighted, has the cost at every boundary as a suffix sum: up to 4096 bins, then up to 2048 of single patterns.
//
// What bounds it: one CU's vector ALU and LDS (51,200 norms are 800 wave instructions for every instruction of a pass,
// and an LDS atomic of a wave takes 12 cycles) and, for small buckets, the barriers and scans of the levels.
// 51,200 norms take 18.4 us, 8,192 8.1; with a histogram for each of the thresholds at every level, and bounds of the cost gathered from them, 21.0 and 11.3 (a
// whole allocation with 16-bit widths 22.8 and 10.8 instead of 27.8 and 16.4; of 51,200 norms within a tenth of each other 28.2 instead of 29.5, within a
// factor of two 28.7 instead of 27.2, of equal ones 62 instead of 109).
constexpr uint32_t kCopies = 8;
constexpr uint32_t kKept = 15;  // of a thread's up to 64 norms; up to 16 always fit
constexpr uint32_t kPlaces = 4096, kLastPlaces = 2048;  // bins of the second and third level
static_assert(kPlaces == 4 * kAllocThreads && kLastPlaces == 2 * kAllocThreads, "four and two per thread");

// Inclusive sum over the lanes of a row of 16, and over the wave
__device__ __forceinline__ uint32_t row_scan(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, false);  // row_shr 1, 2, 4, 8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xF, 0xF, false);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xF, 0xF, false);
  return x;
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t x) {
  x = row_scan(x);
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xA, 0xF, false);  // row 0 into 1, row 2 into 3
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xC, 0xF, false);  // rows 0 and 1 into 2 and 3
  return x;
}

template <uint32_t BINS>
struct OwnBins {
  uint32_t n[BINS / kAllocThreads], before;
};

// The least s with x >> s < bins (bins between 2^12 and 2^13; thresholds' denormal ranges hold up to 510 patterns to one)
__device__ __forceinline__ uint32_t shift_to(uint32_t x, uint32_t bins) {
  const uint32_t s = x >> 13 ? 19u - (uint32_t)__builtin_clz(x) : 0u;
  return s + (x >> s >= bins ? 1u : 0u);
}

// The last pattern T with tied(T) <= v, where tied multiplies by `by`, as far as [lo, hi] goes (lo - 1: none of it; hi: all): within a few of v
// divided by it, but where either is denormal or infinite.
__device__ __forceinline__ uint32_t last_tied(uint32_t v, float by, float back, uint32_t lo, uint32_t hi) {
  auto at_most = [&](uint32_t T) { return f2u(u2f(T) * by) <= v; };
  const uint32_t x = max(f2u(u2f(v) * back), 2u) - 2u;
  if (at_most(x) && !at_most(x + 5)) return x + (at_most(x + 1) ? 1u : 0u) + (at_most(x + 2) ? 1u : 0u) + (at_most(x + 3) ? 1u : 0u) + (at_most(x + 4) ? 1u : 0u);
  if (!at_most(lo)) return lo - 1;
  if (at_most(hi)) return hi;
  uint32_t below = lo, above = hi;
  while (above - below > 1) {
    const uint32_t mid = below + (above - below) / 2;
    if (at_most(mid)) below = mid; else above = mid;
  }
  return below;
}

// A block's LDS: the first level's counters, over which the threads then lay their norms that the other levels look at, and those levels' counters: 91,520 bytes.  A search that
// runs beside a whole replay waits for a CU that has that much in one piece, and registers for sixteen waves; two blocks
// of k_walk (29 KB, 96 registers) may stay beside k_search, k_search_listed and k_search_positions (91,520 to 92,032 bytes), one beside k_search_arrange (116,768), whose first
// blocks make the replay's tables.
constexpr uint32_t kFirstWords = (kBins + 1) * kCopies;
static_assert((kKept + 1) * kAllocThreads <= kFirstWords, "the norms set aside");

struct SearchSpace {
  alignas(16) uint32_t room[kFirstWords];
  alignas(16) uint32_t places[kPlaces + 4], last_places[kLastPlaces];  // places[kPlaces]: beyond the bracket
  uint32_t wsum[2][kAllocWaves], wfit[kAllocWaves], row_n[kRegs][3], crossing[2][2], exact[2][3][kAllocWaves];
};
static_assert(sizeof(SearchSpace) == 91520, "two blocks of k_walk beside one that searches");
// h[b] for b < BINS becomes the sum of h[b], h[b + 1], ..., the thread's own bins in x between the two halves, which a
// barrier separates
template <typename X>
__device__ __forceinline__ void sums_begin(X &x, uint32_t *wsum) {
  uint32_t sum = 0;
  for (uint32_t one : x.n) sum += one;
  const uint32_t upto = wave_scan(sum);
  x.before = upto - sum;  // in the wave, before the thread's own bins
  if ((threadIdx.x & 63u) == 63) wsum[threadIdx.x >> 6] = upto;
}
template <typename X>
__device__ __forceinline__ void sums_end(const X &x, const uint32_t *wsum, uint32_t *h) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t upto = row_scan(wsum[threadIdx.x & 15u]), all = __builtin_amdgcn_readlane(upto, 15);
  uint32_t left = all - (wave ? __builtin_amdgcn_readlane(upto, wave - 1) : 0u) - x.before;
  uint32_t *own = h + threadIdx.x * (sizeof(x.n) / 4);
  for (uint32_t one : x.n) {
    *own++ = left;
    left -= one;
  }
}
// The last of the bin boundaries 0 .. n-1 that surely does not fit and the last that may not (boundary 0 is the
// bracket's lower end): every PER-th first, then, by every wave for itself, those between.  fails(bin, over, may) says it of one.
template <uint32_t PER, typename F>
__device__ __forceinline__ void last_failing(uint32_t n, F cost_fails, uint32_t *wfit, uint32_t &surely, uint32_t &perhaps) {
  const uint32_t lane = threadIdx.x & 63u;
  auto fails = [&](uint32_t bin, bool &over, bool &may) {
    over = may = true;
    if (bin) cost_fails(min(bin, n - 1), over, may);
    over = over && bin < n;
    may = may && bin < n;
  };
  bool over, may;
  fails(threadIdx.x * PER, over, may);
  const uint32_t both = (uint32_t)__builtin_popcountll(__ballot(over)) + ((uint32_t)__builtin_popcountll(__ballot(may)) << 16);
  if (lane == 0) wfit[threadIdx.x >> 6] = both;
  __syncthreads();
  const uint32_t all = __builtin_amdgcn_readlane(row_scan(wfit[lane & 15u]), 15);
  surely = ((all & 0xFFFFu) - 1) * PER;
  perhaps = ((all >> 16) - 1) * PER;
  const bool between = (lane & 31u) < PER - 1;
  fails((lane < 32 ? surely : perhaps) + 1 + (lane & 31u), over, may);
  surely += (uint32_t)__builtin_popcountll(__ballot(between && lane < 32 && over));
  perhaps += (uint32_t)__builtin_popcountll(__ballot(between && lane >= 32 && may));
}

// What is left of a search: T lies above lo, which does not fit (or is 0), and at most at hi, which does; lo4 .. hi16: around their tied ones.
struct Bracket {
  uint32_t lo, hi, lo4, hi4, lo16, hi16;
  uint32_t base;    // cost at hi, but for tied norms that the first level puts beyond it
  uint32_t n_kept;  // norms inside that the thread has set aside
};
// An event: a norm costs `weight` more up to a threshold; of what kind, and how far above the bracket's lower end that is.
constexpr uint32_t kMostAbove = 1u << 30;
__device__ __forceinline__ uint32_t event_of(uint32_t kind, uint32_t upto) { return kind << 30 | upto; }  // 0, 1, 2: T_{4,8}, T_{2,4}, T_{8,16}
__device__ __forceinline__ uint32_t kind_of(uint32_t event) { return event >> 30; }
__device__ __forceinline__ uint32_t upto_of(uint32_t event) { return event & (kMostAbove - 1u); }
__device__ __forceinline__ uint32_t weight_of(uint32_t event) { return 0x824u >> (4 * (event >> 30)) & 15u; }
__device__ __forceinline__ uint32_t tied4_of(uint32_t pattern) { return f2u(u2f(pattern) * (17.0f / 512.0f)); }
__device__ __forceinline__ uint32_t tied16_of(uint32_t pattern) { return f2u(u2f(pattern) * (131072.0f / 257.0f)); }

// Down to a width of one pattern: hi is T.  The norms set aside lie in S.room, thread by thread; each_event(body) has what others cost and up to where
// (event_of).
struct NoEvents {};
template <bool ALLOW16, typename Events>
__device__ __forceinline__ void to_one_pattern(Bracket &bracket, uint32_t budget, SearchSpace &S, Events each_event) {
  auto &places = S.places;
  auto &last_places = S.last_places;
  auto &wsum = S.wsum;
  auto &crossing = S.crossing;
  using std::integral_constant;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_kept = bracket.n_kept;
  uint32_t(*const kept)[kAllocThreads] = reinterpret_cast<uint32_t(*)[kAllocThreads]>(S.room);
  uint32_t lo = bracket.lo, hi = bracket.hi, lo4 = bracket.lo4, hi4 = bracket.hi4, lo16 = bracket.lo16, hi16 = bracket.hi16, base = bracket.base;
  [[maybe_unused]] const uint32_t start = lo;
  // One level: of the boundaries lo + (b << s) the last that does not fit (the first, if none: lo) and the one behind it are the new bracket.
  auto level = [&](uint32_t *h, auto per_thread, uint32_t s, uint32_t turn) {
    constexpr uint32_t kOwn = decltype(per_thread)::value;
    const uint32_t width = hi - lo, width4 = hi4 - lo4, width16 = hi16 - lo16;
    // a norm of a tied bracket: beyond the bracket, or in the bin of the last pattern whose tied one is at most v, which v divided by the
    // ratio misses by two patterns at most
    auto fall = [&](uint32_t v, float by, float back, uint32_t from, uint32_t end, uint32_t weight) {
      if (v >= end) {
        atomicAdd(&places[kPlaces], weight);
      } else if (v >= from) {
        uint32_t b;
        if (kOwn > 2 && s >= 2 && v >= 0x06000000u) {  // nothing denormal: a bin before or behind, at most
          auto at_most = [&](uint32_t T) { return f2u(u2f(T) * by) <= v; };
          b = (min(max(f2u(u2f(v) * back), lo), hi - 1) - lo) >> s;
          const uint32_t T = lo + (b << s);
          b = at_most(T + (1u << s)) ? b + 1 : at_most(T) ? b : b - 1;
        } else {
          b = (last_tied(v, by, back, lo, hi) - lo) >> s;
        }
        atomicAdd(&h[b], weight);
      }
    };
    const uint32_t from4 = tied4_of(lo), end4 = tied4_of(hi), from16 = ALLOW16 ? tied16_of(lo) : 0u, end16 = ALLOW16 ? tied16_of(hi) : 0u;
    auto count = [&](uint32_t v) {
      if (v - lo < width) atomicAdd(&h[(v - lo) >> s], 4u);
      if (v - lo4 < width4) fall(v, 17.0f / 512.0f, 512.0f / 17.0f, from4, end4, 2u);
      if (ALLOW16 && v - lo16 < width16) fall(v, 131072.0f / 257.0f, 257.0f / 131072.0f, from16, end16, 8u);
    };
    for (uint32_t i = 0; i < n_kept; ++i) count(kept[i][tid]);
    if constexpr (!__is_same(Events, NoEvents))
      each_event([&](uint32_t event) {
        const uint32_t at = start + upto_of(event) - lo;
        if (at < width) atomicAdd(&h[at >> s], weight_of(event));
      });
    __syncthreads();
    uint32_t own[kOwn], sum = 0;
#pragma unroll
    for (uint32_t i = 0; i < kOwn; ++i) {
      own[i] = h[tid * kOwn + i];
      sum += own[i];
    }
    const uint32_t beyond = kOwn > 2 ? places[kPlaces] : 0u;
    const uint32_t upto = wave_scan(sum);
    if (lane == 63) wsum[turn][wave] = upto;
    __syncthreads();
    const uint32_t waves_upto = row_scan(wsum[turn][lane & 15u]), all = __builtin_amdgcn_readlane(waves_upto, 15);
    uint32_t behind = base + beyond + all - (wave ? __builtin_amdgcn_readlane(waves_upto, wave - 1) : 0u) - upto;  // cost behind the thread's bins
    if (behind <= budget && (behind + sum > budget || tid == 0)) {
      uint32_t b = kOwn - 1;  // of the thread's bins
#pragma unroll
      for (uint32_t i = kOwn - 1; i > 0; --i)
        if (b == i && behind + own[i] <= budget) {
          behind += own[i];
          b = i - 1;
        }
      crossing[turn][0] = tid * kOwn + b;
      crossing[turn][1] = behind;
    }
    __syncthreads();
    const bool none = base + beyond > budget;  // infinite norms: not even +inf fits
    const uint32_t bin = none ? (width - 1) >> s : crossing[turn][0];
    base = none ? base + beyond : crossing[turn][1];
    lo += bin << s;
    hi = min(hi, lo + (1u << s));
    lo4 = tied4_of(lo);
    hi4 = tied4_of(hi);
    if (ALLOW16) {
      lo16 = tied16_of(lo);
      hi16 = tied16_of(hi);
    }
  };
  if (hi - lo > 1) level(places, integral_constant<uint32_t, 4>{}, shift_to(hi - lo - 1, kPlaces), 0);
  while (hi - lo > kLastPlaces) {  // a first bracket of more than four bins
    places[4 * tid] = places[4 * tid + 1] = places[4 * tid + 2] = places[4 * tid + 3] = 0;
    if (tid == 0) places[kPlaces] = 0;
    __syncthreads();
    level(places, integral_constant<uint32_t, 4>{}, shift_to(hi - lo - 1, kPlaces), 0);
    __syncthreads();
  }
  if (hi - lo > 1) level(last_places, integral_constant<uint32_t, 2>{}, 0, 1);
  bracket.hi = hi;
}

// The threshold's pattern; S.row_n holds, for every row, how many norms are at or above the three thresholds.
// ASIDE: buckets of more than 16 rows, whose threads hold up to 64 norms each, so that those inside the brackets may be more than the kKept that have room.
// given: a bracket to go on from instead of the first level's (for 2, 4 and 8 bits), with the norms at or above its ends and the costs there.
struct NoBracket {};
struct Given {
  uint32_t lo, hi, at_lo, at_hi, cost_lo, base;
};
template <bool ALLOW16, bool ASIDE, typename G = NoBracket>
__device__ __forceinline__ uint32_t search_block(const float *F, uint32_t J, uint64_t max_code_bits, SearchSpace &S, const G &given = G()) {
  constexpr bool kGiven = !__is_same(G, NoBracket);
  static_assert(!kGiven || !ALLOW16, "");
  auto &room = S.room;
  auto &places = S.places;
  auto &last_places = S.last_places;
  auto &wsum = S.wsum;
  auto &wfit = S.wfit;
  auto &row_n = S.row_n;
  auto &exact = S.exact;
  uint32_t *const h8 = room;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t(*const kept)[kAllocThreads] = reinterpret_cast<uint32_t(*)[kAllocThreads]>(room);  // per thread its norms inside the brackets
  int32_t fr[kRegs];
  auto each_group = [&](auto body) {
#pragma unroll
    for (int g = 0; g < kRegs / 4; ++g)
      if (g * 4u * kAllocThreads < J) body(g);
  };
  auto each_norm = [&](auto body) {
    each_group([&](int g) {
#pragma unroll
      for (int k = 4 * g; k < 4 * g + 4; ++k) body(k);
    });
  };
  each_group([&](int g) {  // all loads in flight at once; those beyond the end read the last four
    const uint32_t e = (g * kAllocThreads + tid) * 4u;
    if (J >= 4) {
      typedef float Float4 __attribute__((ext_vector_type(4), aligned(4)));
      const Float4 f = *(const __attribute__((address_space(1))) Float4 *)(uintptr_t)(F + min(e, J - 4));
#pragma unroll
      for (int q = 0; q < 4; ++q) fr[4 * g + q] = (int32_t)f2u(f[q]);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) fr[4 * g + q] = (int32_t)f2u(gld<float>(F + min(e + q, J - 1)));
    }
  });
  for (uint32_t b = tid; b < kFirstWords / 4; b += kAllocThreads) reinterpret_cast<uint4 *>(room)[b] = make_uint4(0, 0, 0, 0);
  reinterpret_cast<uint4 *>(places)[tid] = make_uint4(0, 0, 0, 0);
  last_places[tid] = last_places[tid + kAllocThreads] = 0;
  if (tid == 0) places[kPlaces] = 0;
  if (tid < kRegs * 3) (&row_n[0][0])[tid] = 0;
  each_group([&](int g) {
    const uint32_t e = (g * kAllocThreads + tid) * 4u;
    const uint32_t skip = J >= 4 && e > J - 4 ? e - (J - 4) : 0u;  // the four that were read start that much earlier
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int32_t v = pattern_of(u2f((uint32_t)fr[4 * g + q]));
      fr[4 * g + q] = J >= 4 ? ((uint32_t)q >= skip ? v : -1) : (e + q < J ? v : -1);
    }
  });
  using std::integral_constant;

  // level 1: bins of 2^20 patterns, 2040 << 20 is +infinity.  The norms of a bucket share a few dozen bins: kCopies
  // counters of each, in banks next to each other, keep the lanes of a wave from queueing for one word.  The bin before
  // the first takes the threads beyond the bucket's end.
  uint32_t lo, hi, lo4, hi4, lo16 = 0, hi16 = 0;
  uint32_t base;            // cost at hi, but for the tied norms between its tied thresholds and the bins' ends
  uint32_t at_lo, at_hi;    // norms at or above the brackets' ends, in all
  uint32_t cost_lo;         // at most
  if constexpr (kGiven) {
    lo = given.lo;
    hi = given.hi;
    lo4 = tied4_of(lo);
    hi4 = tied4_of(hi);
    base = given.base;
    at_lo = given.at_lo;
    at_hi = given.at_hi;
    cost_lo = given.cost_lo;
    __syncthreads();
  } else {
    __syncthreads();
    uint32_t *mine = room + kCopies + (lane & (kCopies - 1));
    each_norm([&](int k) { atomicAdd(mine + (fr[k] >> 20) * (int)kCopies, 1u); });
    __syncthreads();
    OwnBins<kBins> first;
    for (uint32_t i = 0; i < kBins / kAllocThreads; ++i) {
      first.n[i] = 0;
#pragma unroll
      for (uint32_t c = 0; c < kCopies; ++c) first.n[i] += room[(kBins / kAllocThreads * tid + i + 1) * kCopies + c];
    }
    sums_begin(first, wsum[0]);
    __syncthreads();
    sums_end(first, wsum[0], h8);
    if (tid < 2) h8[kBins + tid] = 0;
    __syncthreads();
    uint32_t surely, perhaps;
    last_failing<kBins / kAllocThreads>(kBins - 8, [&](uint32_t b, bool &over, bool &may) {
      const uint32_t b4 = tied4_of(b << 20) >> 20;
      uint64_t c_min = 2ull * J + 4ull * h8[b] + 2ull * h8[b4 + 1], c_max = 2ull * J + 4ull * h8[b] + 2ull * h8[b4];
      if (ALLOW16) {
        const uint32_t b16 = tied16_of(b << 20) >> 20;
        c_min += 8ull * h8[b16 + 1];
        c_max += 8ull * h8[b16];
      }
      over = c_min > max_code_bits;
      may = c_max > max_code_bits;
    }, wfit, surely, perhaps);
    lo = surely << 20;
    hi = (perhaps + 1) << 20;
    lo4 = tied4_of(lo) >> 20 << 20;
    hi4 = ((tied4_of(hi) >> 20) + 1) << 20;
    uint32_t base8 = h8[hi >> 20], base4 = h8[hi4 >> 20], base16 = 0;  // norms at or above the brackets
    if (ALLOW16) {
      lo16 = tied16_of(lo) >> 20 << 20;
      hi16 = ((tied16_of(hi) >> 20) + 1) << 20;
      base16 = h8[hi16 >> 20];
    }

    base = 2 * J + 4 * base8 + 2 * base4 + 8 * base16;  // cost at hi, but for the tied norms between its tied thresholds and the bins' ends
    at_lo = h8[lo >> 20] + h8[lo4 >> 20];
    at_hi = base8 + base4;
    cost_lo = 2 * J + 4 * h8[lo >> 20] + 2 * h8[lo4 >> 20];
    if (ALLOW16) {
      at_lo += h8[lo16 >> 20];
      cost_lo += 8 * h8[lo16 >> 20];
      at_hi += base16;
    }
    __syncthreads();  // everybody has read the counts
  }
  // Looking at every norm takes a level some 4 us for 51,200, though few of them lie in the brackets: the threads set theirs aside first and the levels
  // look at those.  Where more than a tenth are inside (norms within a factor of two of each other, masses of equal ones), or one thread has more of its
  // up to 64 inside than fit, the bracket is halved by exact counts: until a tenth is left, or to its end.  Up to 16 norms per thread always fit, and the levels take up
  // to 8 per thread in less time than the counts, half a us to a round of some twenty: an allocation of 8 norms 8.1 us, with a tenth there too 20.6; of 1,000 equal
  // ones 11.4 and 20.3, of 8,192 24.9 and 24.1, of 16,384 (the other way here) 41 and 30.  More: three per thread are as good as a tenth or better.
  uint32_t n_kept = 0;
  const uint32_t budget = (uint32_t)min(max_code_bits, (uint64_t)0xFFFFFFFFu);
  bool fits = true, last_fit = false;
  for (uint32_t probe = 0; hi - lo > 1; ++probe) {
    const uint32_t turn = probe & 1u;
    if (fits && at_lo - at_hi <= (ASIDE ? max(J / 10, 3u * kAllocThreads) : 8u * kAllocThreads)) {
      const uint32_t width = hi - lo, width4 = hi4 - lo4, width16 = hi16 - lo16;
      n_kept = 0;
      each_norm([&](int k) {
        if (!ASIDE && k >= 16) return;
        const uint32_t v = (uint32_t)fr[k];
        kept[ASIDE ? min(n_kept, kKept) : n_kept][tid] = v;
        n_kept += ((v - lo < width) | (v - lo4 < width4) | (ALLOW16 && v - lo16 < width16)) ? 1u : 0u;
      });
      if (!ASIDE) break;
      fits = !__syncthreads_or(n_kept > kKept);
      if (fits) break;
    }
    // The first three where the cost would meet the budget if it fell evenly; the second and third a little to the side on which the one before was not,
    // so that they close the bracket from there.  (Halved only: 51,200 norms within a tenth 34.8 us instead of 28.2, half of them equal 74.5 and 63.3; equal ones
    // all, which fall at one place, 60.4 and 62.4.)
    const uint32_t width = hi - lo;
    uint32_t mid = lo + width / 2;
    if (probe < 3 && lo && cost_lo > budget && base <= budget) {  // (beyond the budget where norms are infinite and even +inf is too dear)
      const int32_t even = (int32_t)((float)width * ((float)(cost_lo - budget) / (float)(cost_lo - base))), off = (int32_t)(width >> (probe == 1 ? 5 : 4));
      mid = lo + (uint32_t)min(max(probe == 0 ? even : last_fit ? even - off : even + off, 1), (int32_t)width - 1);
    }
    const uint32_t p4 = tied4_of(mid), p16 = ALLOW16 ? tied16_of(mid) : 0u;
    uint32_t n8 = 0, n4 = 0, n16 = 0;
    each_norm([&](int k) {  // per lane: ballots, whose bits the scalar unit counts, take twice as long
      n8 += fr[k] >= (int32_t)mid ? 1u : 0u;
      n4 += fr[k] >= (int32_t)p4 ? 1u : 0u;
      if (ALLOW16) n16 += fr[k] >= (int32_t)p16 ? 1u : 0u;
    });
    n8 = wave_scan(n8);
    n4 = wave_scan(n4);
    if (ALLOW16) n16 = wave_scan(n16);
    if (lane == 63) {
      exact[turn][0][wave] = n8;
      exact[turn][1][wave] = n4;
      exact[turn][2][wave] = n16;
    }
    __syncthreads();
    n8 = __builtin_amdgcn_readlane(row_scan(exact[turn][0][lane & 15u]), 15);
    n4 = __builtin_amdgcn_readlane(row_scan(exact[turn][1][lane & 15u]), 15);
    if (ALLOW16) n16 = __builtin_amdgcn_readlane(row_scan(exact[turn][2][lane & 15u]), 15);
    const uint32_t cost = 2 * J + 4 * n8 + 2 * n4 + 8 * n16;
    last_fit = cost <= budget;
    if (last_fit) {
      hi = mid;
      hi4 = p4;
      hi16 = p16;
      base = cost;
      at_hi = n8 + n4 + n16;
    } else {
      lo = mid;
      lo4 = p4;
      lo16 = p16;
      at_lo = n8 + n4 + n16;
      cost_lo = cost;
    }
  }
  Bracket bracket = {lo, hi, lo4, hi4, lo16, hi16, base, n_kept};
  to_one_pattern<ALLOW16>(bracket, budget, S, NoEvents());
  hi = bracket.hi;
  // How many norms of each row are at or above the thresholds; the first wave turns that into the rows' first places.
  const int32_t p8 = (int32_t)hi, p4 = p4_from(hi), p16 = p16_from(hi, ALLOW16);
  uint32_t n4 = 0, n8 = 0, n16 = 0;  // lane g: of the wave's norms in group g
  each_group([&](int g) {
    uint32_t g4 = 0, g8 = 0, g16 = 0;
#pragma unroll
    for (int k = 4 * g; k < 4 * g + 4; ++k) {
      g4 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= p4));
      g8 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= p8));
      if (ALLOW16) g16 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= p16));
    }
    n4 = lane == (uint32_t)g ? g4 : n4;
    n8 = lane == (uint32_t)g ? g8 : n8;
    if (ALLOW16) n16 = lane == (uint32_t)g ? g16 : n16;
  });
  if (lane < kRegs / 4) {
    uint32_t *const row = row_n[4 * lane + wave / 4];
    atomicAdd(row, n4);
    atomicAdd(row + 1, n8);
    if (ALLOW16) atomicAdd(row + 2, n16);
  }
  __syncthreads();
  return hi;
}

// In lane k: the first place of every class in row k.  In all lanes: the classes' sizes.
struct RowPlaces {
  uint32_t first[4], n_class[4];
};
__device__ __forceinline__ RowPlaces row_places(uint32_t J, const SearchSpace &S) {
  const uint32_t lane = threadIdx.x & 63u, from = lane * kAllocThreads, in_row = J > from ? min(J - from, (uint32_t)kAllocThreads) : 0u;
  const uint32_t r4 = S.row_n[lane][0], r8 = S.row_n[lane][1], r16 = S.row_n[lane][2];
  const uint32_t x[4] = {in_row - r4, r4 - r8, r8 - r16, r16};
  RowPlaces p;
  uint32_t class_first = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t upto = wave_scan(x[c]);
    p.n_class[c] = __builtin_amdgcn_readlane(upto, 63);
    p.first[c] = class_first + upto - x[c];
    class_first += p.n_class[c];
  }
  return p;
}
// Widths and positions by a block that has searched for itself: its row's super-group of norm f, one per thread.
// from_end: the last row, whose places end where the classes do (search_lists does not count it by itself).
__device__ __forceinline__ Placed place_searched(float f, bool there, uint32_t row, uint32_t pattern, bool allow16, const RowPlaces &p,
                                                 uint32_t (*mine_w)[4], bool from_end = false) {
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t first[4];  // as lane `row` says it
#pragma unroll
  for (int c = 0; c < 4; ++c) first[c] = (uint32_t)__builtin_amdgcn_readlane((int)p.first[c], (int)row);
  const int32_t p8 = (int32_t)pattern, p4 = p4_from(pattern), p16 = p16_from(pattern, allow16);
  const uint32_t k = there ? class_of(pattern_of(f), p4, p8, p16) : 4u;
  const uint64_t b[4] = {__ballot(k == 0), __ballot(k == 1), __ballot(k == 2), __ballot(k == 3)};
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < 4; ++c) mine_w[wave][c] = (uint32_t)__builtin_popcountll(b[c]);
  }
  uint32_t at = k == 0 ? first[0] : k == 1 ? first[1] : k == 2 ? first[2] : first[3];
  __syncthreads();
  if (k == 4) return Placed{4u, 0u};
  if (from_end) {
    at = 0;
    for (uint32_t c = 0; c < 4; ++c) at += c <= k ? p.n_class[c] : 0u;
    for (uint32_t w = 0; w < kAllocWaves; ++w) at -= mine_w[w][k];
  }
  for (uint32_t w = 0; w < wave; ++w) at += mine_w[w][k];
  const uint64_t mine = k == 0 ? b[0] : (k == 1 ? b[1] : (k == 2 ? b[2] : b[3]));
  return Placed{k, at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u))};
}
__device__ __forceinline__ void tell(const uint32_t (&n)[4], const dq::Announce &announce, uint32_t bucket) {
  if (announce.host)  // one store, so that nothing needs to be ordered; the fourth class is the rest
    __hip_atomic_store(announce.host + bucket, n[0] | (uint64_t)n[1] << 17 | (uint64_t)n[2] << 34 | (uint64_t)announce.tag << 51, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void put_counts(const uint32_t (&n)[4], uint32_t T, uint32_t *cnt, const dq::Announce &announce, uint32_t bucket) {
#pragma unroll
  for (int c = 0; c < 4; ++c) gst<uint32_t>(cnt + c, n[c]);
  gst<uint32_t>(cnt + 4, T);
  tell(n, announce, bucket);
}

// A search's results, by its first wave: every row's first places where the row's own positions go, the counts, the threshold.
__device__ __forceinline__ void put_search(uint32_t J, uint32_t T, const SearchSpace &S, uint32_t *pos, uint32_t *cnt, const dq::Announce &announce) {
  const RowPlaces p = row_places(J, S);
  const uint32_t from = threadIdx.x * kAllocThreads;
  if (from + kAllocThreads < J) {  // not the last row
#pragma unroll
    for (int c = 0; c < 4; ++c) gst<uint32_t>(pos + from + c, p.first[c]);
  }
  if (threadIdx.x == 0) put_counts(p.n_class, T, cnt, announce, blockIdx.x);
}

template <bool ALLOW16, bool ASIDE>
__global__ void __launch_bounds__(kAllocThreads) k_search(const float *F_all, uint32_t J, uint64_t max_code_bits, uint32_t *pos_all,
                                                          uint32_t *counts_all, dq::Announce announce) {
  __shared__ SearchSpace S;
  const uint32_t T = search_block<ALLOW16, ASIDE>(F_all + (uint64_t)blockIdx.x * J, J, max_code_bits, S);
  if (threadIdx.x < 64) put_search(J, T, S, pos_all + (uint64_t)blockIdx.x * J, counts_all + 5ull * blockIdx.x, announce);
}

// ---------------------------------------------------------------------------------------
// Buckets of 40 rows and more at 2, 4 and 8 bits, few enough that a block for each of their rows has a CU: what takes the search above most of its time, looking at every
// norm to find the tenth of them that matters, in a launch of its own on as many CUs as there are rows (k_list), the rest by every row's block behind it
// (k_search_positions) or by one (k_search_listed).  Every block of k_list brackets the threshold by itself, from the same sample of 8,192 norms and bins of 2^18 patterns, four standard
// deviations of the sampled cost to either side, and lists what its own 1,024 norms cost up to where inside the bracket, with how many lie above.  A list
// goes to memory of its own, or where the row's positions go (the last whole row's block also has what follows it, up to 1,023 norms).  Sums over the lists' heads are exact: where the
// threshold is not inside the bracket (norms in an order that the sample's steps meet) a block searches as without lists.  Rows with more inside than their list holds
// it looks at itself, up to 16; where there are more, it goes on as before from the bracket, whose costs are known.
// What bounds both is their chains, 6 to 8 us each.  Kernels' time for 51,200 norms, one search -> both: lognormal 18.6 -> 12.5, sorted 20.2 -> 20.7, rows of
// like norms 18.8 -> 17.6, within a factor of two of each other 22.4 -> 20.3, within a tenth 27.2 -> 27.6, equal 56.8 -> 51.8 (a bucket's statistics and
// allocation 76.1 -> 69.6, search and positions in one launch).  Not with 16-bit widths, whose brackets are wider (20.9 -> 21.2), nor below some 41,000 norms, where all in one launch, which the host enqueues
// sooner, is the better (statistics and allocation, one launch and listed in three: 2 workers' 33,000 28.2 and 31.0, 40,000 30.6 and 30.7, 4 workers' 50,000 44.9 and 41.4; all-reduces
// over 6 of 30,000 62.5 and 64.2, over 8 of 42,664 88.9 and 86.9, the listed ones with k_arrange apart, 1.5 more than now).  An all-reduce of one bucket has
// the second part in every block of its next launch (k_search_arrange).
// Beside a replay the short blocks of k_list and one block behind them hold up less than the search by one block (51,200 norms and a 25 MB replay, enqueued in turn, 51.9 us
// a pair and 53.2; the replay alone 50.4).
constexpr uint32_t kSample = 8192, kFine = 18, kFineBins = 8192;  // bins of 2^18 patterns: 0x7F8 << 2 of them are finite
struct ListHead {
  uint32_t n;                        // events, or kTooLong: more than the list holds
  uint32_t above8, above4, in8, in4;  // norms at or above the brackets' ends, and inside
  uint32_t lo, hi;
};
constexpr uint32_t kListHead = 8, kListMost = kAllocThreads - kListHead, kTooLong = 0xFFFFFFFFu;
static_assert(sizeof(ListHead) <= 4 * kListHead, "");

__global__ void __launch_bounds__(kAllocThreads) k_list(const float *F_all, uint32_t J, uint64_t max_code_bits, uint32_t *lists_all) {
  __shared__ alignas(16) uint32_t counters[kFineBins + 4];
  __shared__ uint32_t wsum[kAllocWaves], wfit[kAllocWaves], found[kAllocWaves][4];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float *F = F_all + (uint64_t)blockIdx.y * J;
  uint32_t *list = lists_all + (uint64_t)blockIdx.y * J + (uint64_t)blockIdx.x * kAllocThreads;
  float sample[kSample / kAllocThreads], own[2];
#pragma unroll
  for (uint32_t i = 0; i < kSample / kAllocThreads; ++i) sample[i] = gld<float>(F + (uint32_t)(((uint64_t)(i * kAllocThreads + tid) * J) / kSample));
  const uint32_t j0 = blockIdx.x * kAllocThreads + tid, j1 = blockIdx.x + 1 == gridDim.x ? j0 + kAllocThreads : J;
  own[0] = gld<float>(F + j0);
  own[1] = j1 < J ? gld<float>(F + j1) : 0.0f;
  for (uint32_t b = tid; b < kFineBins / 4; b += kAllocThreads) reinterpret_cast<uint4 *>(counters)[b] = make_uint4(0, 0, 0, 0);
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kSample / kAllocThreads; ++i) {
    const uint32_t bin = (uint32_t)pattern_of(sample[i]) >> kFine, one = __builtin_amdgcn_readfirstlane(bin);
    const bool all = __ballot(bin == one) == ~0ull;  // norms that are equal do not queue
    if (!all || lane == 0) atomicAdd(counters + bin, all ? 64u : 1u);
  }
  __syncthreads();
  OwnBins<kFineBins> first;
#pragma unroll
  for (uint32_t i = 0; i < kFineBins / kAllocThreads; ++i) first.n[i] = counters[kFineBins / kAllocThreads * tid + i];
  sums_begin(first, wsum);
  __syncthreads();
  sums_end(first, wsum, counters);
  if (tid < 4) counters[kFineBins + tid] = 0;
  __syncthreads();
  // the budget above 2 bits a norm, for the sample, and what the sample's cost may be off: its variance is at most (mean)(most - mean) per norm
  constexpr float kMost = 6.0f;
  const float mean = min((float)(max_code_bits - 2ull * J) / (float)J, kMost), budget = mean * (float)kSample;
  const float off = 4.0f * __builtin_sqrtf(mean * (kMost - mean) * (float)kSample) + kMost;
  uint32_t surely, perhaps;
  last_failing<kFineBins / kAllocThreads>(0x7F800000u >> kFine, [&](uint32_t b, bool &over, bool &may) {
    const uint32_t b4 = tied4_of(b << kFine) >> kFine;
    over = (float)(4 * counters[b] + 2 * counters[b4 + 1]) > budget + off;
    may = (float)(4 * counters[b] + 2 * counters[b4]) > budget - off;
  }, wfit, surely, perhaps);
  const uint32_t lo = surely << kFine, hi = (perhaps + 1) << kFine, lo4 = tied4_of(lo), hi4 = tied4_of(hi);
  uint32_t event[2][2], at[2][2], n_in[2] = {0, 0}, above[2] = {0, 0};
  bool in[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const bool there = i == 0 || j1 < J;
    const uint32_t v = (uint32_t)pattern_of(own[i]);
#pragma unroll
    for (int kind = 0; kind < 2; ++kind) {
      const uint32_t from = kind == 0 ? lo : lo4, to = kind == 0 ? hi : hi4;
      in[i][kind] = there && v - from < to - from;
      uint32_t upto = v;
      if (kind == 1 && in[i][kind]) upto = last_tied(v, 17.0f / 512.0f, 512.0f / 17.0f, lo, hi);
      event[i][kind] = event_of(kind, upto - lo);
      const uint64_t inside = __ballot(in[i][kind]);
      at[i][kind] = n_in[0] + n_in[1] + __builtin_amdgcn_mbcnt_hi((uint32_t)(inside >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)inside, 0u));
      n_in[kind] += (uint32_t)__builtin_popcountll(inside);
      above[kind] += (uint32_t)__builtin_popcountll(__ballot(there && v >= to));
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int kind = 0; kind < 2; ++kind) {
      found[wave][kind] = n_in[kind];
      found[wave][2 + kind] = above[kind];
    }
  }
  __syncthreads();
  uint32_t all[4], before = 0;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint32_t upto = row_scan(found[lane & 15u][c]);
    all[c] = __builtin_amdgcn_readlane(upto, 15);
    if (c < 2) before += (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)wave) - n_in[c];
  }
  const bool too_long = all[0] + all[1] > kListMost || hi - lo > kMostAbove;
  if (tid == 0) {
    const ListHead head = {too_long ? kTooLong : all[0] + all[1], all[2], all[3], all[0], all[1], lo, hi};
    struct Words { uint32_t w[sizeof(ListHead) / 4]; };
    const Words words = __builtin_bit_cast(Words, head);
#pragma unroll
    for (uint32_t i = 0; i < sizeof(ListHead) / 4; ++i) gst<uint32_t>(list + i, words.w[i]);
  }
  if (too_long) return;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int kind = 0; kind < 2; ++kind)
      if (in[i][kind]) gst<uint32_t>(list + kListHead + before + at[i][kind], event[i][kind]);
}

// From the lists: T, and how many norms of each row are at or above the thresholds, in S.row_n.
__device__ __forceinline__ uint32_t search_lists(const float *F, const uint32_t *lists, uint32_t J, uint64_t max_code_bits, SearchSpace &S) {
  constexpr uint32_t kPerWave = kRegs / kAllocWaves, kAtOnce = 128;  // lists per wave; of each, events asked for before its length is known
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6), n_lists = J / kAllocThreads;
  struct Words { uint32_t w[sizeof(ListHead) / 4]; } words;
#pragma unroll
  for (uint32_t i = 0; i < sizeof(ListHead) / 4; ++i) words.w[i] = gld<uint32_t>(lists + min(lane, n_lists - 1) * kAllocThreads + i);
  const ListHead head = __builtin_bit_cast(ListHead, words);
  uint32_t ahead[kPerWave][kAtOnce / 64];
#pragma unroll
  for (uint32_t i = 0; i < kPerWave; ++i) {
    const uint32_t *list = lists + min(wave + i * kAllocWaves, n_lists - 1) * kAllocThreads + kListHead;
#pragma unroll
    for (uint32_t k = 0; k < kAtOnce / 64; ++k) ahead[i][k] = gld<uint32_t>(list + k * 64 + lane);
  }
  reinterpret_cast<uint4 *>(S.places)[tid] = make_uint4(0, 0, 0, 0);
  S.last_places[tid] = S.last_places[tid + kAllocThreads] = 0;
  if (tid == 0) S.places[kPlaces] = 0;
  const bool there = lane < n_lists;
  auto sum = [&](uint32_t x) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan(there ? x : 0u), 63); };
  const uint32_t all8 = sum(head.above8), all4 = sum(head.above4), all_in8 = sum(head.in8), all_in4 = sum(head.in4);
  Bracket bracket = {};
  bracket.lo = __builtin_amdgcn_readfirstlane(head.lo);
  bracket.hi = __builtin_amdgcn_readfirstlane(head.hi);
  bracket.lo4 = tied4_of(bracket.lo);
  bracket.hi4 = tied4_of(bracket.hi);
  bracket.base = 2 * J + 4 * all8 + 2 * all4;
  const uint32_t budget = (uint32_t)min(max_code_bits, (uint64_t)0xFFFFFFFFu), cost_lo = bracket.base + 4 * all_in8 + 2 * all_in4;
  if (bracket.base > budget || (bracket.lo && cost_lo <= budget)) {  // not inside
    __syncthreads();
    return search_block<false, true>(F, J, max_code_bits, S);
  }
  const uint64_t dense = __ballot(there && head.n == kTooLong);  // rows whose norms are looked at themselves
  const bool tail = J % kAllocThreads != 0 && dense >> (n_lists - 1) & 1u;  // what follows the last of them is a row more
  const uint32_t n_dense = (uint32_t)__builtin_popcountll(dense) + (tail ? 1u : 0u);
  // what a list has beyond the first kAtOnce goes to S.room
  const uint32_t n_in = there && head.n != kTooLong ? head.n : 0u, longer = n_in > kAtOnce ? n_in - kAtOnce : 0u;
  const uint32_t upto = wave_scan(longer), all = __builtin_amdgcn_readlane(upto, 63);
  if (all + n_dense * kAllocThreads > 16u * kAllocThreads) {
    const Given given = {bracket.lo, bracket.hi, all8 + all4 + all_in8 + all_in4, all8 + all4, cost_lo, bracket.base};
    __syncthreads();
    return search_block<false, true>(F, J, max_code_bits, S, given);
  }
  uint32_t n[kPerWave];  // of the wave's lists
#pragma unroll
  for (uint32_t i = 0; i < kPerWave; ++i) {
    const uint32_t l = wave + i * kAllocWaves, len = (uint32_t)__builtin_amdgcn_readlane((int)n_in, (int)(l & 63u));
    n[i] = l < n_lists ? len : 0u;
  }
  for (uint64_t more = __ballot(longer != 0); more;) {  // by all threads, four lists at a time
    uint32_t to[4], event[4];
    bool in[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t l = (uint32_t)__builtin_ctzll(more | 1ull << 63), len = more ? (uint32_t)__builtin_amdgcn_readlane((int)longer, (int)l) : 0u;
      to[i] = n_dense * kAllocThreads + (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)l) - len + tid;
      in[i] = tid < len;
      event[i] = in[i] ? gld<uint32_t>(lists + l * kAllocThreads + kListHead + kAtOnce + tid) : 0u;
      more &= more - 1;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (in[i]) S.room[to[i]] = event[i];
  }
  uint32_t n_rows = 0;
  for (uint64_t more = dense; more;) {
    float f[4];
    uint32_t some = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t l = (uint32_t)__builtin_ctzll(more | 1ull << 63);
      f[i] = more ? gld<float>(F + l * kAllocThreads + tid) : 0.0f;
      some += more ? 1u : 0u;
      more &= more - 1;
    }
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i)
      if (i < some) S.room[(n_rows + i) * kAllocThreads + tid] = (uint32_t)pattern_of(f[i]);
    n_rows += some;
  }
  if (tail) {
    const uint32_t j = n_lists * kAllocThreads + tid;
    S.room[n_rows * kAllocThreads + tid] = j < J ? (uint32_t)pattern_of(gld<float>(F + j)) : 0xFFFFFFFFu;
  }
  __syncthreads();
  const uint32_t *const longer_lists = S.room + n_dense * kAllocThreads;
  const uint32_t n_longer = all > tid ? (all - tid + kAllocThreads - 1) / kAllocThreads : 0u;
  bracket.n_kept = n_dense;
  const Bracket whole = bracket;
  to_one_pattern<false>(bracket, budget, S, [&](auto body) {
#pragma unroll
    for (uint32_t i = 0; i < kPerWave; ++i)
#pragma unroll
      for (uint32_t k = 0; k < kAtOnce / 64; ++k)
        if (k * 64 + lane < n[i]) body(ahead[i][k]);
    for (uint32_t i = 0; i < n_longer; ++i) body(longer_lists[i * kAllocThreads + tid]);
  });
  const uint32_t T = bracket.hi, p4 = tied4_of(T);
  uint32_t n4 = head.above4, n8 = head.above8;  // lane l: norms of row l at or above
#pragma unroll
  for (uint32_t i = 0; i < kPerWave; ++i) {
    uint32_t a4 = 0, a8 = 0;
    auto count = [&](bool valid, uint32_t event) {
      const bool reached = valid && whole.lo + upto_of(event) >= T;
      a8 += (uint32_t)__builtin_popcountll(__ballot(reached && kind_of(event) == 0));
      a4 += (uint32_t)__builtin_popcountll(__ballot(reached && kind_of(event) == 1));
    };
#pragma unroll
    for (uint32_t k = 0; k < kAtOnce / 64; ++k) count(k * 64 + lane < n[i], ahead[i][k]);
    if (n[i] > kAtOnce) {
      const uint32_t end = (uint32_t)__builtin_amdgcn_readlane((int)upto, (int)((wave + i * kAllocWaves) & 63u));
      for (uint32_t k = end - (n[i] - kAtOnce); k < end; k += 64) count(k + lane < end, longer_lists[min(k + lane, end - 1)]);
    }
    const bool mine = lane == wave + i * kAllocWaves;
    n4 += mine ? a4 : 0u;
    n8 += mine ? a8 : 0u;
  }
  if ((lane & (kAllocWaves - 1)) == wave) {  // the wave's rows; beyond the lists there is none
    S.row_n[lane][0] = there ? n4 : 0u;
    S.row_n[lane][1] = there ? n8 : 0u;
    S.row_n[lane][2] = 0;
  }
  __syncthreads();
  if (dense) {
    uint64_t more = dense;
    for (uint32_t i = 0; i < n_dense; ++i) {
      const uint32_t l = i < n_rows ? (uint32_t)__builtin_ctzll(more) : n_lists - 1, v = S.room[i * kAllocThreads + tid];
      more &= more - 1;
      const uint32_t a4 = (uint32_t)__builtin_popcountll(__ballot(v < whole.hi4 && v >= p4)), a8 = (uint32_t)__builtin_popcountll(__ballot(v < whole.hi && v >= T));
      if (lane == 0) {
        atomicAdd(&S.row_n[l][0], a4);
        atomicAdd(&S.row_n[l][1], a8);
      }
    }
    __syncthreads();
  }
  return T;  // (the last list's row has what follows it, too: of the row after it nobody reads the first places, and sums over all are the same)
}

// The lists lie in `pos`: for callers without other memory for them, beside other work, and for several buckets of an all-reduce (whose k_arrange is behind it).
__global__ void __launch_bounds__(kAllocThreads) k_search_listed(const float *F_all, uint32_t J, uint64_t max_code_bits, uint32_t *pos_all,
                                                                 uint32_t *counts_all, dq::Announce announce) {
  __shared__ SearchSpace S;
  uint32_t *pos = pos_all + (uint64_t)blockIdx.x * J;
  const uint32_t T = search_lists(F_all + (uint64_t)blockIdx.x * J, pos, J, max_code_bits, S);
  if (threadIdx.x < 64) put_search(J, T, S, pos, counts_all + 5ull * blockIdx.x, announce);
}

// Widths and positions by the blocks that search: grid (rows, buckets), every block searches for itself, on a CU that has nothing else to do, and then places its row.  Against a
// search in one block and the positions behind it, a launch and the places' trip to memory and back are fewer; the device's time and the
// host's are both less (statistics and allocation: 2 workers' 17,000 28.7 -> 26.4 us, 8 workers' 30,000 56.3 -> 53.7, of two buckets of 9,000 61.5 -> 59.3, 12 workers'
// 60,000 up to 16 bits 113.4 -> 111.7).  While there is a CU for every row: more would search one after the other.  (Buckets of one row keep the two launches that
// tests/test_launch_limits.py describes, though one is the better there, too: an allocation of 1,000 9.7 -> 8.1 us.)
// LISTED: behind k_list, the lists in memory of their own (a block writes its positions while another may still be reading).  Against k_search_listed and
// k_alloc_positions, 51,200 norms in one bucket 15.6 -> 14.7 us, in each of four 16.2 -> 14.6; 8 workers' statistics and allocation 63.7 -> 61.7, waited for
// 98.1 -> 94.7 (a search by one block 68.7 and 93.8: what is waited for behind eight launches is the host's, and a launch more its 4 us).
template <bool ALLOW16, bool ASIDE, bool LISTED>
__global__ void __launch_bounds__(kAllocThreads) k_search_positions(const float *F_all, const uint32_t *lists_all, uint32_t J, uint64_t max_code_bits,
                                                                    uint8_t *widths_all, uint32_t *pos_all, uint32_t *counts_all, dq::Announce announce) {
  static_assert(!LISTED || (ASIDE && !ALLOW16), "");
  __shared__ SearchSpace S;
  __shared__ uint32_t mine_w[kAllocWaves][4];
  const uint64_t first = (uint64_t)blockIdx.y * J;
  const uint32_t row = blockIdx.x, j = row * kAllocThreads + threadIdx.x;
  const float f = gld<float>(F_all + first + min(j, J - 1));
  uint32_t T;
  if constexpr (LISTED) T = search_lists(F_all + first, lists_all + first, J, max_code_bits, S);
  else T = search_block<ALLOW16, ASIDE>(F_all + first, J, max_code_bits, S);
  const RowPlaces p = row_places(J, S);
  if (row == 0 && threadIdx.x == 0) put_counts(p.n_class, T, counts_all + 5ull * blockIdx.y, announce, blockIdx.y);
  const Placed x = place_searched(f, j < J, row, T, ALLOW16, p, mine_w, LISTED && row == J / kAllocThreads);
  if (x.k < 4) {
    gst<uint8_t>(widths_all + first + j, (uint8_t)(2u << x.k));
    gst<uint32_t>(pos_all + first + j, x.at);
  }
}

// Behind the search of an all-reduce that replays on the original tensors: what k_alloc_positions and k_reorder_mean do between them, but for the
// widths and positions themselves, which nobody reads, and in the first blocks the replay's tables.
//
// The tables, as plan_walk and split_walk (dq_walk.hip) make them on the host: a thread per path, then the most tiles per wave of every width, then a
// share per thread; what is common to all shares every block works out for itself.  What bounds it is latency: a chain of 5.3 us, beside the other blocks' 3.6
// (8 workers, 8,192 super-groups, 4,096 shares; with all shares in one block, four to a thread, 6.1; the search's block doing this and the positions too: 8.7 behind the
// search).  Divisions are products with v_rcp_f32's
// result: that the fullest wave's tiles come out one more than they might be costs nothing but time, and any costs give shares that
// cover the tiles once, as a share ends where the next begins.  Sums of costs are whole numbers below 2^53, so doubles hold them exactly.
__device__ __forceinline__ float quick(float x) { return __builtin_amdgcn_rcpf(x); }

// Costs of a tile by width such that equal shares hold at most the bounded number of tiles (split_walk); by one wave.
__device__ __forceinline__ void raise_costs(const float (&tiles)[4], const dq::Costs &c, float waves, uint32_t lane, float (&cost)[4], float &fullest) {
  float each[4], most[4], all = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    each[w] = (float)c.of[w];
    all += tiles[w] * each[w];
  }
  const float mean = floorf(all * quick(waves)), step = 1.0f + floorf(mean * (1.0f / 64.0f));
  // Sums that come out a little high still fit: replays of tiles of one have a wave for each tile and hardly one over.  (Refused, waves took two tiles of the
  // cheapest width and others none: 32 workers' halving of 128 super-groups 46.1 us instead of 37.8, 26 workers' ring of 1,144 45.4 instead of 37.5.)
  const float most_waves = waves * (1.0f + 1e-6f);
  // the least cost of the fullest wave: 64 candidates at a time
  float s = 0.0f;
  for (float from = mean; ; from += 64.0f * step) {
    const float mine = from + step * (float)lane;
    float need = 0.0f;
    bool ok = true;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float k = floorf((mine + 0.5f) * quick(each[w]));
      ok = ok && (tiles[w] == 0.0f || k >= 1.0f);
      need += tiles[w] * quick(fmaxf(k, 1.0f));
    }
    const uint64_t fit = __ballot(ok && need <= most_waves);
    if (fit || from > all + 64.0f) {  // a wave that could take all of it: such a cost always fits four waves
      s = from + step * (float)(fit ? __builtin_ctzll(fit) : 63);
      break;
    }
  }
  fullest = 0.0f;
  float need = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    most[w] = fmaxf(floorf((s + 0.5f) * quick(each[w])), 1.0f);
    need += tiles[w] * quick(most[w]);
  }
  // each most as small as the waves allow, the dearest first
  bool done[4] = {tiles[0] == 0.0f, tiles[1] == 0.0f, tiles[2] == 0.0f, tiles[3] == 0.0f};
  for (int turn = 0; turn < 4; ++turn) {
    int at = -1;
    float dearest = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (!done[w] && most[w] * each[w] > dearest) {
        dearest = most[w] * each[w];
        at = w;
      }
#pragma unroll
    for (int w = 0; w < 4; ++w)
      if (w == at) {
        done[w] = true;
        const float others = need - tiles[w] * quick(most[w]), room = most_waves - others;
        if (room > 0.0f) {
          const float least = fmaxf(ceilf(tiles[w] * quick(room)), 1.0f);
          if (least < most[w]) most[w] = least;
        }
        need = others + tiles[w] * quick(most[w]);
      }
  }
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    cost[w] = each[w];
    if (tiles[w] != 0.0f) fullest = fmaxf(fullest, most[w] * each[w]);
  }
  for (int round = 0; round <= 8; ++round) {
    float share = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) share += tiles[w] * cost[w];
    share = round < 8 ? share * quick(waves) : fullest;
#pragma unroll
    for (int w = 0; w < 4; ++w) cost[w] = fmaxf(cost[w], share * quick(most[w]));
  }
}

__device__ __host__ __forceinline__ uint32_t table_parts(const dq::Tables &T) { return T.waves / kAllocThreads + 1; }  // a share per thread
struct TableSpace {
  double upto[dq::kMostTablePaths];  // cost of the paths before
  uint32_t tiles[dq::kMostTablePaths][4];
  uint32_t total[4], cost[4];
  double wave_sum[kAllocWaves];
};
// Path p's super-groups by width; count(b, w): of bucket b.
template <typename C>
__device__ __forceinline__ dq::WalkPath path_of(const dq::Tables &T, uint32_t p, C count) {
  const uint32_t b = T.by_chunk ? p % T.n_buckets : p / T.n_chunks, c = T.by_chunk ? p / T.n_buckets : p % T.n_chunks;
  const uint32_t lo = c * T.chunk_sgs, hi = lo + T.chunk_sgs;
  const uint64_t sg = (uint64_t)b * T.bucket_sgs + lo;
  dq::WalkPath x = {};
  x.job.local = reinterpret_cast<const void *>((uintptr_t)((uint64_t)b * T.bucket_sgs * kSG * T.entry_bytes));
  x.job.mu = T.mu ? T.mu + sg : nullptr;
  x.job.src = T.origin + sg;
  x.job.out = T.out + (uint64_t)b * T.bucket_sgs * kSG;
  x.job.dest = T.origin + sg;
  x.job.back = x.job.mu;
  x.job.first_sg = sg;
  x.chunk = c;
  uint32_t edge = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t end = edge + count(b, w), from = max(lo, edge), to = min(hi, end);
    x.job.n_sg[w] = to > from ? to - from : 0u;
    edge = end;
  }
  return x;
}
template <typename C>
__device__ __forceinline__ void make_tables(const dq::Tables &T, C count, uint32_t part, TableSpace &L) {
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t n_paths = T.n_chunks * T.n_buckets;
  if (T.slots) {  // every path has so many waves, a tile or none for each: nothing to be weighed, no barrier
    const uint32_t v = part * kAllocThreads + tid, p = v / T.slots, t = v - p * T.slots;
    const dq::WalkPath x = path_of(T, min(p, n_paths - 1), count);
    uint32_t tiles = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) tiles += (x.job.n_sg[w] + (1u << T.tile_log) - 1u) >> T.tile_log;
    if (p < n_paths && t == 0) T.paths[p] = x;
    if (v <= T.waves) T.shares[v] = p >= n_paths ? dq::WalkShare{n_paths, 0} : t < tiles ? dq::WalkShare{p, t} : dq::WalkShare{p + 1, 0};
    return;
  }
  if (tid < 4) L.total[tid] = 0;
  __syncthreads();
  uint32_t t[4] = {0, 0, 0, 0};
  if (wave * 64 < n_paths) {
    const dq::WalkPath x = path_of(T, min(tid, n_paths - 1), count);
    if (tid < n_paths) {
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        t[w] = (x.job.n_sg[w] + (1u << T.tile_log) - 1u) >> T.tile_log;
        L.tiles[tid][w] = t[w];
      }
      if (part == 0) T.paths[tid] = x;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t sum = __builtin_amdgcn_readlane(wave_scan(t[w]), 63);
      if (lane == 0) atomicAdd(&L.total[w], sum);
    }
  }
  __syncthreads();
  if (wave == 0) {
    float tiles[4], cost[4], fullest;
#pragma unroll
    for (int w = 0; w < 4; ++w) tiles[w] = (float)L.total[w];
    raise_costs(tiles, T.cost, (float)T.waves, lane, cost, fullest);
    const float unit = fullest < 16384.0f ? 65536.0f : 128.0f;
    if (lane < 4) L.cost[lane] = (uint32_t)ceilf(unit * (lane == 0 ? cost[0] : lane == 1 ? cost[1] : lane == 2 ? cost[2] : cost[3]));
  }
  __syncthreads();
  double mine = 0.0, sum;
#pragma unroll
  for (int w = 0; w < 4; ++w) mine += (double)t[w] * (double)L.cost[w];
  sum = mine;
  if (wave * 64 < n_paths) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const double up = __shfl_up(sum, d, 64);
      if (lane >= (uint32_t)d) sum += up;
    }
  }
  if (lane == 63) L.wave_sum[wave] = sum;
  __syncthreads();
  double before = 0.0, total = 0.0;
#pragma unroll
  for (int w = 0; w < kAllocWaves; ++w) {
    before += (uint32_t)w < wave ? L.wave_sum[w] : 0.0;
    total += L.wave_sum[w];
  }
  if (tid < n_paths) L.upto[tid] = before + sum - mine;
  __syncthreads();
  const double ratio = total / (double)T.waves;
  const uint32_t v = part * kAllocThreads + tid;
  if (v <= T.waves) {
    uint32_t path = n_paths, tile = 0;
    if (v < T.waves) {
      const double want = floor((double)v * ratio);
      path = 0;
      for (uint32_t span = n_paths; span > 1;) {  // the last path that begins at or before `want`
        const uint32_t half = span / 2;
        if (L.upto[path + half] <= want) path += half;
        span -= half;
      }
      double rest = want - L.upto[path];
      bool found = false;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t n = L.tiles[path][w];
        const double each = (double)L.cost[w];
        if (!found && n) {
          // a thousandth of a tile short counts as reached: where the costs fill the shares to the last tile, their rounding would leave a wave out
          if (rest <= ((double)(n - 1) + 1.0 / 1024.0) * each) {
            tile += min((uint32_t)ceil(fmax(0.0, rest / each - 1.0 / 1024.0)), n - 1);
            found = true;
          } else {
            rest = fmax(0.0, rest - (double)n * each);
            tile += n;
          }
        }
      }
      if (!found) {  // within the path's last tile
        ++path;
        tile = 0;
      }
    }
    T.shares[v] = dq::WalkShare{path, tile};
  }
}

__global__ void __launch_bounds__(kAllocThreads) k_arrange(const float *F_all, const float *mu_all, uint32_t J, bool allow16, const uint32_t *counts_all,
                                                           const uint32_t *places_all, float *mu_main, uint32_t *origin, dq::Tables T) {
  __shared__ uint32_t mine_w[kAllocWaves][4];
  __shared__ TableSpace space;
  const uint32_t parts = table_parts(T);
  if (blockIdx.x < parts) {
    if (blockIdx.y == 0) make_tables(T, [&](uint32_t b, int w) { return gld<uint32_t>(counts_all + 5ull * b + w); }, blockIdx.x, space);
    return;
  }
  const uint32_t row = blockIdx.x - parts;
  const uint64_t first = (uint64_t)blockIdx.y * J;
  const uint32_t j = row * kAllocThreads + threadIdx.x;
  const float m = mu_all ? gld<float>(mu_all + first + min(j, J - 1)) : 0.0f;
  const Placed x = place_row(F_all + first, J, allow16, counts_all + 5ull * blockIdx.y, places_all + first, row, row + parts + 1 == gridDim.x, mine_w);
  if (x.k < 4) {
    if (mu_all) gst<float>(mu_main + first + x.at, x.k == 3 ? 0.0f : m);
    gst<uint32_t>(origin + first + x.at, j);
  }
}

// The search and k_arrange in one launch, for one bucket: every block searches for itself, which costs nothing but a CU that has
// nothing else to do, and goes on with what it has in LDS.  Against two launches, a launch's start and the trips of places and counts to memory and back
// are fewer: 8 workers' 8,192 super-groups 8.2 and 5.2 us -> 9.6, 6 workers' 48 6.9 and 5.1 -> 7.8 (all-reduces 36.1 -> 31.9, 23.2 -> 21.9; 16 workers' halving
// of 1,312 31.5 -> 27.9, 3 workers' 15,000 30.6 -> 27.4, 4 workers' 17,980 36.5 -> 32.5).  What bounds it is the search's chain, whose every piece of code is fetched and run once.
// LISTED: behind k_list, against k_search_listed and k_arrange as launches of their own (all-reduces over 8 of 42,664 94.1 -> 92.6 us, 6 of 48,000 82.1 -> 80.5,
// halving over 4 of 65,536 86.1 -> 84.5, 2 of 40,960 44.8 -> 43.4).
template <bool ALLOW16, bool ASIDE, bool LISTED>
__global__ void __launch_bounds__(kAllocThreads) k_search_arrange(const float *F, const float *mu, const uint32_t *lists, uint32_t J, uint64_t max_code_bits,
                                                                  float *mu_main, uint32_t *origin, dq::Announce announce, dq::Tables T) {
  static_assert(!LISTED || (ASIDE && !ALLOW16), "");
  __shared__ SearchSpace S;
  __shared__ uint32_t mine_w[kAllocWaves][4];
  __shared__ TableSpace space;
  const uint32_t parts = table_parts(T), tid = threadIdx.x;
  const bool tables = blockIdx.x < parts;
  const uint32_t row = tables ? 0u : blockIdx.x - parts, j = row * kAllocThreads + tid;
  const float f = gld<float>(F + min(j, J - 1)), m = mu ? gld<float>(mu + min(j, J - 1)) : 0.0f;
  uint32_t pattern;
  if constexpr (LISTED) pattern = search_lists(F, lists, J, max_code_bits, S);
  else pattern = search_block<ALLOW16, ASIDE>(F, J, max_code_bits, S);
  const RowPlaces p = row_places(J, S);
  if (tables) {
    if (blockIdx.x == 0 && tid == 0) tell(p.n_class, announce, 0);
    make_tables(T, [&](uint32_t, int w) { return p.n_class[w]; }, blockIdx.x, space);
    return;
  }
  const Placed x = place_searched(f, j < J, row, pattern, ALLOW16, p, mine_w, LISTED && row == J / kAllocThreads);
  if (x.k == 4) return;
  if (mu) gst<float>(mu_main + x.at, x.k == 3 ? 0.0f : m);
  gst<uint32_t>(origin + x.at, j);
}

// Buckets of more than 65,536 super-groups: the norms are read again in every round of a bisection, widths and positions
// are written here, 64 rows of 1024 at a time.
__global__ void __launch_bounds__(kAllocThreads) k_allocate_large(const float *F_all, uint32_t J, uint64_t max_code_bits,
                                                            bool allow16, uint8_t *widths_all, uint32_t *pos_all,
                                                            uint32_t *counts_all) {
  __shared__ uint32_t red[2][3][kAllocWaves];
  __shared__ uint32_t tot[kRegs * kAllocWaves][4];  // per (row, wave): class counts, then their exclusive scan
  __shared__ uint32_t wsum[kAllocWaves][4];
  const float *F = F_all + (uint64_t)blockIdx.x * J;
  uint8_t *widths = widths_all + (uint64_t)blockIdx.x * J;
  uint32_t *pos = pos_all + (uint64_t)blockIdx.x * J;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t rows = (J + kAllocThreads - 1) / kAllocThreads;
  // Counts over the wave of super-groups at or above the thresholds.
  auto count = [&](int32_t p4, int32_t p8, int32_t p16, uint32_t &c4, uint32_t &c8, uint32_t &c16) {
    uint32_t a4 = 0, a8 = 0, a16 = 0;
    for (uint32_t j = tid; j < J; j += kAllocThreads) {
      const int32_t v = pattern_of(gld<float>(F + j));
      a4 += v >= p4 ? 1u : 0u;
      a8 += v >= p8 ? 1u : 0u;
      a16 += v >= p16 ? 1u : 0u;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      a4 += __shfl_xor(a4, d, 64);
      a8 += __shfl_xor(a8, d, 64);
      a16 += __shfl_xor(a16, d, 64);
    }
    c4 = a4; c8 = a8; c16 = a16;
  };
  // The waves' counts meet in LDS, in one of two buffers by turns, so that one barrier per round
  // is enough: a wave can only be one round ahead of the slowest reader.
  uint32_t turn = 0;
  auto block_counts = [&](uint32_t pattern, uint32_t &s4, uint32_t &s8, uint32_t &s16) {
    uint32_t c4, c8, c16;
    count(p4_from(pattern), (int32_t)pattern, p16_from(pattern, allow16), c4, c8, c16);
    if (lane == 0) {
      red[turn][0][wave] = c4;
      red[turn][1][wave] = c8;
      red[turn][2][wave] = c16;
    }
    __syncthreads();
    s4 = 0; s8 = 0; s16 = 0;
#pragma unroll
    for (int w = 0; w < kAllocWaves; ++w) {
      s4 += red[turn][0][w];
      s8 += red[turn][1][w];
      s16 += red[turn][2][w];
    }
    turn ^= 1u;
  };
  // Wanted: the smallest fp32 pattern in [1, +inf] whose allocation fits (the host has checked
  // 2J <= budget).  An SG at or above T_{4,8} is also at or above T_{2,4}, so
  // cost = 2J + 2*c4 + 4*c8, which never increases with the threshold: bisection from any
  // bracket (lo does not fit or is 0, hi fits) ends at the same pattern.
  uint32_t lo = 0, hi = 0x7F800000u;
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    uint32_t s4, s8, s16;
    block_counts(mid, s4, s8, s16);
    const uint64_t cost = 2ull * J + 2ull * s4 + 4ull * s8 + 8ull * s16;
    if (cost <= max_code_bits) hi = mid; else lo = mid;
  }
  uint32_t s4, s8, s16;
  block_counts(hi, s4, s8, s16);
  const int32_t p8 = (int32_t)hi, p4 = p4_from(hi), p16 = p16_from(hi, allow16);
  const uint32_t n_class[4] = {J - s4, s4 - s8, s8 - s16, s16};
  // first position of each class in the reordered bucket, advanced chunk by chunk
  uint32_t next[4] = {0, n_class[0], n_class[0] + n_class[1], n_class[0] + n_class[1] + n_class[2]};

  // Positions of the stable reorder (buckets too large for registers), 64 rows of 1024 super-groups
  // at a time, the norms read again: the rank of a super-group inside its class is (members in
  // earlier rows and waves) + (members in lower lanes).
  for (uint32_t r0 = 0; r0 < rows; r0 += kRegs) {
    const uint32_t nr = min((uint32_t)kRegs, rows - r0);
    auto slot = [&](uint32_t k) -> int32_t {
      const uint32_t j = (r0 + k) * kAllocThreads + tid;
      return j < J ? pattern_of(gld<float>(F + j)) : -1;
    };
    // pass 1: class counts of every (row, wave)
    for (uint32_t k = 0; k < nr; ++k) {
      const uint32_t c = class_of(slot(k), p4, p8, p16);
      const uint64_t b0 = __ballot(c == 0), b1 = __ballot(c == 1), b2 = __ballot(c == 2), b3 = __ballot(c == 3);
      if (lane == 0) {
        tot[k * kAllocWaves + wave][0] = (uint32_t)__builtin_popcountll(b0);
        tot[k * kAllocWaves + wave][1] = (uint32_t)__builtin_popcountll(b1);
        tot[k * kAllocWaves + wave][2] = (uint32_t)__builtin_popcountll(b2);
        tot[k * kAllocWaves + wave][3] = (uint32_t)__builtin_popcountll(b3);
      }
    }
    __syncthreads();
    // pass 2: exclusive scan of the counts in (row, wave) order; thread e owns entry e
    uint32_t x[4], inc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      x[c] = tid < nr * kAllocWaves ? tot[tid][c] : 0u;
      inc[c] = x[c];
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t up = __shfl_up(inc[c], d, 64);
        if (lane >= (uint32_t)d) inc[c] += up;
      }
      if (lane == 63) wsum[wave][c] = inc[c];
    }
    __syncthreads();
    uint32_t chunk_total[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      uint32_t before = 0, all = 0;
#pragma unroll
      for (int w = 0; w < kAllocWaves; ++w) {
        const uint32_t t = wsum[w][c];
        before += (uint32_t)w < wave ? t : 0u;
        all += t;
      }
      chunk_total[c] = all;
      if (tid < nr * kAllocWaves) tot[tid][c] = next[c] + before + inc[c] - x[c];
    }
    __syncthreads();
    // pass 3: widths and positions, coalesced
    auto emit = [&](uint32_t k, int32_t v) {
      const uint32_t j = (r0 + k) * kAllocThreads + tid;
      const uint32_t c = class_of(v, p4, p8, p16);
      const uint64_t b0 = __ballot(c == 0), b1 = __ballot(c == 1), b2 = __ballot(c == 2), b3 = __ballot(c == 3);
      const uint64_t mine = c == 0 ? b0 : (c == 1 ? b1 : (c == 2 ? b2 : b3));
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
      if (c < 4) {
        gst<uint8_t>(widths + j, (uint8_t)(2u << c));
        gst<uint32_t>(pos + j, tot[k * kAllocWaves + wave][c] + rank);
      }
    };
    for (uint32_t k = 0; k < nr; ++k) emit(k, slot(k));
#pragma unroll
    for (int c = 0; c < 4; ++c) next[c] += chunk_total[c];
    __syncthreads();  // tot and wsum are reused by the next chunk
  }
  if (tid == 0) {
    uint32_t *cnt = counts_all + 5ull * blockIdx.x;
    gst<uint32_t>(cnt, n_class[0]);
    gst<uint32_t>(cnt + 1, n_class[1]);
    gst<uint32_t>(cnt + 2, n_class[2]);
    gst<uint32_t>(cnt + 3, n_class[3]);
    gst<uint32_t>(cnt + 4, hi);
  }
}

// ---------------------------------------------------------------------------------------
// Reorder and restore move whole super-groups in 16-byte pieces: piece c of the source
// belongs to super-group c / pps (pps = pieces per SG) and lands at the same offset inside
// the destination super-group.  Each thread moves kUnroll pieces per round, 1 KB apart, so a
// wave has 4 KB in flight.
constexpr int kUnroll = 4;

template <uint32_t PPS>  // 16-byte pieces per super-group: 64 (fp32) or 32 (bf16)
__global__ void __launch_bounds__(kThreads) k_reorder(const void *x_all, const uint32_t *pos_all, uint32_t J, void *out_all) {
  const uint64_t bucket_first = (uint64_t)blockIdx.y * J;  // blockIdx.y = bucket
  const uint8_t *x = static_cast<const uint8_t *>(x_all) + bucket_first * PPS * 16;
  uint8_t *out = static_cast<uint8_t *>(out_all) + bucket_first * PPS * 16;
  const uint32_t *pos = pos_all + bucket_first;
  const uint32_t n_pieces = J * PPS;
  const uint32_t stride = gridDim.x * kThreads * kUnroll;
  for (uint32_t base = blockIdx.x * kThreads * kUnroll + threadIdx.x; base < n_pieces; base += stride) {
    u32x4 d[kUnroll];
    uint32_t dst[kUnroll];
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      const uint32_t c = base + i * kThreads;
      if (c < n_pieces) {
        d[i] = gld<u32x4>(x + (uint64_t)c * 16);
        dst[i] = gld<uint32_t>(pos + c / PPS) * PPS + c % PPS;
      }
    }
#pragma unroll
    for (int i = 0; i < kUnroll; ++i)
      if (base + i * kThreads < n_pieces) gst<u32x4>(out + (uint64_t)dst[i] * 16, d[i]);
  }
}

// The means the main stage subtracts, in reordered order; zero for the 16-bit super-groups (the
// last counts[5b + 3] places of bucket b); and the inverse of the positions.  One thread per super-group.
__global__ void __launch_bounds__(kThreads) k_reorder_mean(const float *mu_all, const uint32_t *pos_all, const uint32_t *counts,
                                                           uint32_t J, float *mu_main, uint32_t *origin) {
  const uint64_t bucket_first = (uint64_t)blockIdx.y * J;
  const uint32_t n16 = counts ? gld<uint32_t>(counts + 5ull * blockIdx.y + 3) : 0u;
  for (uint32_t j = blockIdx.x * kThreads + threadIdx.x; j < J; j += gridDim.x * kThreads) {
    const uint32_t p = gld<uint32_t>(pos_all + bucket_first + j);
    if (mu_main) {
      const float m = gld<float>(mu_all + bucket_first + j);
      gst<float>(mu_main + bucket_first + p, (p < J - n16) ? m : 0.0f);
    }
    if (origin) gst<uint32_t>(origin + bucket_first + p, j);
  }
}

__global__ void __launch_bounds__(kThreads) k_restore(const float *sum_all, const uint32_t *pos_all, const float *mu_all,
                                                      float n, uint32_t J, float *out_all) {
  constexpr uint32_t pps = kSG * 4 / 16;
  const uint64_t bucket_first = (uint64_t)blockIdx.y * J;
  const uint8_t *sum = reinterpret_cast<const uint8_t *>(sum_all) + bucket_first * pps * 16;
  uint8_t *out = reinterpret_cast<uint8_t *>(out_all) + bucket_first * pps * 16;
  const uint32_t *pos = pos_all + bucket_first;
  const float *mu = mu_all ? mu_all + bucket_first : nullptr;  // in reordered order
  const uint32_t n_pieces = J * pps;
  const uint32_t stride = gridDim.x * kThreads * kUnroll;
  for (uint32_t base = blockIdx.x * kThreads * kUnroll + threadIdx.x; base < n_pieces; base += stride) {
    f32x4 d[kUnroll];
    float back[kUnroll];
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      const uint32_t c = base + i * kThreads;
      if (c < n_pieces) {
        const uint32_t p = gld<uint32_t>(pos + c / pps);
        d[i] = gld<f32x4>(sum + ((uint64_t)p * pps + c % pps) * 16);
        back[i] = mu ? n * gld<float>(mu + p) : 0.0f;
      }
    }
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
      const uint32_t c = base + i * kThreads;
      if (c < n_pieces) {
        f32x4 o = d[i];
        if (mu) { o.x = d[i].x + back[i]; o.y = d[i].y + back[i]; o.z = d[i].z + back[i]; o.w = d[i].w + back[i]; }
        gst<f32x4>(out + (uint64_t)c * 16, o);
      }
    }
  }
}

bool aligned(const void *p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

uint32_t compute_units() {
  int dev = 0, n_cu = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  return (uint32_t)n_cu;
}

// blocks per grid row: enough for the units of one row, at most the GPU's resident share
uint32_t stream_blocks(uint64_t units_per_block_round, uint64_t units, uint32_t rows = 1) {
  const uint32_t n_cu = compute_units();
  const uint64_t need = (units + units_per_block_round - 1) / units_per_block_round;
  const uint64_t cap = ((uint64_t)n_cu * 8 + rows - 1) / rows;  // 8 blocks of 256 threads per CU in all
  return (uint32_t)(need < 1 ? 1 : (need < cap ? need : cap));
}

// A launch has fewer than 2^32 threads.
constexpr uint32_t kMostBlocks = 0xFFFFFFFFu / kThreads;

dq_status launched() { return dq::hip_status(hipGetLastError()); }

}  // namespace

namespace dq {

dq_status stats_all(const void *const *tensors, uint32_t n_workers, dq_dtype dtype, uint64_t n_sg, float *mu, float *F, const void **grads,
                    hipStream_t s) {
  if (n_sg == 0) return DQ_OK;
  if (!tensors || !mu || !F || n_workers == 0 || (dtype != DQ_F32 && dtype != DQ_BF16)) return DQ_EINVAL;
  if (n_workers > kMostTensors) return DQ_EUNSUPPORTED;
  WorkerTensors W = {};
  for (uint32_t w = 0; w < n_workers; ++w) {
    if (!aligned(tensors[w], 16)) return DQ_EALIGN;
    W.x[w] = tensors[w];
  }
  const uint64_t n_tiles = (n_sg + 3) / 4, waves = n_workers > 4 ? compute_units() * (dtype == DQ_F32 ? 7ull : 11ull) : 0;  // as many as pay (k_stats_split)
  if (n_tiles * 2 <= waves) {
    uint32_t slots = (uint32_t)(waves / n_tiles < kMostSlots ? waves / n_tiles : kMostSlots);
    slots = slots < n_workers ? slots : n_workers;
    const uint32_t rounds = (n_workers + slots - 1) / slots;
    slots = (n_workers + rounds - 1) / rounds;
    const uint32_t tiles = slots < 4 ? 2 : 1;
    const auto split = dtype == DQ_F32 ? k_stats_split<float> : k_stats_split<uint16_t>;
    hipLaunchKernelGGL(split, dim3((uint32_t)((n_tiles + tiles - 1) / tiles)), dim3(64 * slots * tiles), tiles * n_workers * 4 * sizeof(float2), s, W,
                       n_workers, slots, tiles, n_sg, mu, F, grads);
    return launched();
  }
  const uint32_t blocks = stream_blocks(4 * (kThreads / 64), n_sg);
  const auto kernel = dtype == DQ_F32 ? k_stats_all<float> : k_stats_all<uint16_t>;
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kThreads), 0, s, W, n_workers, n_sg, mu, F, grads);
  return launched();
}

// Whether the rows of a bucket list their norms first (the threshold is where that pays against k_search_positions and k_search_arrange)
constexpr uint32_t kLeastListed = 40 * kAllocThreads;
static bool takes_lists(uint32_t J, uint32_t n_buckets, uint32_t max_width) {
  return max_width == 8 && J >= kLeastListed && J <= kMostSearched && (uint64_t)(J / kAllocThreads) * n_buckets <= compute_units();  // a CU for each list
}
static_assert(kMostSearched == (uint32_t)kRegs * kAllocThreads && kMostTablePaths <= (uint32_t)kAllocThreads, "a register per norm, a thread per path");
dq_status search(const float *F, uint32_t J, uint32_t n_buckets, uint64_t max_code_bits, uint32_t max_width, uint32_t *places, uint32_t *counts,
                 Announce announce, hipStream_t s) {
  const bool allow16 = max_width == 16, aside = J > 16u * kAllocThreads;
  auto kernel = aside ? (allow16 ? k_search<true, true> : k_search<false, true>) : (allow16 ? k_search<true, false> : k_search<false, false>);
  if (takes_lists(J, n_buckets, max_width)) {
    hipLaunchKernelGGL(k_list, dim3(J / kAllocThreads, n_buckets), dim3(kAllocThreads), 0, s, F, J, max_code_bits, places);
    const dq_status st = launched();
    if (st != DQ_OK) return st;
    kernel = k_search_listed;
  }
  hipLaunchKernelGGL(kernel, dim3(n_buckets), dim3(kAllocThreads), 0, s, F, J, max_code_bits, places, counts, announce);
  return launched();
}

// While there is a CU for every block (up to 64 rows and a few of tables): more would search one after the other, as a block's LDS leaves room for no other.
bool takes_search_arrange(uint32_t J, uint32_t n_buckets, const Tables &tables) {
  return n_buckets == 1 && J <= kMostSearched && (J + kAllocThreads - 1) / kAllocThreads + table_parts(tables) <= compute_units();
}
dq_status search_arrange(const float *F, const float *mu, uint32_t J, uint64_t max_code_bits, uint32_t max_width, uint32_t *places, float *mu_main,
                         uint32_t *origin, Announce announce, const Tables &tables, hipStream_t s) {
  auto kernel = J > 16u * kAllocThreads ? (max_width == 16 ? k_search_arrange<true, true, false> : k_search_arrange<false, true, false>)
                                        : (max_width == 16 ? k_search_arrange<true, false, false> : k_search_arrange<false, false, false>);
  if (takes_lists(J, 1, max_width)) {
    hipLaunchKernelGGL(k_list, dim3(J / kAllocThreads), dim3(kAllocThreads), 0, s, F, J, max_code_bits, places);
    const dq_status st = launched();
    if (st != DQ_OK) return st;
    kernel = k_search_arrange<false, true, true>;
  }
  hipLaunchKernelGGL(kernel, dim3((J + kAllocThreads - 1) / kAllocThreads + table_parts(tables)), dim3(kAllocThreads), 0, s, F, mu, places, J, max_code_bits,
                     mu_main, origin, announce, tables);
  return launched();
}

dq_status arrange(const float *F, const float *mu, uint32_t J, uint32_t n_buckets, uint32_t max_width, const uint32_t *counts, const uint32_t *places,
                  float *mu_main, uint32_t *origin, const Tables &tables, hipStream_t s) {
  const uint32_t rows = (J + kAllocThreads - 1) / kAllocThreads;
  hipLaunchKernelGGL(k_arrange, dim3(rows + table_parts(tables), n_buckets), dim3(kAllocThreads), 0, s, F, mu, J, max_width == 16, counts, places, mu_main, origin, tables);
  return launched();
}

}  // namespace dq

extern "C" {

dq_status dq_sg_stats(const void *x, dq_dtype dtype, uint64_t n_sg, float *mu_out, float *F_out, void *hip_stream) {
  if (n_sg == 0) return DQ_OK;
  if (!x || !mu_out || !F_out || (dtype != DQ_F32 && dtype != DQ_BF16)) return DQ_EINVAL;
  if (!aligned(x, 16) || !aligned(mu_out, 4) || !aligned(F_out, 4)) return DQ_EALIGN;
  hipStream_t s = (hipStream_t)hip_stream;
  constexpr uint32_t kPerBlock = 4 * (kThreads / 64);
  constexpr uint64_t kMost = (uint64_t)kMostBlocks * kPerBlock;  // from 2^28 super-groups on, 137 GB in bf16, several launches
  for (uint64_t first = 0; first < n_sg; first += kMost) {
    const uint64_t n = n_sg - first < kMost ? n_sg - first : kMost;
    const void *from = static_cast<const uint8_t *>(x) + first * kSG * (dtype == DQ_F32 ? 4 : 2);
    const dim3 grid((uint32_t)((n + kPerBlock - 1) / kPerBlock));
    if (dtype == DQ_F32) hipLaunchKernelGGL(k_stats<float>, grid, dim3(kThreads), 0, s, from, n, mu_out + first, F_out + first);
    else hipLaunchKernelGGL(k_stats<uint16_t>, grid, dim3(kThreads), 0, s, from, n, mu_out + first, F_out + first);
    const dq_status st = launched();
    if (st != DQ_OK) return st;
  }
  return DQ_OK;
}

dq_status dq_stats_combine(const float *mu_all, const float *F_all, uint32_t n_workers, uint64_t n_sg, float *mu,
                           float *F, void *hip_stream) {
  if (n_sg == 0) return DQ_OK;
  if (!mu_all || !F_all || !mu || !F || n_workers == 0) return DQ_EINVAL;
  if (!aligned(mu_all, 4) || !aligned(F_all, 4) || !aligned(mu, 4) || !aligned(F, 4)) return DQ_EALIGN;
  constexpr uint64_t kMost = (uint64_t)kMostBlocks * kThreads;
  for (uint64_t first = 0; first < n_sg; first += kMost) {
    const uint64_t count = n_sg - first < kMost ? n_sg - first : kMost;
    hipLaunchKernelGGL(k_combine, dim3((uint32_t)((count + kThreads - 1) / kThreads)), dim3(kThreads), 0, (hipStream_t)hip_stream,
                       mu_all + first, F_all + first, n_workers, n_sg, count, mu + first, F + first);
    const dq_status st = launched();
    if (st != DQ_OK) return st;
  }
  return DQ_OK;
}

int dqx_searches_and_arranges(uint32_t n_sg_per_bucket, uint32_t n_buckets, uint32_t waves) {
  dq::Tables tables = {};
  tables.waves = waves;
  return dq::takes_search_arrange(n_sg_per_bucket, n_buckets, tables);
}

dq_status dqx_stats_all(const void *const *tensors, uint32_t n_workers, dq_dtype dtype, uint64_t n_sg, float *mu, float *F,
                        void *hip_stream) {
  return dq::stats_all(tensors, n_workers, dtype, n_sg, mu, F, nullptr, (hipStream_t)hip_stream);
}

// Whether every row's block searches (k_search_positions).
static bool rows_search(uint32_t J, uint32_t n_buckets) {
  const uint32_t rows = (J + kAllocThreads - 1) / kAllocThreads;
  return rows > 1 && rows <= (uint32_t)kRegs && (uint64_t)rows * n_buckets <= compute_units();
}
// lists: memory for the rows' lists (dqx_allocate_lists), or null: they lie in `pos`, and a launch of its own overwrites them.
// beside: another stream's work has the chip, and no more than a CU of each bucket is taken for the search (lists of large buckets aside, whose blocks are short).
// Beside replays of 25 MB over 8 workers (50.3 us alone), one of each enqueued in turn, us a pair, every row's block searching -> so: 8,192 norms 52.6 -> 51.5,
// 16,384 53.9 -> 51.0, 30,000 56.2 -> 51.7, five buckets of them 59.1 -> 51.8, 51,200 (lists either way) 53.4 -> 52.7, in each of four buckets 58.5 -> 53.2, up to 16
// bits 61.0 -> 55.3; alone 9.7 and 12.0, 11.8 and 14.2, 16.0 and 18.8, 16.1 and 18.9, 15.0 and 16.8, 15.1 and 17.4, 23.2 and 25.2.
static dq_status allocate(const float *F, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint64_t max_code_bits, uint32_t max_width, uint8_t *widths,
                          uint32_t *pos, uint32_t *counts, uint32_t *lists, bool beside, dq::Announce announce, void *hip_stream) {
  if (n_sg_per_bucket == 0 || n_buckets == 0) return DQ_OK;
  if (!F || !widths || !pos || !counts || (max_width != 8 && max_width != 16)) return DQ_EINVAL;
  if (max_code_bits < 2ull * n_sg_per_bucket) return DQ_EINVAL;  // fewer than 2 code bits per coordinate
  if (!aligned(F, 4) || !aligned(pos, 4) || !aligned(counts, 4) || !aligned(lists, 4)) return DQ_EALIGN;
  hipStream_t s = (hipStream_t)hip_stream;
  const bool allow16 = max_width == 16;
  const uint32_t J = n_sg_per_bucket, rows = (J + kAllocThreads - 1) / kAllocThreads;
  for (uint32_t b0 = 0; b0 < n_buckets;) {  // the grid's second dimension holds 65,535; the counts are announced of fewer only
    const uint32_t nb = n_buckets - b0 < 65535u ? n_buckets - b0 : 65535u;
    const uint64_t off = (uint64_t)b0 * J;
    uint32_t *const cnt = counts + 5ull * b0;
    const bool listed = dq::takes_lists(J, nb, max_width);
    if (!beside && rows_search(J, n_buckets) && (lists || !listed)) {
      if (listed) {
        hipLaunchKernelGGL(k_list, dim3(J / kAllocThreads, nb), dim3(kAllocThreads), 0, s, F + off, J, max_code_bits, lists + off);
        const dq_status st = launched();
        if (st != DQ_OK) return st;
      }
      const auto kernel = listed      ? k_search_positions<false, true, true>
                          : rows > 16 ? (allow16 ? k_search_positions<true, true, false> : k_search_positions<false, true, false>)
                                      : (allow16 ? k_search_positions<true, false, false> : k_search_positions<false, false, false>);
      hipLaunchKernelGGL(kernel, dim3(rows, nb), dim3(kAllocThreads), 0, s, F + off, listed ? lists + off : nullptr, J, max_code_bits, widths + off, pos + off,
                         cnt, announce);
    } else if (rows <= (uint32_t)kRegs) {
      const dq_status st = dq::search(F + off, J, nb, max_code_bits, max_width, pos + off, cnt, announce, s);
      if (st != DQ_OK) return st;
      hipLaunchKernelGGL(k_alloc_positions, dim3(rows, nb), dim3(kAllocThreads), 0, s, F + off, J, allow16, cnt, widths + off, pos + off);
    } else
      hipLaunchKernelGGL(k_allocate_large, dim3(nb), dim3(kAllocThreads), 0, s, F + off, J, max_code_bits, allow16, widths + off, pos + off, cnt);
    const dq_status st = launched();
    if (st != DQ_OK) return st;
    b0 += nb;
  }
  return DQ_OK;
}

dq_status dq_allocate(const float *F, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint64_t max_code_bits,
                      uint32_t max_width, uint8_t *widths, uint32_t *pos, uint32_t *counts, void *hip_stream) {
  return allocate(F, n_sg_per_bucket, n_buckets, max_code_bits, max_width, widths, pos, counts, nullptr, false, dq::Announce{nullptr, 0}, hip_stream);
}

uint64_t dqx_allocate_lists(uint32_t n_sg_per_bucket, uint32_t n_buckets, uint32_t max_width) {
  return rows_search(n_sg_per_bucket, n_buckets) && dq::takes_lists(n_sg_per_bucket, n_buckets, max_width) ? (uint64_t)n_sg_per_bucket * n_buckets : 0;
}

dq_status dqx_allocate_begin(const float *F, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint64_t max_code_bits, uint32_t max_width,
                             uint8_t *widths, uint32_t *pos, uint32_t *counts, uint32_t *lists, int beside, void *hip_stream, void **ticket) {
  dq::Announce announce = {nullptr, 0};
  if (ticket) *ticket = nullptr;
  if (ticket && n_buckets != 0 && n_sg_per_bucket != 0 && n_sg_per_bucket <= (uint32_t)(kRegs * kAllocThreads)) {
    const hipError_t e = dq::announce_begin(n_buckets, (hipStream_t)hip_stream, &announce, ticket);
    if (e != hipSuccess) return dq::hip_status(e);
  }
  const dq_status st = allocate(F, n_sg_per_bucket, n_buckets, max_code_bits, max_width, widths, pos, counts, lists, beside != 0, announce, hip_stream);
  if (st != DQ_OK && ticket && *ticket) {
    dq::announce_drop(*ticket);
    *ticket = nullptr;
  }
  return st;
}

dq_status dq_reorder(const void *x, dq_dtype dtype, const uint32_t *pos, uint32_t n_sg_per_bucket, uint32_t n_buckets,
                     void *out, void *hip_stream) {
  if (n_sg_per_bucket == 0 || n_buckets == 0) return DQ_OK;
  if (!x || !pos || !out || x == out || (dtype != DQ_F32 && dtype != DQ_BF16)) return DQ_EINVAL;
  if (n_sg_per_bucket > (1u << 24) || n_buckets > 65535u) return DQ_EUNSUPPORTED;
  if (!aligned(x, 16) || !aligned(out, 16) || !aligned(pos, 4)) return DQ_EALIGN;
  const uint64_t pieces = (uint64_t)n_sg_per_bucket * (dtype == DQ_F32 ? 64 : 32);
  const uint32_t blocks = stream_blocks((uint64_t)kThreads * kUnroll, pieces, n_buckets);
  hipStream_t s = (hipStream_t)hip_stream;
  if (dtype == DQ_F32)
    hipLaunchKernelGGL(k_reorder<64>, dim3(blocks, n_buckets), dim3(kThreads), 0, s, x, pos, n_sg_per_bucket, out);
  else
    hipLaunchKernelGGL(k_reorder<32>, dim3(blocks, n_buckets), dim3(kThreads), 0, s, x, pos, n_sg_per_bucket, out);
  return launched();
}

dq_status dq_reorder_mean(const float *mu_or_null, const uint32_t *pos, const uint32_t *counts_or_null,
                          uint32_t n_sg_per_bucket, uint32_t n_buckets, float *mu_main_or_null, uint32_t *origin_or_null,
                          void *hip_stream) {
  if (n_sg_per_bucket == 0 || n_buckets == 0) return DQ_OK;
  if (!pos || (!mu_main_or_null && !origin_or_null) || (mu_main_or_null && (!mu_or_null || mu_or_null == mu_main_or_null)) ||
      origin_or_null == pos)
    return DQ_EINVAL;
  if (n_sg_per_bucket > (1u << 24) || n_buckets > 65535u) return DQ_EUNSUPPORTED;
  if (!aligned(mu_or_null, 4) || !aligned(pos, 4) || !aligned(counts_or_null, 4) || !aligned(mu_main_or_null, 4) ||
      !aligned(origin_or_null, 4))
    return DQ_EALIGN;
  const uint32_t blocks = stream_blocks(kThreads, n_sg_per_bucket, n_buckets);
  hipLaunchKernelGGL(k_reorder_mean, dim3(blocks, n_buckets), dim3(kThreads), 0, (hipStream_t)hip_stream, mu_or_null, pos,
                     counts_or_null, n_sg_per_bucket, mu_main_or_null, origin_or_null);
  return launched();
}

dq_status dq_restore(const float *sum, const uint32_t *pos, const float *mu_main_or_null, uint32_t n_workers,
                     uint32_t n_sg_per_bucket, uint32_t n_buckets, float *out, void *hip_stream) {
  if (n_sg_per_bucket == 0 || n_buckets == 0) return DQ_OK;
  if (!sum || !pos || !out || sum == out || n_workers == 0) return DQ_EINVAL;
  if (n_sg_per_bucket > (1u << 24) || n_buckets > 65535u) return DQ_EUNSUPPORTED;
  if (!aligned(sum, 16) || !aligned(out, 16) || !aligned(pos, 4) || !aligned(mu_main_or_null, 4)) return DQ_EALIGN;
  const uint32_t blocks = stream_blocks((uint64_t)kThreads * kUnroll, (uint64_t)n_sg_per_bucket * 64, n_buckets);
  hipLaunchKernelGGL(k_restore, dim3(blocks, n_buckets), dim3(kThreads), 0, (hipStream_t)hip_stream, sum, pos,
                     mu_main_or_null, (float)n_workers, n_sg_per_bucket, out);
  return launched();
}

}  // extern "C"
