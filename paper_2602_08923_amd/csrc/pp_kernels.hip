// Steps before and after the main all-reduce stage, for gfx950: per-super-group statistics
// (Section 3.1), their combination over workers with the bf16 exchange format (Sections 3.1,
// 3.5), the bit allocation with tied thresholds (Section 3.2, Appendix A), the reorder into
// increasing width order (Section 3.5), the means the main stage subtracts in that order
// (Section 3.1) and the final restore (Section 3.4, last paragraph).  All of them stream each entry once; the allocation
// works on 4 bytes per super-group.
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
// Statistics.  One wave handles 4 super-groups at a time: lane l owns group l (16 entries,
// 32 or 64 consecutive bytes), sums them left to right in fp32 (squares by fma), and the 16
// lanes of a row are combined by a butterfly (partner distance 1, 2, 4, 8).
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
// Sum and sum of squares over the row's super-group, the same bits in all 16 lanes.
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
#pragma unroll
  for (int d = 1; d < 16; d <<= 1) {
    s += __shfl_xor(s, d, 64);
    f += __shfl_xor(f, d, 64);
  }
}

template <typename LT>
__global__ void __launch_bounds__(kThreads) k_stats(const void *x, uint64_t n_sg, float *mu, float *F) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint64_t wave = (uint64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
  const uint64_t n_waves = (uint64_t)gridDim.x * (kThreads / 64);
  const uint64_t n_tiles = (n_sg + 3) / 4;
  for (uint64_t t = wave; t < n_tiles; t += n_waves) {
    const uint64_t sg = min(t * 4 + (lane >> 4), n_sg - 1);  // idle rows redo the last SG, store nothing
    float s, f;
    row_sums<LT>(load_entries<LT>(x, sg * kSG + (lane & 15u) * 16), s, f);
    if ((lane & 15u) == 0 && t * 4 + (lane >> 4) < n_sg) {
      gst<float>(mu + sg, s * (1.0f / kSG));
      gst<float>(F + sg, f);
    }
  }
}

// k_stats of every worker and k_combine in one pass: a simulated all-reduce, which holds all workers' tensors, has no use for
// the single workers' statistics.  One launch instead of n + 1.
constexpr uint32_t kStatsWorkers = 256;
struct WorkerTensors {
  const void *x[kStatsWorkers];
};
template <typename LT>
__global__ void __launch_bounds__(kThreads) k_stats_all(WorkerTensors W, uint32_t n, uint64_t n_sg, float *mu, float *F) {
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

// Combination over workers: contributions rounded to bf16 (what is exchanged), summed in rank
// order in fp32; the mean of the means by one division.
__global__ void __launch_bounds__(kThreads) k_combine(const float *mu_all, const float *F_all, uint32_t n, uint64_t J,
                                                      float *mu, float *F) {
  const uint64_t j = (uint64_t)blockIdx.x * kThreads + threadIdx.x;
  if (j >= J) return;
  float sm = 0.0f, sf = 0.0f;
  for (uint32_t i = 0; i < n; ++i) {
    sm = sm + u2f(bf16_rne(gld<float>(mu_all + (uint64_t)i * J + j)) << 16);
    sf = sf + u2f(bf16_rne(gld<float>(F_all + (uint64_t)i * J + j)) << 16);
  }
  gst<float>(mu + j, sm / (float)n);
  gst<float>(F + j, sf);
}

// ---------------------------------------------------------------------------------------
// Allocation: the search in one block of 1024 threads per bucket.  Super-group j = 1024*k + t sits in slot k
// of thread t (a register when the bucket has at most 64 rows of 1024), so every global access
// is coalesced.  Values are handled as int32 bit patterns: non-negative floats order like their
// patterns, and the difference of two patterns below 2^31 has the sign of the comparison,
// F >= theta  <=>  bits(F) - bits(theta) >= 0.  Negative values and NaN count as +0; slots past
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
__global__ void __launch_bounds__(kAllocThreads) k_alloc_positions(const float *F_all, uint32_t J, bool allow16,
                                                                   const uint32_t *counts_all, uint8_t *widths_all,
                                                                   uint32_t *pos_all) {
  __shared__ uint32_t mine_w[kAllocWaves][4];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint64_t first = (uint64_t)blockIdx.y * J;
  const uint32_t *cnt = counts_all + 5ull * blockIdx.y;
  const uint32_t j = blockIdx.x * kAllocThreads + tid;
  const bool last = blockIdx.x + 1 == gridDim.x;
  const float f = gld<float>(F_all + first + min(j, J - 1));
  uint32_t at_row[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) at_row[c] = last ? gld<uint32_t>(cnt + c) : gld<uint32_t>(pos_all + first + (uint64_t)blockIdx.x * kAllocThreads + c);
  const uint32_t pattern = gld<uint32_t>(cnt + 4);
  const int32_t p8 = (int32_t)pattern, p4 = p4_from(pattern), p16 = p16_from(pattern, allow16);
  const uint32_t k = j < J ? class_of(pattern_of(f), p4, p8, p16) : 4u;
  const uint64_t b[4] = {__ballot(k == 0), __ballot(k == 1), __ballot(k == 2), __ballot(k == 3)};
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) mine_w[wave][i] = (uint32_t)__builtin_popcountll(b[i]);
  }
  __syncthreads();
  if (k < 4) {
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
    at += before + __builtin_amdgcn_mbcnt_hi((uint32_t)(mine >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mine, 0u));
    gst<uint8_t>(widths_all + first + j, (uint8_t)(2u << k));
    gst<uint32_t>(pos_all + first + j, at);
  }
}

// The search for buckets of at most 64 rows of 1024, the norms' patterns in registers (kRegs per thread; every pass skips
// the rows that the bucket does not have, four at a time).
//
// Wanted: the smallest fp32 pattern in [1, +inf] whose allocation fits (the host has checked 2J <= budget).  With
// c8, c4, c16 = norms at or above T_{4,8} and its tied thresholds, cost = 2J + 4 c8 + 2 c4 + 8 c16 never increases with
// the threshold, so a bracket (lo does not fit or is 0, hi fits) is narrowed level by level: a histogram of the patterns
// around each of the three thresholds, suffix counts, and for every bin boundary of the bracket a lower and an upper bound of its
// cost (c8 is exact there, c4 and c16 lie between the counts of two bins).  2048 bins a level: the top 11 bits of
// everything, then what is left of the bracket, 1 to 3 bins of 2^20, then single patterns.
//
// What bounds it: one CU's vector ALU (51,200 norms are 800 wave instructions for every instruction of a pass) and
// the barriers.  It replaced a gather of the candidates (two LDS atomics with a result per row, 20 us), a
// bisection with a barrier per step, and full counts per step where 16 bits are allowed.
constexpr uint32_t kBins4 = 3072, kBins16 = 5120;  // the tied thresholds' brackets in bins of the same size: up to 1.07 and 2 times as many
__global__ void __launch_bounds__(kAllocThreads) k_search(const float *F_all, uint32_t J, uint64_t max_code_bits, bool allow16,
                                                          uint32_t *pos_all, uint32_t *counts_all) {
  __shared__ uint32_t h8[kBins + 2], h4[kBins4 + 2], h16[kBins16 + 2];
  __shared__ uint32_t wsum[3][kAllocWaves], wbase[2][kAllocWaves], wfit[2][kAllocWaves];
  __shared__ uint32_t tot[kRegs * kAllocWaves][4];  // per (row, wave): class counts, then their exclusive scan
  const float *F = F_all + (uint64_t)blockIdx.x * J;
  uint32_t *pos = pos_all + (uint64_t)blockIdx.x * J;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  int32_t fr[kRegs];
  const uint32_t rows = (J + kAllocThreads - 1) / kAllocThreads;
  auto each_row = [&](auto body) {
#pragma unroll
    for (int g = 0; g < kRegs; g += 4)
      if ((uint32_t)g < rows) {
#pragma unroll
        for (int k = g; k < g + 4; ++k) body(k);
      }
  };
  each_row([&](int k) { fr[k] = (int32_t)f2u(gld<float>(F + min(k * kAllocThreads + tid, J - 1))); });  // all in flight at once
  each_row([&](int k) { fr[k] = k * kAllocThreads + tid < J ? pattern_of(u2f((uint32_t)fr[k])) : -1; });
  auto p16_of = [&](uint32_t pattern) { return allow16 ? f2u(u2f(pattern) * (131072.0f / 257.0f)) : (uint32_t)kNever; };
  auto p4_of = [](uint32_t pattern) { return f2u(u2f(pattern) * (17.0f / 512.0f)); };
  // h[b] for b < PER * 1024 becomes the sum of h[b], h[b + 1], ...; two barriers, shared by up to three histograms
  uint32_t inc[3], own[3];
  auto sums_begin = [&](int which, const uint32_t *h, int per) {
    uint32_t sum = 0;
    for (int i = 0; i < per; ++i) sum += h[tid * per + i];
    own[which] = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t up = __shfl_up(sum, d, 64);
      if (lane >= (uint32_t)d) sum += up;
    }
    inc[which] = sum;
    if (lane == 63) wsum[which][wave] = sum;
  };
  auto sums_end = [&](int which, uint32_t *h, int per) {
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kAllocWaves; ++w) {
      const uint32_t t = wsum[which][w];
      before += (uint32_t)w < wave ? t : 0u;
      all += t;
    }
    uint32_t left = all - (before + inc[which] - own[which]);  // from this thread's first bin on
    for (int i = 0; i < per; ++i) {
      const uint32_t x = h[tid * per + i];
      h[tid * per + i] = left;
      left -= x;
    }
  };
  // How many of the bin boundaries 1 .. n-1 surely do not fit, and how many may not: the bracket is between them.
  auto bracket = [&](uint32_t n, auto cost_bounds, uint32_t &surely, uint32_t &perhaps) {
    uint32_t a = 0, c = 0;
    for (uint32_t b0 = 0; b0 < n; b0 += kAllocThreads) {  // uniform trips: every thread takes part in the ballots
      const uint32_t bin = b0 + tid;
      bool over = false, may = false;
      if (bin >= 1 && bin < n) {
        uint64_t c_min, c_max;
        cost_bounds(bin, c_min, c_max);
        over = c_min > max_code_bits;
        may = c_max > max_code_bits;
      }
      a += (uint32_t)__builtin_popcountll(__ballot(over));
      c += (uint32_t)__builtin_popcountll(__ballot(may));
    }
    if (lane == 0) {
      wfit[0][wave] = a;
      wfit[1][wave] = c;
    }
    __syncthreads();
    surely = 0;
    perhaps = 0;
#pragma unroll
    for (int w = 0; w < kAllocWaves; ++w) {
      surely += wfit[0][w];
      perhaps += wfit[1][w];
    }
  };

  // level 1: bins of 2^20 patterns, 2040 << 20 is +infinity
  for (uint32_t b = tid; b < kBins + 2; b += kAllocThreads) h8[b] = 0;
  __syncthreads();
  each_row([&](int k) {
    if (fr[k] >= 0) atomicAdd(&h8[(uint32_t)fr[k] >> 20], 1u);
  });
  __syncthreads();
  sums_begin(0, h8, kBins / kAllocThreads);
  __syncthreads();
  sums_end(0, h8, kBins / kAllocThreads);
  __syncthreads();
  uint32_t surely, perhaps;
  bracket(kBins - 8, [&](uint32_t b, uint64_t &c_min, uint64_t &c_max) {
    const uint32_t b4 = p4_of(b << 20) >> 20, b16 = p16_of(b << 20) >> 20;
    const uint64_t fixed = 2ull * J + 4ull * h8[b];
    c_min = fixed + 2ull * h8[b4 + 1] + 8ull * h8[b16 + 1];
    c_max = fixed + 2ull * h8[b4] + 8ull * h8[b16];
  }, surely, perhaps);
  uint32_t lo = surely << 20, hi = (perhaps + 1) << 20;
  uint32_t base8 = h8[perhaps + 1];  // norms at or above hi

  bool exact = false;
  while (hi - lo > 1 && !exact) {
    const uint32_t width = hi - lo, lo4 = p4_of(lo), hi4 = p4_of(hi), lo16 = p16_of(lo), hi16 = p16_of(hi);
    uint32_t s = 0, s4 = 0, s16 = 0;
    while ((width - 1) >> s >= kBins) ++s;
    while ((hi4 - lo4) >> s4 >= kBins4 || s4 < s) ++s4;
    while ((hi16 - lo16) >> s16 >= kBins16 || s16 < s) ++s16;  // denormal thresholds: up to 510 patterns to one
    const uint32_t n = ((width - 1) >> s) + 1;
    __syncthreads();  // everybody has read the level before
    for (uint32_t b = tid; b < kBins + 2; b += kAllocThreads) h8[b] = 0;
    for (uint32_t b = tid; b < kBins4 + 2; b += kAllocThreads) h4[b] = 0;
    if (allow16) for (uint32_t b = tid; b < kBins16 + 2; b += kAllocThreads) h16[b] = 0;
    __syncthreads();
    uint32_t above4 = 0, above16 = 0;
    each_row([&](int k) {
      const uint32_t v = (uint32_t)fr[k];
      if (v - lo < width) atomicAdd(&h8[(v - lo) >> s], 1u);
      if (v - lo4 < hi4 - lo4) atomicAdd(&h4[(v - lo4) >> s4], 1u);
      above4 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= (int32_t)hi4));
      if (allow16) {
        if (v - lo16 < hi16 - lo16) atomicAdd(&h16[(v - lo16) >> s16], 1u);
        above16 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= (int32_t)hi16));
      }
    });
    if (lane == 0) {
      wbase[0][wave] = above4;
      wbase[1][wave] = above16;
    }
    __syncthreads();
    sums_begin(0, h8, kBins / kAllocThreads);
    sums_begin(1, h4, kBins4 / kAllocThreads);
    if (allow16) sums_begin(2, h16, kBins16 / kAllocThreads);
    __syncthreads();
    sums_end(0, h8, kBins / kAllocThreads);
    sums_end(1, h4, kBins4 / kAllocThreads);
    if (allow16) sums_end(2, h16, kBins16 / kAllocThreads);
    uint32_t base4 = 0, base16 = 0;
#pragma unroll
    for (int w = 0; w < kAllocWaves; ++w) {
      base4 += wbase[0][w];
      base16 += wbase[1][w];
    }
    __syncthreads();
    bracket(n, [&](uint32_t b, uint64_t &c_min, uint64_t &c_max) {
      const uint32_t T = lo + (b << s), b4 = (p4_of(T) - lo4) >> s4;
      // a tied threshold on a bin's first pattern has that bin's count exactly
      const bool on4 = ((p4_of(T) - lo4) & ((1u << s4) - 1u)) == 0;
      const uint64_t fixed = 2ull * J + 4ull * (base8 + h8[b]);
      c_min = fixed + 2ull * (base4 + h4[on4 ? b4 : b4 + 1]);
      c_max = fixed + 2ull * (base4 + h4[b4]);
      if (allow16) {
        const uint32_t at = p16_of(T) - lo16, b16 = at >> s16;
        c_min += 8ull * (base16 + h16[(at & ((1u << s16) - 1u)) == 0 ? b16 : b16 + 1]);
        c_max += 8ull * (base16 + h16[b16]);
      }
    }, surely, perhaps);
    const uint32_t new_lo = surely ? lo + (surely << s) : lo;
    const uint32_t new_hi = perhaps + 1 < n ? lo + ((perhaps + 1) << s) : hi;
    if (perhaps + 1 < n) base8 += h8[perhaps + 1];
    exact = new_hi - new_lo > width / 2 && new_hi - new_lo > 1;  // bounds too loose to go on: count exactly below
    lo = new_lo;
    hi = new_hi;
  }
  // Exact counts at one threshold.
  uint32_t turn = 0;
  auto block_counts = [&](uint32_t pattern, uint32_t &c4, uint32_t &c8, uint32_t &c16) {
    const int32_t p4 = p4_from(pattern), p8 = (int32_t)pattern, p16 = p16_from(pattern, allow16);
    uint32_t a4 = 0, a8 = 0, a16 = 0;
    each_row([&](int k) {
      a4 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= p4));
      a8 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= p8));
      if (allow16) a16 += (uint32_t)__builtin_popcountll(__ballot(fr[k] >= p16));
    });
    // the waves' counts meet in one of two buffers by turns, so that one barrier per round is enough
    if (lane == 0) {
      tot[turn * kAllocWaves + wave][0] = a4;
      tot[turn * kAllocWaves + wave][1] = a8;
      tot[turn * kAllocWaves + wave][2] = a16;
    }
    __syncthreads();
    c4 = c8 = c16 = 0;
#pragma unroll
    for (int w = 0; w < kAllocWaves; ++w) {
      c4 += tot[turn * kAllocWaves + w][0];
      c8 += tot[turn * kAllocWaves + w][1];
      c16 += tot[turn * kAllocWaves + w][2];
    }
    turn ^= 1u;
  };
  while (hi - lo > 1) {
    const uint32_t mid = lo + (hi - lo) / 2;
    uint32_t c4, c8, c16;
    block_counts(mid, c4, c8, c16);
    const uint64_t cost = 2ull * J + 2ull * c4 + 4ull * c8 + 8ull * c16;
    if (cost <= max_code_bits) hi = mid; else lo = mid;
  }
  __syncthreads();
  // class counts of every (row, wave), their exclusive scan in that order: the rows' first places
  const int32_t p8 = (int32_t)hi, p4 = p4_from(hi), p16 = p16_from(hi, allow16);
  each_row([&](int k) {
    const int32_t v = fr[k];
    const uint32_t at0 = (uint32_t)__builtin_popcountll(__ballot(v >= 0)), at4 = (uint32_t)__builtin_popcountll(__ballot(v >= p4)),
                   at8 = (uint32_t)__builtin_popcountll(__ballot(v >= p8)),
                   at16 = allow16 ? (uint32_t)__builtin_popcountll(__ballot(v >= p16)) : 0u;
    if (lane == 0) {
      tot[k * kAllocWaves + wave][0] = at0 - at4;
      tot[k * kAllocWaves + wave][1] = at4 - at8;
      tot[k * kAllocWaves + wave][2] = at8 - at16;
      tot[k * kAllocWaves + wave][3] = at16;
    }
  });
  __syncthreads();
  uint32_t x[4], sum[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    x[c] = tid < rows * kAllocWaves ? tot[tid][c] : 0u;
    sum[c] = x[c];
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t up = __shfl_up(sum[c], d, 64);
      if (lane >= (uint32_t)d) sum[c] += up;
    }
  }
  __syncthreads();
  if (lane == 63) {
#pragma unroll
    for (int c = 0; c < 4; ++c) h8[4 * wave + c] = sum[c];
  }
  __syncthreads();
  uint32_t n_class[4], row_first[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kAllocWaves; ++w) {
      const uint32_t t = h8[4 * w + c];
      before += (uint32_t)w < wave ? t : 0u;
      all += t;
    }
    n_class[c] = all;
    row_first[c] = before + sum[c] - x[c];
  }
  const uint32_t row = tid / kAllocWaves, class_first[4] = {0u, n_class[0], n_class[0] + n_class[1], n_class[0] + n_class[1] + n_class[2]};
  if (tid % kAllocWaves == 0 && (row + 1) * kAllocThreads < J) {  // not the last row
#pragma unroll
    for (int c = 0; c < 4; ++c) gst<uint32_t>(pos + row * kAllocThreads + c, class_first[c] + row_first[c]);
  }
  if (tid == 0) {
    uint32_t *cnt = counts_all + 5ull * blockIdx.x;
#pragma unroll
    for (int c = 0; c < 4; ++c) gst<uint32_t>(cnt + c, n_class[c]);
    gst<uint32_t>(cnt + 4, hi);
  }
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

// blocks per grid row: enough for the units of one row, at most the GPU's resident share
uint32_t stream_blocks(uint64_t units_per_block_round, uint64_t units, uint32_t rows = 1) {
  int dev = 0, n_cu = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  const uint64_t need = (units + units_per_block_round - 1) / units_per_block_round;
  const uint64_t cap = ((uint64_t)n_cu * 8 + rows - 1) / rows;  // 8 blocks of 256 threads per CU in all
  return (uint32_t)(need < 1 ? 1 : (need < cap ? need : cap));
}

dq_status launched() { return dq::hip_status(hipGetLastError()); }

}  // namespace

extern "C" {

dq_status dq_sg_stats(const void *x, dq_dtype dtype, uint64_t n_sg, float *mu_out, float *F_out, void *hip_stream) {
  if (n_sg == 0) return DQ_OK;
  if (!x || !mu_out || !F_out || (dtype != DQ_F32 && dtype != DQ_BF16)) return DQ_EINVAL;
  if (!aligned(x, 16) || !aligned(mu_out, 4) || !aligned(F_out, 4)) return DQ_EALIGN;
  const uint32_t blocks = stream_blocks(4 * (kThreads / 64), n_sg);
  hipStream_t s = (hipStream_t)hip_stream;
  if (dtype == DQ_F32) hipLaunchKernelGGL(k_stats<float>, dim3(blocks), dim3(kThreads), 0, s, x, n_sg, mu_out, F_out);
  else hipLaunchKernelGGL(k_stats<uint16_t>, dim3(blocks), dim3(kThreads), 0, s, x, n_sg, mu_out, F_out);
  return launched();
}

dq_status dq_stats_combine(const float *mu_all, const float *F_all, uint32_t n_workers, uint64_t n_sg, float *mu,
                           float *F, void *hip_stream) {
  if (n_sg == 0) return DQ_OK;
  if (!mu_all || !F_all || !mu || !F || n_workers == 0) return DQ_EINVAL;
  if (!aligned(mu_all, 4) || !aligned(F_all, 4) || !aligned(mu, 4) || !aligned(F, 4)) return DQ_EALIGN;
  if ((n_sg + kThreads - 1) / kThreads > 0x7FFFFFFFull) return DQ_EUNSUPPORTED;
  hipLaunchKernelGGL(k_combine, dim3((uint32_t)((n_sg + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                     (hipStream_t)hip_stream, mu_all, F_all, n_workers, n_sg, mu, F);
  return launched();
}

dq_status dqx_stats_all(const void *const *tensors, uint32_t n_workers, dq_dtype dtype, uint64_t n_sg, float *mu, float *F,
                        void *hip_stream) {
  if (n_sg == 0) return DQ_OK;
  if (!tensors || !mu || !F || n_workers == 0 || (dtype != DQ_F32 && dtype != DQ_BF16)) return DQ_EINVAL;
  if (n_workers > kStatsWorkers) return DQ_EUNSUPPORTED;
  WorkerTensors W = {};
  for (uint32_t w = 0; w < n_workers; ++w) {
    if (!aligned(tensors[w], 16)) return DQ_EALIGN;
    W.x[w] = tensors[w];
  }
  const uint32_t blocks = stream_blocks(4 * (kThreads / 64), n_sg);
  hipStream_t s = (hipStream_t)hip_stream;
  if (dtype == DQ_F32) hipLaunchKernelGGL(k_stats_all<float>, dim3(blocks), dim3(kThreads), 0, s, W, n_workers, n_sg, mu, F);
  else hipLaunchKernelGGL(k_stats_all<uint16_t>, dim3(blocks), dim3(kThreads), 0, s, W, n_workers, n_sg, mu, F);
  return launched();
}

// k_alloc_positions over all buckets, 65,535 (the grid's second dimension) per launch
static void launch_positions(const float *F, uint32_t J, uint32_t n_buckets, bool allow16, const uint32_t *counts,
                             uint8_t *widths, uint32_t *pos, hipStream_t s) {
  for (uint32_t b0 = 0; b0 < n_buckets; b0 += 65535u) {
    const uint32_t nb = n_buckets - b0 < 65535u ? n_buckets - b0 : 65535u;
    const uint64_t off = (uint64_t)b0 * J;
    hipLaunchKernelGGL(k_alloc_positions, dim3((J + kAllocThreads - 1) / kAllocThreads, nb), dim3(kAllocThreads), 0, s,
                       F + off, J, allow16, counts + 5ull * b0, widths + off, pos + off);
  }
}

dq_status dq_allocate(const float *F, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint64_t max_code_bits,
                      uint32_t max_width, uint8_t *widths, uint32_t *pos, uint32_t *counts, void *hip_stream) {
  if (n_sg_per_bucket == 0 || n_buckets == 0) return DQ_OK;
  if (!F || !widths || !pos || !counts || (max_width != 8 && max_width != 16)) return DQ_EINVAL;
  if (max_code_bits < 2ull * n_sg_per_bucket) return DQ_EINVAL;  // fewer than 2 code bits per coordinate
  if (!aligned(F, 4) || !aligned(pos, 4) || !aligned(counts, 4)) return DQ_EALIGN;
  hipStream_t s = (hipStream_t)hip_stream;
  const bool allow16 = max_width == 16;
  const uint32_t J = n_sg_per_bucket, rows = (J + kAllocThreads - 1) / kAllocThreads;
  if (rows <= (uint32_t)kRegs) {
    hipLaunchKernelGGL(k_search, dim3(n_buckets), dim3(kAllocThreads), 0, s, F, J, max_code_bits, allow16, pos, counts);
    launch_positions(F, J, n_buckets, allow16, counts, widths, pos, s);
  } else
    hipLaunchKernelGGL(k_allocate_large, dim3(n_buckets), dim3(kAllocThreads), 0, s, F, J, max_code_bits, allow16, widths, pos, counts);
  return launched();
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
