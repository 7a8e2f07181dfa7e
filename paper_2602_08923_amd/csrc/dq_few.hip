// Single calls (compress, DAR hop, decompress) on chunks of few super-groups: one super-group per wave, four entries per lane.
//
// Why: with a tile of four super-groups per wave (dq_kernels.hip) such a call is a chain of latencies: the arguments, the
// tables' trip, the tile's trip, then the instructions of 16 entries one after the other, one every four cycles, as a wave has its SIMD
// almost to itself.  Here the arguments are read at once, the tile is requested before the tables, the draws are made while both are on
// their way, and the chain of the entries is a quarter as long.  Measured, us per call back to back, bf16, 2- to 8-bit super-groups, tiles of
// four -> one per wave (the host takes 3.2 to 3.9 for a launch):
//                 3,000          4,096          6,000          8,192          10,240         12,288
//   hop           4.9 -> 4.0     5.1 -> 4.05    5.25 -> 4.7    5.5 -> 5.4     5.85 -> 6.15   6.15 -> 6.85
//   compress      4.75 -> 3.65   4.8 -> 3.75    5.0 -> 4.3     5.25 -> 5.0    5.45 -> 5.65   5.7 -> 6.3
//   sink          4.2 -> 3.3     4.35 -> 3.4    4.45 -> 3.75   4.6 -> 4.2     4.75 -> 4.7    5.0 -> 5.2
//   receive       4.0 -> 3.2     4.05 -> 3.35   4.2 -> 3.65    4.45 -> 4.0    4.65 -> 4.45   4.75 -> 4.85
// What bounds it: up to one block per CU the latencies, from there vector-ALU issue (370 instructions per super-group and
// wave, against 100 per super-group in tiles of four; 450 when every wave drew its super-group's numbers itself, and 0.8 us
// more per block and CU).
#include "dq_bounds.h"
#include "dq_codec.h"

namespace dq {
namespace {

constexpr uint32_t kFewWaves = 8;  // per block (with four, twice the copies of the tables: 0.3 to 0.9 us more from 4,096 super-groups on)
constexpr int kEntries = 4;        // per lane
constexpr uint32_t kFewTableBytes = 24576;  // tables up to this size: three 16-byte words per thread
static_assert(kOffLut4 * 4 <= 2 * kFewWaves * 64 * 16, "what decompress reads of them: two");

// What a lane fetches: its four entries, their codes, and what its group and super-group share.
template <typename LT>
struct Piece {
  uint32_t loc[sizeof(LT) == 4 ? 4 : 2];
  float mu, back;
  uint32_t code, code_hi;  // four codes of 2, 4, 8 or (both words) 16 bits
  uint32_t rg, sf;
  uint32_t dest;
};

// Where the wave's super-group sits.
struct Place {
  uint32_t sg;  // in the chunk
  uint32_t wi;
  size_t code, gs, sf;  // byte offsets inside a packed buffer
};
__device__ __forceinline__ Place place_of(const Job &job, uint32_t sg) {
  const size_t n0 = job.n_sg[0], n1 = job.n_sg[1], n2 = job.n_sg[2], n3 = job.n_sg[3];
  const size_t c4 = 64 * n0, c8 = c4 + 128 * n1, c16 = c8 + 256 * n2, gs0 = c16 + 512 * n3;
  Place p;
  p.sg = sg;
  p.wi = sg < n0 ? 0u : sg < n0 + n1 ? 1u : sg < n0 + n1 + n2 ? 2u : 3u;
  const size_t first = p.wi == 0 ? 0 : p.wi == 1 ? n0 : p.wi == 2 ? n0 + n1 : n0 + n1 + n2;
  p.code = (p.wi == 0 ? 0 : p.wi == 1 ? c4 : p.wi == 2 ? c8 : c16) + ((sg - first) << (6 + p.wi));
  p.gs = gs0 + 16 * (size_t)sg;
  p.sf = gs0 + 16 * (n0 + n1 + n2) + 2 * (size_t)sg;
  return p;
}

template <Kind KIND, typename LT>
__device__ __forceinline__ Piece<LT> fetch_piece(const Job &job, const Place &p, uint32_t src_limit) {
  constexpr bool kHasLocal = !__is_same(LT, NoLocal);
  const uint32_t lane = threadIdx.x & 63u;
  Piece<LT> f;
  uint64_t from = p.sg;
  if constexpr (kHasLocal)
    if (job.src) from = min(gld<uint32_t>(job.src + p.sg), src_limit - 1u);
  if constexpr (KIND != kCompress) {
    const uint8_t *code = job.in + p.code;
    f.code = f.code_hi = f.rg = f.sf = 0;
    if (p.wi == 0) f.code = gld<uint8_t>(code + lane);
    else if (p.wi == 1) f.code = gld<uint16_t>(code + lane * 2);
    else if (p.wi == 2) f.code = gld<uint32_t>(code + lane * 4);
    else {
      const u32x2 t = gld<u32x2>(code + lane * 8);
      f.code = t.x;
      f.code_hi = t.y;
    }
    if (p.wi < 3) {
      f.rg = gld<uint8_t>(job.in + p.gs + (lane >> 2));
      f.sf = gld<uint16_t>(job.in + p.sf);
    }
  }
  if constexpr (KIND == kDecompress) {
    f.back = job.back ? gld<float>(job.back + p.sg) : 0.0f;
    f.dest = job.dest ? gld<uint32_t>(job.dest + p.sg) : p.sg;
  }
  if constexpr (kHasLocal) {
    f.mu = job.mu ? gld<float>(job.mu + p.sg) : 0.0f;  // taking off 0 changes nothing
    const uint8_t *x = static_cast<const uint8_t *>(job.local) + (from * kSG + lane * kEntries) * sizeof(LT);
    if constexpr (sizeof(LT) == 4) {
      const u32x4 t = gld<u32x4>(x);
      f.loc[0] = t.x; f.loc[1] = t.y; f.loc[2] = t.z; f.loc[3] = t.w;
    } else {
      const u32x2 t = gld<u32x2>(x);
      f.loc[0] = t.x; f.loc[1] = t.y;
    }
  }
  return f;
}

template <typename LT>
__device__ __forceinline__ void widen_piece(const Piece<LT> &f, float (&v)[kEntries]) {
  if constexpr (__is_same(LT, NoLocal)) {
#pragma unroll
    for (int k = 0; k < kEntries; ++k) v[k] = 0.0f;
  } else if constexpr (sizeof(LT) == 4) {
#pragma unroll
    for (int k = 0; k < kEntries; ++k) v[k] = u2f(f.loc[k]) - f.mu;
  } else {
#pragma unroll
    for (int k = 0; k < kEntries / 2; ++k) {
      v[2 * k] = u2f(f.loc[k] << 16) - f.mu;
      v[2 * k + 1] = u2f(f.loc[k] & 0xFFFF0000u) - f.mu;
    }
  }
}

template <int B>
__device__ __forceinline__ void levels_of(uint32_t code, float (&t)[kEntries]) {
  constexpr uint32_t dec0 = HopTables::template dec<B>();
  if constexpr (B == 2) {
    const u32x4 e = lds_ld4(dec0 + code * 16);
    t[0] = u2f(e.x); t[1] = u2f(e.y); t[2] = u2f(e.z); t[3] = u2f(e.w);
  } else if constexpr (B == 4) {
    const u32x2 a = lds_ld2(dec0 + (code & 0xFFu) * 8), b = lds_ld2(dec0 + (code >> 8) * 8);
    t[0] = u2f(a.x); t[1] = u2f(a.y); t[2] = u2f(b.x); t[3] = u2f(b.y);
  } else {
#pragma unroll
    for (int k = 0; k < kEntries; ++k) t[k] = u2f(lds_ld1(dec0 + ((code >> (8 * k)) & 0xFFu) * 4));
  }
}

template <typename LT>
__device__ __forceinline__ void put_result(const Job &job, const Params &P, const Piece<LT> &f, float (&v)[kEntries]) {
  if (job.back) {  // Section 3.4, last paragraph: the mean comes back, n times
    const float back = (float)P.n_workers * f.back;
#pragma unroll
    for (int k = 0; k < kEntries; ++k) v[k] = v[k] + back;
  }
  float *out = static_cast<float *>(job.out) + (size_t)f.dest * kSG + (threadIdx.x & 63u) * kEntries;
  gst_once<f32x4>(out, f32x4{v[0], v[1], v[2], v[3]});
}

template <int B, Kind KIND, typename LT>
__device__ __forceinline__ void finish_piece(const Job &job, const Params &P, const Place &p, const Piece<LT> &f, const Draws &d) {
  const uint32_t lane = threadIdx.x & 63u, g = lane >> 2, q = lane & 3u;
  float v[kEntries];
  widen_piece<LT>(f, v);
  if constexpr (B == 16) {
    if constexpr (KIND != kCompress) {
      const uint32_t w[2] = {f.code, f.code_hi};
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        v[2 * k] = u2f(w[k] << 16) + v[2 * k];
        v[2 * k + 1] = u2f(w[k] & 0xFFFF0000u) + v[2 * k + 1];
      }
    }
    if constexpr (KIND == kDecompress) put_result<LT>(job, P, f, v);
    else gst<u32x2>(static_cast<uint8_t *>(job.out) + p.code + lane * 8, u32x2{bf16_rne_pair(v[0], v[1]), bf16_rne_pair(v[2], v[3])});
    return;
  } else {
    if constexpr (KIND != kCompress) {
      const float sfg = (float)f.rg * sf_over_255(f.sf, kRec0);
      float t[kEntries];
      levels_of<B>(f.code, t);
#pragma unroll
      for (int k = 0; k < kEntries; ++k) v[k] = __is_same(LT, NoLocal) ? t[k] * sfg : __builtin_fmaf(t[k], sfg, v[k]);
    }
    if constexpr (KIND == kDecompress) {
      put_result<LT>(job, P, f, v);
    } else {
      float m = 0.0f;
#pragma unroll
      for (int k = 0; k < kEntries; ++k) m = fmaxf(m, fabsf(v[k]));
      const uint32_t mg = group_max<kEntries>(f2u(m));
      const Scales s = scales_of(u2f(mg), u2f(sg_max<kEntries>(mg)), d.us, kRec0);
      const uint32_t gx = d.gam.x, gy = d.gam.y, gz = d.gam.z, gw = d.gam.w, lo = q & 1u ? +gy : +gx, hi = q & 1u ? +gw : +gz;
      const uint32_t gam = q & 2u ? +hi : +lo;
      float xs[kEntries];
      u32x4 t[kEntries];
#pragma unroll
      for (int k = 0; k < kEntries; ++k) xs[k] = v[k] * s.inv;
      if constexpr (B != 2) {
        u32x2 e[kEntries];
#pragma unroll
        for (int k = 0; k < kEntries; ++k) e[k] = lds_ld2(f2u(fabsf(xs[k]) + P.magic[B == 4 ? 1 : 2]) & 0x1FFF8u);
        __builtin_amdgcn_sched_barrier(0);  // all searches, then all levels
#pragma unroll
        for (int k = 0; k < kEntries; ++k) t[k] = load_level(or_and(f2u(fabsf(xs[k]) - u2f(e[k].x)) >> 27, 16u, e[k].y));
      }
      uint32_t word = 0;
#pragma unroll
      for (int k = kEntries - 1; k >= 0; --k) {  // a group whose scale rounded to zero: xs is a zero, the code its sign
        const float u = __builtin_fmaf((float)((gam >> (8 * k)) & 0xFFu), P.s_n, d.o_pi), x = fabsf(xs[k]);
        // as in quantize: the difference's sign rounds up
        uint32_t level;
        if constexpr (B == 2) level = f2u(u - x) >> 31;
        else level = (t[k].w >> (32 - B)) + (f2u(__builtin_fmaf(u, u2f(t[k].y), u2f(t[k].x)) - x) >> 31);
        word = (word << B) | (f2u(xs[k]) >> 31 << (B - 1)) | level;
      }
      uint8_t *out = static_cast<uint8_t *>(job.out);
      if constexpr (B == 2) gst<uint8_t>(out + p.code + lane, (uint8_t)word);
      else if constexpr (B == 4) gst<uint16_t>(out + p.code + lane * 2, (uint16_t)word);
      else gst<uint32_t>(out + p.code + lane * 4, word);
      if (q == 0) gst<uint8_t>(out + p.gs + g, (uint8_t)s.rg);
      if (lane == 0) gst<uint16_t>(out + p.sf, (uint16_t)s.sfb);
    }
  }
}

// A check of the call's indices in its own blocks: every block looks at all of them, so that all know the verdict; the largest index
// decides.  That takes up to 64 KB per block out of the L2, beside what the block waits for anyway.  A gathered hop of 3,187 super-groups
// takes 7.3 us, which is the host's time from one launch to the next with a look at the verdict between; 9.7 to 10.3 with the check as a launch
// in front of the call.
__device__ __forceinline__ uint32_t largest_index(const Bound &x) {
  typedef uint32_t Four __attribute__((ext_vector_type(4), aligned(4)));
  constexpr uint32_t kRound = kFewWaves * 64;
  const uint32_t fours = x.n / 4;
  uint32_t most = 0;
  for (uint32_t i = threadIdx.x; i < fours; i += 4 * kRound) {
    Four v[4];
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) v[k] = gld<Four>(x.index + 4 * min(i + k * kRound, fours - 1));
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) most = max(max(max(most, v[k].x), max(v[k].y, v[k].z)), v[k].w);
  }
  if (threadIdx.x < (x.n & 3u)) most = max(most, gld<uint32_t>(x.index + 4 * fours + threadIdx.x));
  return most;
}
// Bit k: this wave has found an index of array k out of bounds.
__device__ __forceinline__ uint32_t wave_verdict(const OwnCheck &c) {
  const uint32_t a = largest_index(c.a);
  uint32_t bits = __builtin_amdgcn_ballot_w64(a >= c.a.limit) ? 1u : 0u;
  if (c.b.n) {
    const uint32_t b = same_array(c.a, c.b) ? a : largest_index(c.b);  // a restore of what was gathered: one array
    bits |= __builtin_amdgcn_ballot_w64(b >= c.b.limit) ? 2u : 0u;
  }
  return bits;
}

// The block's, at whose barrier the waves' meet in LDS.
__device__ __forceinline__ void put_verdict(const OwnCheck &c, uint32_t at) {
  const uint32_t bits = wave_verdict(c);
  if ((threadIdx.x & 63u) == 0) lds_st1(at + (threadIdx.x >> 6) * 4, bits);
}
__device__ __forceinline__ uint32_t verdict_at(uint32_t at) {
  static_assert(kFewWaves == 8, "two reads");
  const u32x4 a = lds_ld4(at), b = lds_ld4(at + 16);
  return __builtin_amdgcn_readfirstlane(a.x | a.y | a.z | a.w | b.x | b.y | b.z | b.w);
}

// The first block of a checked call does nothing but look and tell the host, which waits for it.  Told by a block that also worked, behind the
// tables' trip and the draws, the verdict came a microsecond later (a gathered hop of 3,187 super-groups 8.4 us a call instead of 7.3).
__device__ __forceinline__ void post_verdict(const OwnCheck &check) {
  put_verdict(check, 0);
  __syncthreads();
  const uint32_t bits = verdict_at(0);
  if (threadIdx.x == 0)
    __hip_atomic_store(check.host, 4 * check.call + bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // nothing else to order
}

template <Kind KIND, typename LT, bool CHECK>
__global__ __launch_bounds__(kFewWaves * 64) void k_few(Job job_, Params P_, OwnCheck check) {
  extern __shared__ uint4 lds_raw[];
  uint32_t *lds = reinterpret_cast<uint32_t *>(lds_raw);
  if constexpr (CHECK)
    if (blockIdx.x == 0) {
      post_verdict(check);
      return;
    }
  const uint32_t block = blockIdx.x - (CHECK ? 1 : 0);
  // every argument in one go: read where it is used, each would be a trip of its own
  Job job = job_;
  Params P = P_;
  asm volatile("" : "+s"(job.in), "+s"(job.local), "+s"(job.mu), "+s"(job.src), "+s"(job.out), "+s"(job.dest), "+s"(job.back),
               "+s"(job.first_sg), "+s"(job.n_sg[0]), "+s"(job.n_sg[1]), "+s"(job.n_sg[2]), "+s"(job.n_sg[3]), "+s"(job.rank));
  asm volatile("" : "+s"(P.blob), "+s"(P.blob_dwords), "+s"(P.magic[1]), "+s"(P.magic[2]), "+s"(P.key0),
               "+s"(P.key1), "+s"(P.round), "+s"(P.n_workers), "+s"(P.perm_bits), "+s"(P.n_slots), "+s"(P.slot_keep), "+s"(P.g_mod),
               "+s"(P.inv_n), "+s"(P.inv_n512), "+s"(P.s_n));
  const uint32_t total = job.n_sg[0] + job.n_sg[1] + job.n_sg[2] + job.n_sg[3];
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t sg = block * kFewWaves + wave;
  const Place p = place_of(job, min(sg, total - 1));
  const Piece<LT> f = fetch_piece<KIND, LT>(job, p, CHECK ? check.src_limit : 0xFFFFFFFFu);
  // all tables, whatever widths the block meets: to choose would take longer
  const uint32_t words = KIND == kDecompress ? kOffLut4 / 4 : P.blob_dwords / 4;
  constexpr uint32_t kRounds = KIND == kDecompress ? 2 : kFewTableBytes / (kFewWaves * 64 * 16);
  uint4 part[kRounds];
  uint32_t at[kRounds];
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) {
    at[r] = min(r * kFewWaves * 64 + threadIdx.x, words - 1) * 4;
    part[r] = gld16(&P.blob[at[r]]);
  }
  Draws d = {};
  const uint32_t area = words * 16;  // the super-groups' draws, 32 bytes each: slot of the permutation, scale stream
  const uint32_t verdicts = area + kFewWaves * 32;
  if constexpr (KIND != kDecompress) {
    if (wave == 0) {  // lanes 2i, 2i + 1: the shared draw of the block's i-th super-group, the worker's for its scales
      const uint64_t G = job.first_sg + min(block * kFewWaves + (lane >> 1), total - 1);
      const U4 w = philox4x32_10((uint32_t)G, (uint32_t)(G >> 32), P.round, lane & 1u ? (1u << 16) | (job.rank & 0xFFFFu) : (2u << 16) | 0xFFFFu,
                                 P.key0, P.key1);
      const uint32_t w0 = lane & 1u ? w.x : perm_slot(w, P, job.rank);
      if (lane < 2 * kFewWaves) lds_st4(area + lane * 16, u32x4{w0, w.y, w.z, w.w});
    }
    const uint64_t gi = (job.first_sg + p.sg) * 16 + (lane >> 2);
    d.gam = philox4x32_10((uint32_t)gi, (uint32_t)(gi >> 32), P.round, job.rank & 0xFFFFu, P.key0, P.key1);
  }
#pragma unroll
  for (uint32_t r = 0; r < kRounds; ++r) *reinterpret_cast<uint4 *>(&lds[at[r]]) = part[r];
  if constexpr (CHECK) put_verdict(check, verdicts);
  __syncthreads();
  if constexpr (CHECK)
    if (verdict_at(verdicts)) return;
  if (sg >= total) return;  // not the last super-group once more: a hop may write where it reads
  if constexpr (KIND != kDecompress) {
    const uint32_t g = lane >> 2, mine = area + wave * 32;
    draw_offsets(P, lds_ld1(mine), lds_ld1(mine + 16 + (g >> 2) * 4), g, d);
  }
  if (p.wi == 0) finish_piece<2, KIND, LT>(job, P, p, f, d);
  else if (p.wi == 1) finish_piece<4, KIND, LT>(job, P, p, f, d);
  else if (p.wi == 2) finish_piece<8, KIND, LT>(job, P, p, f, d);
  else finish_piece<16, KIND, LT>(job, P, p, f, d);
}

template <Kind KIND, typename LT>
hipError_t go_few(const Job &job, const Params &p, uint32_t super_groups, hipStream_t s) {
  const size_t lds = (KIND == kDecompress ? (size_t)kOffLut4 * 4 : (size_t)p.blob_dwords * 4) + kFewWaves * 36;
  const uint32_t blocks = (super_groups + kFewWaves - 1) / kFewWaves;
  const dim3 block(kFewWaves * 64);
  OwnCheck check = {};
  if (take_own_check(job.src, &check)) hipLaunchKernelGGL((k_few<KIND, LT, true>), dim3(blocks + 1), block, lds, s, job, p, check);
  else hipLaunchKernelGGL((k_few<KIND, LT, false>), dim3(blocks), block, lds, s, job, p, check);
  return hipGetLastError();
}

}  // namespace

// Super-groups per CU up to which one per wave is faster (us per call at 256 CUs, bf16, one per wave against tiles of four):
//   several widths, or 8- and 16-bit ones only: hop 32 (9,000: 6.05 against 5.85), decompress 40;
//   2- or 4-bit ones only, whose wide tiles run one short piece of code: 24 (6,144: hop 4.7 against 4.85; 7,000: 5.4 against 5.0; sink 3.8
//   against 4.0; 4.25 against 4.05);
//   with a check of indices armed, which the wide kernel leaves to a launch in front of it: hop and compress 48 (12,288: hop 10.2 against 10.6;
//   14,336: 11.5 against 11.0), decompress 64 (16,384: sink 10.8 against 10.95, in fp32 11.2 against 11.5; 18,432: 13.4 against 11.0), of two
//   different arrays 40: every block looks at every index.
// Tables larger than the default level sets' (21 KB) are copied by more blocks than they are worth here.
bool takes_few(Kind kind, const Job &job, const Params &P, uint32_t n_cu) {
  const uint64_t n = (uint64_t)job.n_sg[0] + job.n_sg[1] + job.n_sg[2] + job.n_sg[3], due = own_check_due();
  if (due == ~0ull || (kind != kDecompress && P.blob_dwords * 4 > kFewTableBytes)) return false;
  uint32_t most;
  if (due) most = due > n ? 40 : kind == kDecompress ? 64 : 48;
  else if (n == job.n_sg[0] || n == job.n_sg[1]) most = 24;
  else most = kind == kDecompress ? 40 : 32;
  return n <= (uint64_t)most * n_cu;
}

hipError_t launch_few(Kind kind, dq_dtype dtype, bool has_local, const Job &job, const Params &p, hipStream_t s) {
  const uint32_t n = job.n_sg[0] + job.n_sg[1] + job.n_sg[2] + job.n_sg[3];
  const bool f32 = dtype == DQ_F32;
  switch (kind) {
    case kCompress: return f32 ? go_few<kCompress, float>(job, p, n, s) : go_few<kCompress, uint16_t>(job, p, n, s);
    case kDar: return f32 ? go_few<kDar, float>(job, p, n, s) : go_few<kDar, uint16_t>(job, p, n, s);
    default:
      if (!has_local) return go_few<kDecompress, NoLocal>(job, p, n, s);
      return f32 ? go_few<kDecompress, float>(job, p, n, s) : go_few<kDecompress, uint16_t>(job, p, n, s);
  }
}

namespace {
template <Kind KIND, typename LT>
hipError_t static_lds_of(size_t *bytes) {
  const hipError_t e = add_static_lds(k_few<KIND, LT, false>, bytes);
  return e != hipSuccess ? e : add_static_lds(k_few<KIND, LT, true>, bytes);
}
}  // namespace

hipError_t few_static_lds(size_t *bytes) {
  hipError_t e = static_lds_of<kCompress, float>(bytes);
  if (e == hipSuccess) e = static_lds_of<kCompress, uint16_t>(bytes);
  if (e == hipSuccess) e = static_lds_of<kDar, float>(bytes);
  if (e == hipSuccess) e = static_lds_of<kDar, uint16_t>(bytes);
  if (e == hipSuccess) e = static_lds_of<kDecompress, float>(bytes);
  if (e == hipSuccess) e = static_lds_of<kDecompress, uint16_t>(bytes);
  return e != hipSuccess ? e : static_lds_of<kDecompress, NoLocal>(bytes);
}

}  // namespace dq
