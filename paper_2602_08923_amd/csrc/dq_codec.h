// Device code shared by the codec kernels (dq_kernels.hip: one hop per launch; dq_walk.hip: every hop of a
// schedule in one launch): LDS and global accesses, random numbers, where a tile sits, scales, the search
// for the level and the rounding (Section 3.3), and the decode.
#pragma once
#include "dq_device.h"

namespace dq {
namespace {

struct NoLocal {};
constexpr int kBatch = 8;  // tiles whose per-SG random numbers one wave-wide draw covers

__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }

// LDS accesses by byte address (the tables are addressed with folded constants)
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const uint32_t lds_u32;
typedef __attribute__((address_space(3))) const u32x2 lds_u2;
typedef __attribute__((address_space(3))) const u32x4 lds_u4;
typedef __attribute__((address_space(3))) u32x4 lds_w4;
__device__ __forceinline__ uint32_t lds_ld1(uint32_t a) { return *reinterpret_cast<lds_u32 *>(a); }
__device__ __forceinline__ u32x2 lds_ld2(uint32_t a) { return *reinterpret_cast<lds_u2 *>(a); }
__device__ __forceinline__ u32x4 lds_ld4(uint32_t a) { return *reinterpret_cast<lds_u4 *>(a); }
__device__ __forceinline__ void lds_st1(uint32_t a, uint32_t v) {
  *reinterpret_cast<__attribute__((address_space(3))) uint32_t *>(a) = v;
}
__device__ __forceinline__ void lds_st4(uint32_t a, u32x4 v) { *reinterpret_cast<lds_w4 *>(a) = v; }
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) f32x4 lds_f4;
__device__ __forceinline__ void lds_stf4(uint32_t a, f32x4 v) { *reinterpret_cast<lds_f4 *>(a) = v; }
__device__ __forceinline__ f32x4 lds_ldf4(uint32_t a) { return *reinterpret_cast<const lds_f4 *>(a); }

// Global-memory accesses through explicit address-space-1 pointers.  The job's pointers reach
// the kernel inside a struct, where the compiler would otherwise treat them as generic and
// emit FLAT instructions; those also count on the LDS counter, so every wait for a table
// lookup would wait for the outstanding global loads and stores as well.
template <typename T>
__device__ __forceinline__ T gld(const void *p) {
  return *(const __attribute__((address_space(1))) T *)p;
}
template <typename T>
__device__ __forceinline__ void gst(void *p, T v) {
  *(__attribute__((address_space(1))) T *)p = v;
}
__device__ __forceinline__ uint4 gld16(const void *p) {
  const u32x4 t = gld<u32x4>(p);
  return make_uint4(t.x, t.y, t.z, t.w);
}
// A store that leaves the caches first, for the fp32 results: whole lines, the largest stream a launch writes, and none of its own
// reads.  Sinks of 125 M entries 193 -> 187 us, eight 25 MB buffers' ring 78 -> 75 us.  (The packed codes and the loads
// are better off in the caches, where the next launch or the neighbouring tile finds them.)
template <typename T>
__device__ __forceinline__ void gst_once(void *p, T v) {
  __builtin_nontemporal_store(v, (__attribute__((address_space(1))) T *)p);
}
// ---- Philox4x32-10 (Salmon et al., SC'11): counter-based, so every lane draws its numbers
// from (global group index, round, stream, rank) alone.
struct U4 {
  uint32_t x, y, z, w;
};

// a ^ b ^ c in one instruction (three-input bitwise operation, truth table 0x96)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3, uint32_t k0,
                                            uint32_t k1) {
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t a = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t b = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = a;
    c2 = b;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return U4{c0, c1, c2, c3};
}

// ---- max over the 16 lanes of a DPP row, result in every lane of the row
// (the operands are magnitudes, so the order of their bit patterns is the order of the values)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ float row_max16(float m) {
  uint32_t x = f2u(m);
  x = max(x, dpp_u<0x128>(x));  // row_ror:8
  x = max(x, dpp_u<0x124>(x));  // row_ror:4
  x = max(x, dpp_u<0x122>(x));  // row_ror:2
  x = max(x, dpp_u<0x121>(x));  // row_ror:1
  return u2f(x);
}

// With E = 4 or 8 entries per lane: maximum of magnitudes over the lanes of a group, then over those of a super-group.
template <int E>
__device__ __forceinline__ uint32_t group_max(uint32_t x) {
  x = max(x, dpp_u<0xB1>(x));                        // quad_perm 1,0,3,2
  if constexpr (E == 4) x = max(x, dpp_u<0x4E>(x));  // quad_perm 2,3,0,1
  return x;
}
template <int E>
__device__ __forceinline__ uint32_t sg_max(uint32_t x) {  // x: the group's maximum
  if constexpr (E == 8) x = max(x, dpp_u<0x122>(x));  // row_ror:2
  x = max(x, dpp_u<0x124>(x));                        // row_ror:4
  x = max(x, dpp_u<0x128>(x));                        // row_ror:8
  const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);  // rows 0 and 1, 2 and 3
  x = max(a[0], a[1]);
  if constexpr (E == 4) {
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);  // the wave's halves
    x = max(b[0], b[1]);
  }
  return x;
}

template <int B>
struct Width;
template <>
struct Width<2> { static constexpr int words = 1; };
template <>
struct Width<4> { static constexpr int words = 2; };
template <>
struct Width<8> { static constexpr int words = 4; };

// LDS byte addresses of the tables.  The blob sits at LDS byte 0 (these kernels have dynamic LDS
// only), so the fixed-size tables are compile-time constants that the compiler folds into the
// offset field of the LDS instructions; only the two search tables, whose size varies, are found through parameters (Params::magic).
constexpr uint32_t kLds0 = 0;
constexpr uint32_t kRec0 = kLds0 + kOffRec * 4;
struct HopTables {
  template <int B>
  static constexpr uint32_t dec() { return kLds0 + (B == 2 ? kOffDec2 : (B == 4 ? kOffDec4 : kOffDec8)) * 4; }
};
// Where a tile (index t in the job's concatenated 2-, 4-, 8-, 16-bit tile sequence) sits.
struct TilePos {
  uint32_t seg_first;   // position in the chunk of the first SG of the tile's width
  uint32_t n_seg;       // SGs of that width in the chunk
  uint32_t tile_first;  // first SG of the tile inside the segment
  int wi;
};
__device__ __forceinline__ TilePos locate(const Job &job, uint32_t t) {
  const uint32_t n0 = job.n_sg[0], n1 = job.n_sg[1], n2 = job.n_sg[2], n3 = job.n_sg[3];
  const uint32_t t0 = (n0 + kWaveSGs - 1) / kWaveSGs, t1 = (n1 + kWaveSGs - 1) / kWaveSGs,
                 t2 = (n2 + kWaveSGs - 1) / kWaveSGs;
  if (t < t0) return TilePos{0, n0, t * kWaveSGs, 0};
  if (t < t0 + t1) return TilePos{n0, n1, (t - t0) * kWaveSGs, 1};
  if (t < t0 + t1 + t2) return TilePos{n0 + n1, n2, (t - t0 - t1) * kWaveSGs, 2};
  return TilePos{n0 + n1 + n2, n3, (t - t0 - t1 - t2) * kWaveSGs, 3};
}

// Wave-uniform addresses of a tile: 64-bit bases once per tile (scalar registers), so that
// every lane only adds a small 32-bit offset.
template <int B>
struct TileBase {
  size_t code_off, gs_off, sf_off;  // byte offsets inside a packed buffer
  size_t first_entry;               // first entry of the tile inside the chunk
  uint32_t last_row;                // rows 0..last_row hold a super-group
  uint64_t G0;                      // global index of the tile's first super-group
  __device__ __forceinline__ TileBase(const Job &job, const TilePos pos) {
    const size_t n0 = job.n_sg[0], n1 = job.n_sg[1], n2 = job.n_sg[2], n3 = job.n_sg[3];
    const size_t c16 = 64 * n0 + 128 * n1 + 256 * n2;  // the raw 16-bit values follow the codes
    const size_t gs0 = c16 + 512 * n3;                  // then the scales of the coded SGs (2, 4, 8 bits)
    const size_t sg0 = (size_t)pos.seg_first + pos.tile_first;  // position in the chunk
    code_off = (B == 2 ? 0 : (B == 4 ? 64 * n0 : (B == 8 ? 64 * n0 + 128 * n1 : c16))) + (size_t)pos.tile_first * (32 * B);
    gs_off = gs0 + sg0 * 16;
    sf_off = gs0 + 16 * (n0 + n1 + n2) + sg0 * 2;
    first_entry = sg0 * kSG;
    last_row = min((uint32_t)kWaveSGs - 1, pos.n_seg - 1 - pos.tile_first);
    G0 = job.first_sg + sg0;
  }
};

// sf_SG/255 and 255/sf_SG for a bf16 sf_SG without a division: the quotient of the 8-bit
// significand comes from a 128-entry table of correctly rounded values and the exponent is
// added on the bit pattern.  Scaling by a power of two commutes with rounding in the normal
// range, so these are exactly the IEEE quotients (encoders never store scales below 2^-100).
// The table's patterns already hold the exponent's bias ({quotient - bias, reciprocal + bias}),
// so a lookup takes one addition of the scale's exponent field in place.
__device__ __forceinline__ float sf_over_255(uint32_t sfb, uint32_t rec0) {
  const uint32_t q = lds_ld1(rec0 + (sfb & 0x7Fu) * 8);
  return sfb ? u2f(q + ((sfb << 16) & 0x7F800000u)) : 0.0f;
}

// Section 3.1: the mean of a super-group is subtracted from the local entries in fp32 where they
// enter (one operation per entry on the widened value).  job.mu holds one mean per super-group
// of the chunk, or is null.
__device__ __forceinline__ float local_mean(const Job &job, size_t first_entry, uint32_t row) {
  return job.mu ? gld<float>(job.mu + (first_entry / kSG) + row) : 0.0f;
}
// A lane's 16 local entries (group g of the super-group in row `row` of the tile) as raw 128-bit words.
// Without job.src they sit in the chunk's own order: a wave-uniform base plus a small lane offset.
// With job.src the super-group lives at index src[...] of `local` (the reorder of Section 3.5 done by
// addressing: the kernel gathers whole super-groups, 512 B or 1 KB each, from the original tensor).
// Kernels are built twice: the plain local types know no job.src at all (the compiler would otherwise
// merge the two paths' loads and pay a 64-bit per-lane address on both), the Gathered<> types look at it.
template <typename T>
struct Gathered { T x; };  // same size as T: sizeof(LT) keeps telling fp32 from bf16
template <typename LT>
struct IsGathered { static constexpr bool value = false; };
template <typename T>
struct IsGathered<Gathered<T>> { static constexpr bool value = true; };

template <typename LT>
__device__ __forceinline__ void load_local(const Job &job, size_t first_entry, uint32_t row, uint32_t g,
                                           uint4 (&loc)[sizeof(LT) == 4 ? 4 : 2]) {
  constexpr int kWords = sizeof(LT) == 4 ? 4 : 2;  // 128-bit words per group
  constexpr size_t kSgWords = kSG * sizeof(LT) / 16;
  const uint4 *base = static_cast<const uint4 *>(job.local);
  if constexpr (IsGathered<LT>::value) {
    if (job.src) {
      const size_t sg = gld<uint32_t>(job.src + first_entry / kSG + row);
      const uint4 *p = base + sg * kSgWords + g * kWords;
#pragma unroll
      for (int i = 0; i < kWords; ++i) loc[i] = gld16(p + i);
      return;
    }
  }
  const uint4 *p = base + (first_entry / kSG) * kSgWords + (row * 16 + g) * kWords;
#pragma unroll
  for (int i = 0; i < kWords; ++i) loc[i] = gld16(p + i);
}
template <typename LT>
__device__ __forceinline__ void widen_local(const uint4 (&loc)[sizeof(LT) == 4 ? 4 : 2], float (&v)[16]) {
  if constexpr (sizeof(LT) == 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[4 * i] = u2f(loc[i].x); v[4 * i + 1] = u2f(loc[i].y);
      v[4 * i + 2] = u2f(loc[i].z); v[4 * i + 3] = u2f(loc[i].w);
    }
  } else {  // bf16 widens exactly
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t w[4] = {loc[i].x, loc[i].y, loc[i].z, loc[i].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[8 * i + 2 * j] = u2f(w[j] << 16);
        v[8 * i + 2 * j + 1] = u2f(w[j] & 0xFFFF0000u);
      }
    }
  }
}
__device__ __forceinline__ void subtract_mean(const Job &job, float mu, float (&v)[16]) {
  if (job.mu) {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = v[k] - mu;
  }
}

// The shared random permutation pi of 0..n-1 (Section 3.3 "Correlated rounding") at one worker
// index, from the four words of the super-group's shared draw: three rounds of
//   y <- reverse_k(((w_t | 1) * y + (w_t >> 16)) mod 2^k),  k = ceil(log2 n)
// (odd multiply, add and bit reversal are bijections of the k-bit integers), walked again while
// the value is not below n, then rotated by floor(w3 * n / 2^32) so that every worker's slot is
// uniform.  Evaluated once per super-group and job (the rank is the job's), never per entry.
__device__ __forceinline__ uint32_t perm_slot(const U4 &d, const Params &P, uint32_t rank) {
  const uint32_t k = P.perm_bits, mask = (1u << k) - 1u, back = (32u - k) & 31u;
  const uint32_t w[3] = {d.x, d.y, d.z};
  auto rounds = [&](uint32_t y) {
#pragma unroll
    for (int t = 0; t < 3; ++t) y = __brev(((w[t] | 1u) * y + (w[t] >> 16)) & mask) >> back;
    return y;
  };
  uint32_t y = rounds(rank);
  if (P.n_workers & (P.n_workers - 1u))  // n is not a power of two: some k-bit values lie outside 0..n-1
    while (y >= P.n_workers) y = rounds(y);  // ends: the walk is a cycle through `rank` < n
  const uint32_t s = y + __umulhi(d.w, P.n_workers);
  return min(s, s - P.n_workers) & P.slot_keep;
}

__device__ __forceinline__ uint32_t bf16_rne_pair(float lo, float hi) {
  const uint32_t a = f2u(lo), b = f2u(hi);
  const uint32_t ra = (a + 0x7FFFu + ((a >> 16) & 1u)) >> 16;
  const uint32_t rb = (b + 0x7FFFu + ((b >> 16) & 1u)) & 0xFFFF0000u;
  return ra | rb;
}


// A wave tile's 4 KB of fp32 results, v[16] per lane (lane = group), written through the wave's
// LDS area so that every store instruction covers 1 KB of contiguous memory: lane l parks its 4
// float4 at slots 4l..4l+3 (slot index xor-ed with bits 2-3 of l so that the 16 lanes of a pass hit
// different banks); store round r then reads slot r*64 + lane = float4 number r*64 + lane of the tile.
__device__ __forceinline__ void store_tile_f32(const Job &job, const Params &P, float (&v)[16], uint32_t xpose,
                                               size_t first_entry, uint32_t last_row) {
  const uint32_t lane = threadIdx.x & 63u;
  const size_t sg0 = first_entry / kSG;  // the tile's first super-group inside the chunk
  if (job.back) {
    // Section 3.4, last paragraph: the mean comes back, n times (the sum of n workers' entries lost it n times)
    const float back = (float)P.n_workers * gld<float>(job.back + sg0 + min(lane >> 4, last_row));
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = v[k] + back;
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (uint32_t i = 0; i < 4; ++i)
    lds_stf4(xpose + lane * 64 + ((i ^ ((lane >> 2) & 3u)) * 16), f32x4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]});
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  float *out = static_cast<float *>(job.out);
#pragma unroll
  for (uint32_t r = 0; r < (uint32_t)kWaveSGs; ++r) {
    if (r > last_row) break;
    const uint32_t slot = r * 64 + lane, w = slot >> 2, c = slot & 3u;
    const f32x4 o = lds_ldf4(xpose + w * 64 + ((c ^ ((w >> 2) & 3u)) * 16));
    // row r is one super-group, 1 KB: at its place in the chunk, or where job.dest sends it
    const size_t sg = job.dest ? (size_t)gld<uint32_t>(job.dest + sg0 + r) : sg0 + r;
    gst_once<f32x4>(reinterpret_cast<float4 *>(out + sg * kSG) + lane, o);
  }
  __builtin_amdgcn_wave_barrier();
}

// 1 / m, correctly rounded, for m >= 2^-126 and infinity.  Below 2^126 the hardware's reciprocal, good to one unit in the last place, and
// one step on its exactly computed remainder (Markstein's theorem; which also leaves no exception here: every pattern is compared in
// tests/test_gpu_parity.py) are 3 instructions instead of the division's 10.  Quotients of larger m are denormal, which the reciprocal
// is not: a wave that has one divides.  One asm block, as the compiler schedules the code around a branch it knows of
// so much worse that nothing is gained.  Taken by the rings of dq_thin.hip, whose lanes divide once for four entries: 256 workers and 4,096
// super-groups 199.7 -> 193.3 us, 122 and 3,172 77.6 -> 75.7.  (Elsewhere the branch costs what the instructions save: a
// compress of 6,400 super-groups 5.3 -> 5.45, rings of four super-groups per tile within 1 % either way.)
__device__ __forceinline__ float reciprocal(float m) {
  float y, e, d, n, q;
  asm("v_rcp_f32 %0, %5\n\t"
      "s_nop 0\n\t"
      "v_fma_f32 %1, -%5, %0, 1.0\n\t"
      "v_cmp_ngt_f32 vcc, 0x7e800000, %5\n\t"  // 2^126
      "v_fma_f32 %0, %1, %0, %0\n\t"
      "s_cbranch_vccz .Lreciprocal%=\n\t"
      "v_div_scale_f32 %2, vcc, %5, %5, 1.0\n\t"
      "v_rcp_f32 %0, %2\n\t"
      "s_nop 0\n\t"
      "v_fma_f32 %1, -%2, %0, 1.0\n\t"
      "v_fma_f32 %0, %1, %0, %0\n\t"
      "v_div_scale_f32 %3, vcc, 1.0, %5, 1.0\n\t"
      "v_mul_f32 %4, %3, %0\n\t"
      "v_fma_f32 %1, -%2, %4, %3\n\t"
      "v_fma_f32 %4, %1, %0, %4\n\t"
      "v_fma_f32 %1, -%2, %4, %3\n\t"
      "s_nop 0\n\t"
      "v_div_fmas_f32 %0, %1, %0, %4\n\t"
      "v_div_fixup_f32 %0, %0, %5, 1.0\n"
      ".Lreciprocal%=:"
      : "=&v"(y), "=&v"(e), "=&v"(d), "=&v"(n), "=&v"(q)
      : "v"(m)
      : "vcc");
  return y;
}

// ---- one group's encoding (Section 3.3), in pieces: draw, scale, quantize
struct Draws {
  U4 gam;      // one byte per entry, private to the worker
  float o_pi;  // (slot of the shared permutation + 1/512) / n
  float us;    // the group scale's dither, (byte + 1/2) / 256
};
// slot0: this worker's slot of the super-group's permutation (group g uses slot0 + g mod n); sc_word: the word of
// the worker's scale stream that holds group g's byte.  g mod n is a nibble of P.g_mod (g itself above 16 workers),
// so slot0 + it is below 2n and one subtraction and minimum reduce it for any n.
__device__ __forceinline__ void draw_offsets(const Params &P, uint32_t slot0, uint32_t sc_word, uint32_t g, Draws &d) {
  const uint32_t s = slot0 + ((uint32_t)(P.g_mod >> (4 * g)) & 15u);
  const uint32_t slot = min(s, s - P.n_slots);
  d.o_pi = __builtin_fmaf((float)slot, P.inv_n, P.inv_n512);  // (slot + 1/512) * inv_n: the same real number, rounded once
  d.us = __builtin_fmaf((float)((sc_word >> (8 * (g & 3u))) & 0xFFu), 1.0f / 256.0f, 1.0f / 512.0f);  // exact
}
__device__ __forceinline__ Draws draw_group(const Params &P, uint64_t gi, uint32_t rank, uint32_t slot0, uint32_t sc_word,
                                            uint32_t g) {
  Draws d;
  d.gam = philox4x32_10((uint32_t)gi, (uint32_t)(gi >> 32), P.round, rank & 0xFFFFu, P.key0, P.key1);
  draw_offsets(P, slot0, sc_word, g, d);
  return d;
}

struct Scales {
  uint32_t rg, sfb;  // stored group scale (u8) and super-group scale (bf16 pattern)
  float inv;         // 1 / group maximum, 0 for a group whose scale rounded to zero (it keeps only its signs)
  float sfg;         // what the stored scales decode to: rg * (sf / 255)
};
// m, M: maxima of the group and of its super-group
__device__ __forceinline__ Scales scales_of(float m, float M, float us, uint32_t rec0) {
  Scales s;
  uint32_t b = f2u(M) + 0xFFFFu;         // upper half: smallest bf16 >= M
  b = b < 0x0D800000u ? 0u : b;          // below 2^-100: the super-group is encoded as zero
  s.sfb = b >> 16;
  const u32x2 q = lds_ld2(rec0 + ((b >> 13) & 0x3F8u));
  const uint32_t e = b & 0x7F800000u;
  // floor(ts) + [us < ts - floor(ts)] is the ceiling of ts - us: that difference is exact, or lies between -1 and 0
  const float rg = fabsf(ceilf(fminf(m * u2f(q.y - e), 255.0f) - us));
  s.rg = s.sfb ? (uint32_t)rg : 0u;
  s.inv = s.sfb && rg != 0.0f ? 1.0f / m : 0.0f;
  s.sfg = s.sfb ? rg * u2f(q.x + e) : 0.0f;
  return s;
}
__device__ __forceinline__ Scales scale_group(const float (&v)[16], float us, uint32_t rec0) {
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k) m = fmaxf(m, fabsf(v[k]));
  return scales_of(m, row_max16(m), us, rec0);
}

// Launch constants that vector instructions use once per entry, held in vector registers.  On this chip an
// instruction of the simple kind (mul, add, and/or/xor, right shift; fma nearly) whose operands are all vector registers
// or constants issues in little more than half the time of any other; with a scalar-register operand it is of the other
// kind itself.  (1.0 ns per wave instruction against 1.7, measured with eight waves per SIMD: profiles/valu_issue.txt.)
struct Vec {
  float magic4, magic8, s_n;
  uint32_t top;  // the sign bit
  __device__ __forceinline__ explicit Vec(const Params &P) : magic4(P.magic[1]), magic8(P.magic[2]), s_n(P.s_n), top(0x80000000u) {
    asm("" : "+v"(magic4), "+v"(magic8), "+v"(s_n), "+v"(top));
  }
};
// (a & b) | c as the three-input bitwise operation (the compiler's and-or is of the other kind)
__device__ __forceinline__ uint32_t or_and(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xEA);
}

// A level's entry {T, D, T of the next level, index << (32 - B)}, read as 16 bytes also where the index is not wanted: a 12-byte LDS read
// takes three times as long here (of the 14 entries of the 4-bit set 5.9 ns per instruction and CU against 1.8, of the 8-bit
// set's 254 8.5 against 5.1).  25 MB through a ring of eight, half of it 2-bit, is the same; a chain of 64 workers at 5 bits
// 436 -> 412 us, a ring of eight at 6 bits and 100 M entries 504 -> 486, of 8,192 super-groups 20.2 -> 19.5.
__device__ __forceinline__ u32x4 load_level(uint32_t a) { return lds_ld4(a); }

// The 16 entries of a group, quantized (v is consumed).
// x' = |v| * inv needs no clamp: |v| <= m and inv is the correctly rounded 1/m, so the exact
// product is at most 1 + 2^-24, which rounds to 1.  The product is taken with v's sign (xs): the
// magnitude serves the search and the rounding through source modifiers, the top bit is the
// code's sign bit (for inv = 0 the product is a zero with v's sign).
// CODES: the code words grow from the top: entry 15 first, each step shifts the word by one code and
// appends sign and level index, so the lowest entry of a word ends in its low bits.  A group
// whose scale rounded to zero has inv = 0, hence x' = 0 and level 0 throughout: only signs remain.
// LEVELS: v becomes the signed levels the codes stand for, what a decode of them would look up.
template <int B, bool CODES, bool LEVELS>
__device__ __forceinline__ void quantize(float (&v)[16], float inv, const U4 &gam, float o_pi, const Vec &V,
                                         uint32_t (&ow)[Width<B>::words]) {
  const uint32_t gw[4] = {gam.x, gam.y, gam.z, gam.w};
  auto uniform = [&](int k) { return __builtin_fmaf((float)((gw[k >> 2] >> (8 * (k & 3))) & 0xFFu), V.s_n, o_pi); };
  if constexpr (CODES) {
#pragma unroll
    for (int i = 0; i < Width<B>::words; ++i) ow[i] = 0;
  }
  if constexpr (B == 2) {
    // levels {0,1}: T + u*D = u, so the level bit is [u < x'] -- the sign bit of u - x' (the
    // difference of two different binary32 numbers is never zero)
#pragma unroll
    for (int k = 15; k >= 0; --k) {
      const float xs = v[k] * inv;
      const float u = uniform(k);
      if constexpr (CODES) {
        ow[0] = __builtin_amdgcn_alignbit(ow[0], f2u(xs), 31);                // (word << 1) | sign
        ow[0] = __builtin_amdgcn_alignbit(ow[0], f2u(u - fabsf(xs)), 31);  // (word << 1) | level
      }
      if constexpr (LEVELS) v[k] = u2f(or_and(f2u(xs), V.top, f2u(u < fabsf(xs) ? 1.0f : 0.0f)));
    }
  } else {
    // Two dependent table reads per entry, in a pipeline of three stages over groups of kG entries: while a group's
    // level is being picked, the next group's level entry and the one after's search entry are on their way.  (Left
    // to itself the compiler reads, waits, reads, waits entry by entry: 32 trips to LDS in a row.)
    constexpr int kG = 2, kGroups = 16 / kG;
    const float magic = B == 4 ? V.magic4 : V.magic8;
    constexpr int per_word = 32 / B;
    u32x2 e[2][kG];
    u32x4 t[2][kG];
    // search: adding the magic number leaves the search table's LDS address plus round(x * 2^(m+3)) in the low
    // mantissa bits; without its three lowest bits that is the address of entry q = that integer / 8
    auto search = [&](int g) {
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        float &x = v[15 - g * kG - j];
        x = x * inv;
        e[g & 1][j] = lds_ld2(f2u(fabsf(x) + magic) & 0x1FFF8u);
      }
    };
    // the level at or below x' is the candidate's, or the next if x' >= T[next]: the sign of x' - T[next]
    // (exact zero only for equal operands) picks one of the pair's two entries
    auto level = [&](int g) {
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        const u32x2 q = e[g & 1][j];
        t[g & 1][j] = load_level(or_and(f2u(fabsf(v[15 - g * kG - j]) - u2f(q.x)) >> 27, 16u, q.y));
      }
    };
    auto round = [&](int g) {
#pragma unroll
      for (int j = 0; j < kG; ++j) {
        const int k = 15 - g * kG - j;
        const float xs = v[k], x = fabsf(xs);
        const u32x4 q = t[g & 1][j];
        const float theta = __builtin_fmaf(uniform(k), u2f(q.y), u2f(q.x));  // below x': round up
        if constexpr (CODES) {
          // append sign and level index in one funnel shift, then the rounding: level index + 1 <= R, no carry into the sign
          const uint32_t w = __builtin_amdgcn_alignbit(ow[k / per_word], or_and(f2u(xs), V.top, q.w), 32 - B);
          ow[k / per_word] = w + (f2u(theta - x) >> 31);
        }
        if constexpr (LEVELS) v[k] = u2f(or_and(f2u(xs), V.top, theta < x ? q.z : q.x));
      }
    };
    search(0);
    __builtin_amdgcn_sched_barrier(0);
    search(1);
    level(0);
#pragma unroll
    for (int g = 0; g < kGroups; ++g) {
      __builtin_amdgcn_sched_barrier(0);
      if (g + 2 < kGroups) search(g + 2);
      if (g + 1 < kGroups) level(g + 1);
      round(g);
    }
  }
}

// f(k, signed level) for the 16 entries of a group's code words: one table entry per code byte.
template <int B, typename LDS, typename F>
__device__ __forceinline__ void each_level(const uint32_t (&cw)[Width<B>::words], F f) {
  constexpr uint32_t dec0 = LDS::template dec<B>();
#pragma unroll
  for (int j = 0; j < 2 * B; ++j) {
    constexpr uint32_t kStride = 32 / B;  // bytes per table entry: 8/B levels
    constexpr uint32_t kLog = B == 2 ? 4 : (B == 4 ? 3 : 2);
    const uint32_t w = cw[j >> 2], sh = 8 * (j & 3);
    uint32_t at = sh >= kLog ? w >> (sh - kLog) : w << (kLog - sh);
    asm("" : "+v"(at));  // shift and mask, two simple instructions: not a bit-field extract and a left shift
    at &= 0xFFu << kLog;
    static_assert(kStride == 1u << kLog, "");
    if constexpr (B == 2) {
      const u32x4 e = lds_ld4(dec0 + at);
      f(4 * j, u2f(e.x)); f(4 * j + 1, u2f(e.y)); f(4 * j + 2, u2f(e.z)); f(4 * j + 3, u2f(e.w));
    } else if constexpr (B == 4) {
      const u32x2 e = lds_ld2(dec0 + at);
      f(2 * j, u2f(e.x)); f(2 * j + 1, u2f(e.y));
    } else {
      f(j, u2f(lds_ld1(dec0 + at)));
    }
  }
}

template <int B>
__device__ __forceinline__ void load_codes(const void *p, uint32_t (&cw)[Width<B>::words]) {
  if constexpr (B == 2) {
    cw[0] = gld<uint32_t>(p);
  } else if constexpr (B == 4) {
    const u32x2 t = gld<u32x2>(p);
    cw[0] = t.x; cw[1] = t.y;
  } else {
    const u32x4 t = gld<u32x4>(p);
    cw[0] = t.x; cw[1] = t.y; cw[2] = t.z; cw[3] = t.w;
  }
}
// Codes and scales of a lane's group (lg: group inside the tile; row: its super-group's row) into a packed chunk.
// Every lane stores: the idle rows of a ragged tile repeat the last super-group, and the 16 lanes of a row its scale.
template <int B>
__device__ __forceinline__ void store_codes(uint8_t *out, const TileBase<B> &tb, uint32_t lg, uint32_t row,
                                            const uint32_t (&ow)[Width<B>::words], uint32_t rg, uint32_t sfb) {
  uint8_t *cp = out + tb.code_off + lg * (2 * B);
  if constexpr (B == 2) {
    gst<uint32_t>(cp, ow[0]);
  } else if constexpr (B == 4) {
    gst<u32x2>(cp, u32x2{ow[0], ow[1]});
  } else {
    gst<u32x4>(cp, u32x4{ow[0], ow[1], ow[2], ow[3]});
  }
  gst<uint8_t>(out + tb.gs_off + lg, (uint8_t)rg);
  gst<uint16_t>(out + tb.sf_off + row * 2, (uint16_t)sfb);
}

}  // namespace
}  // namespace dq
