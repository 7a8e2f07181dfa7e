// OCP Microscaling (MXFP8 E4M3 / MXFP6 E3M2 / MXFP4 E2M1) versions of compress, DAR and
// decompress(+accumulate) -- the comparison codec of the paper's evaluation (Section 5,
// "Baseline compression schemes") run in the same hop loop.  Conversion per the OCP MX v1.0
// specification: shared exponent floor(log2 max|v|) - emax_elem stored as an E8M0 byte,
// elements rounded to nearest-even and clamped to the largest normal.
//
// Mapping: one lane owns one block of 32 entries (its maximum is in-lane); a wave64 covers
// 2048 entries per tile.
#include <type_traits>

#include "dq_device.h"

namespace dq {
namespace {

struct NoLocal {};

__device__ __forceinline__ uint32_t f2u(float f) { return __builtin_bit_cast(uint32_t, f); }
__device__ __forceinline__ float u2f(uint32_t u) { return __builtin_bit_cast(float, u); }

// explicit global (address space 1) accesses: the job's pointers arrive inside a struct and
// would otherwise be treated as generic, i.e. FLAT instructions
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename T>
__device__ __forceinline__ T gld(const void *p) {
  return *(const __attribute__((address_space(1))) T *)p;
}
template <typename T>
__device__ __forceinline__ void gst(void *p, T v) {
  *(__attribute__((address_space(1))) T *)p = v;
}

typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
__device__ __forceinline__ void lds_put(uint32_t a, f32x4 v) { *reinterpret_cast<lds_f32x4 *>(a) = v; }
__device__ __forceinline__ f32x4 lds_get(uint32_t a) { return *reinterpret_cast<const lds_f32x4 *>(a); }

template <int FMT>
struct Fmt;
template <>
struct Fmt<DQ_MXFP8_E4M3> { static constexpr int emax = 8, cb = 8; };  // largest exponent, code bits
template <>
struct Fmt<DQ_MXFP6_E3M2> { static constexpr int emax = 4, cb = 6; };
template <>
struct Fmt<DQ_MXFP4_E2M1> { static constexpr int emax = 2, cb = 4; };

template <typename LT>
__device__ __forceinline__ void load_local32(const void *base, size_t first, float (&v)[32]) {
  if constexpr (sizeof(LT) == 4) {
    const float4 *p = reinterpret_cast<const float4 *>(static_cast<const float *>(base) + first);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const f32x4 t = gld<f32x4>(p + i);
      v[4 * i] = t.x; v[4 * i + 1] = t.y; v[4 * i + 2] = t.z; v[4 * i + 3] = t.w;
    }
  } else {
    const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(base) + first);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4 t = gld<u32x4>(p + i);
      const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[8 * i + 2 * j] = u2f(w[j] << 16);
        v[8 * i + 2 * j + 1] = u2f(w[j] & 0xFFFF0000u);
      }
    }
  }
}

// One block of 32 entries per lane, converted by gfx950's scaled conversion instructions
// (V_CVT_SCALEF32_*): packed elements <-> fp32 with the block scale applied in the same
// instruction, round to nearest even.  What measurement against the CPU oracle showed about them:
//   - the scale operand is a binary32 whose exponent FIELD is taken as the E8M0 byte (so the
//     pattern e << 23 is passed, also for e = 0);
//   - the E4M3 narrowing turns overflow into NaN (0x7F) where MX saturates: values are clamped
//     to +-448 * 2^(e-127) first (same result as round-then-saturate); E3M2 and E2M1 saturate;
//   - the instruction set's "fp6" is E2M3; OCP's MXFP6 E3M2 is its "bf6";
//   - the 32-wide 6-bit narrowing interleaves its two 16-entry inputs (a0 b0 a1 b1 ...), the
//     widening returns entries in order.
// Decoded element * scale is exact in binary32 for every code and scale byte, so adding the
// local entry afterwards is the single-rounding fma the conversion rule asks for.
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x32 __attribute__((ext_vector_type(32)));

// 32 entries (in the order a0 b0 a1 b1 ...) to 6-bit codes.  The instruction works in several passes, and the compiler may give
// its result the registers of an operand that dies here: with the scale's, later passes met another scale.  So the operands live on
// behind it.
__device__ __forceinline__ u32x6 to_bf6(const f32x16 &a, const f32x16 &b, float X) {
  u32x6 r = __builtin_amdgcn_cvt_scalef32_2xpk16_bf6_f32(a, b, X);
  asm("" : "+v"(r) : "v"(a), "v"(b), "v"(X));
  return r;
}

// A block's code words and scale byte.
template <int FMT>
struct MxMsg {
  uint32_t w[Fmt<FMT>::cb], e;
};
template <int FMT>
__device__ __forceinline__ MxMsg<FMT> mx_load(const uint8_t *packed, uint64_t n_blocks, uint64_t bl) {
  constexpr int cw = Fmt<FMT>::cb;
  MxMsg<FMT> m;
  const uint8_t *src = packed + (size_t)bl * (cw * 4);
  if constexpr (cw == 8) {
    const u32x4 a = gld<u32x4>(src), b = gld<u32x4>(src + 16);
    m.w[0] = a.x; m.w[1] = a.y; m.w[2] = a.z; m.w[3] = a.w; m.w[4] = b.x; m.w[5] = b.y; m.w[6] = b.z; m.w[7] = b.w;
  } else if constexpr (cw == 6) {
    const u32x2 a = gld<u32x2>(src), b = gld<u32x2>(src + 8), c = gld<u32x2>(src + 16);
    m.w[0] = a.x; m.w[1] = a.y; m.w[2] = b.x; m.w[3] = b.y; m.w[4] = c.x; m.w[5] = c.y;
  } else {
    const u32x4 a = gld<u32x4>(src);
    m.w[0] = a.x; m.w[1] = a.y; m.w[2] = a.z; m.w[3] = a.w;
  }
  m.e = gld<uint8_t>(packed + (size_t)n_blocks * (cw * 4) + bl);
  return m;
}
template <int FMT>
__device__ __forceinline__ void mx_store(uint8_t *packed, uint64_t n_blocks, uint64_t bl, const MxMsg<FMT> &m) {
  constexpr int cw = Fmt<FMT>::cb;
  uint8_t *dst = packed + (size_t)bl * (cw * 4);
  if constexpr (cw == 8) {
    gst<u32x4>(dst, u32x4{m.w[0], m.w[1], m.w[2], m.w[3]});
    gst<u32x4>(dst + 16, u32x4{m.w[4], m.w[5], m.w[6], m.w[7]});
  } else if constexpr (cw == 6) {
    gst<u32x2>(dst, u32x2{m.w[0], m.w[1]});
    gst<u32x2>(dst + 8, u32x2{m.w[2], m.w[3]});
    gst<u32x2>(dst + 16, u32x2{m.w[4], m.w[5]});
  } else {
    gst<u32x4>(dst, u32x4{m.w[0], m.w[1], m.w[2], m.w[3]});
  }
  gst<uint8_t>(packed + (size_t)n_blocks * (cw * 4) + bl, (uint8_t)m.e);
}
// v = decoded block (ADD: + v)
template <int FMT, bool ADD>
__device__ __forceinline__ void mx_decode(const MxMsg<FMT> &m, float (&v)[32]) {
  constexpr int cw = Fmt<FMT>::cb;
  const float X = u2f(m.e << 23);  // the instruction reads the exponent field as the E8M0 scale
  float d[32];
  if constexpr (cw == 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const f32x2 lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(m.w[i], X, false);
      const f32x2 hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(m.w[i], X, true);
      d[4 * i] = lo.x; d[4 * i + 1] = lo.y; d[4 * i + 2] = hi.x; d[4 * i + 3] = hi.y;
    }
  } else if constexpr (cw == 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x2 b0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[i], X, 0);
      const f32x2 b1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[i], X, 1);
      const f32x2 b2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[i], X, 2);
      const f32x2 b3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[i], X, 3);
      d[8 * i] = b0.x; d[8 * i + 1] = b0.y; d[8 * i + 2] = b1.x; d[8 * i + 3] = b1.y;
      d[8 * i + 4] = b2.x; d[8 * i + 5] = b2.y; d[8 * i + 6] = b3.x; d[8 * i + 7] = b3.y;
    }
  } else {
    const f32x32 all = __builtin_amdgcn_cvt_scalef32_pk32_f32_bf6(u32x6{m.w[0], m.w[1], m.w[2], m.w[3], m.w[4], m.w[5]}, X);
#pragma unroll
    for (int k = 0; k < 32; ++k) d[k] = all[k];
  }
#pragma unroll
  for (int k = 0; k < 32; ++k) v[k] = ADD ? d[k] + v[k] : d[k];
}
template <int FMT>
__device__ __forceinline__ MxMsg<FMT> mx_encode(float (&v)[32]) {
  using F = Fmt<FMT>;
  constexpr int cw = F::cb;
  MxMsg<FMT> out;
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < 32; ++k) m = fmaxf(m, fabsf(v[k]));
  int e = (int)(f2u(m) >> 23) - F::emax;
  e = e < 0 ? 0 : (e > 254 ? 254 : e);
  const float X = u2f((uint32_t)e << 23);
  if constexpr (cw == 8) {
    // the E4M3 conversion turns overflow into NaN; MX saturates: clamp to the largest normal first
    const float top = 448.0f * X;
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = __builtin_amdgcn_fmed3f(v[k], -top, top);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      s16x2 r = {0, 0};
      r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, v[4 * i], v[4 * i + 1], X, false);
      r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, v[4 * i + 2], v[4 * i + 3], X, true);
      out.w[i] = __builtin_bit_cast(uint32_t, r);
    }
  } else if constexpr (cw == 4) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint32_t r = 0;
      r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * i], v[8 * i + 1], X, 0);
      r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * i + 2], v[8 * i + 3], X, 1);
      r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * i + 4], v[8 * i + 5], X, 2);
      r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[8 * i + 6], v[8 * i + 7], X, 3);
      out.w[i] = r;
    }
  } else {
    f32x16 a, b;
#pragma unroll
    for (int k = 0; k < 16; ++k) { a[k] = v[2 * k]; b[k] = v[2 * k + 1]; }  // the two inputs interleave
    const u32x6 r = to_bf6(a, b, X);
#pragma unroll
    for (int i = 0; i < 6; ++i) out.w[i] = r[i];
  }
  out.e = (uint32_t)e;
  return out;
}
// The wave's 64 blocks, 8 KB of consecutive output from `out` on (n_valid of them exist).  Lane l parks its 8 float4
// in the wave's LDS area (slot index xor-ed with l % 8 against bank conflicts); round r then stores float4
// number 64 r + l of the tile, 1 KB of consecutive memory per instruction.
__device__ __forceinline__ void mx_store_f32(float *out, uint64_t n_valid, const float (&v)[32], uint32_t xpose) {
  const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
  for (uint32_t c = 0; c < 8; ++c)
    lds_put(xpose + lane * 128 + ((c ^ (lane & 7u)) * 16), f32x4{v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]});
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  float4 *o = reinterpret_cast<float4 *>(out);
#pragma unroll
  for (uint32_t r = 0; r < 8; ++r) {
    const uint32_t L = r * 64 + lane, w = L >> 3, c = L & 7u;
    if (w < n_valid) gst<f32x4>(o + L, lds_get(xpose + w * 128 + ((c ^ (w & 7u)) * 16)));
  }
  __builtin_amdgcn_wave_barrier();  // the area is reused by the wave's next tile
}

template <int FMT, Kind KIND, typename LT>
__device__ __forceinline__ void mx_block(const MxJob &job, uint64_t bi, uint64_t n_blocks, bool active, uint32_t xpose) {
  constexpr bool kHasLocal = !__is_same(LT, NoLocal);
  const uint64_t bl = active ? bi : n_blocks - 1;  // block whose inputs this lane reads
  float v[32];
  if constexpr (kHasLocal) load_local32<LT>(job.local, (size_t)bl * 32, v);
  if constexpr (KIND != kCompress) mx_decode<FMT, kHasLocal>(mx_load<FMT>(job.in, n_blocks, bl), v);
  if constexpr (KIND == kDecompress) {
    const uint64_t first = bi - (threadIdx.x & 63u);  // first block of the wave's tile
    mx_store_f32(static_cast<float *>(job.out) + (size_t)first * 32, n_blocks - first, v, xpose);
  } else {
    mx_store<FMT>(static_cast<uint8_t *>(job.out), n_blocks, bi, mx_encode<FMT>(v));
  }
}

template <int FMT, Kind KIND, typename LT>
__device__ __forceinline__ void mx_run(const MxJob &job) {
  const uint64_t n_blocks = job.n_entries / 32;
  const uint64_t stride = (uint64_t)gridDim.x * kBlockThreads;
  if constexpr (KIND == kDecompress) {
    // whole waves walk the tiles of 64 blocks together (the stores are a wave-wide transpose);
    // lanes past the end of a ragged last tile redo the last block and store nothing
    __shared__ float4 park[kBlockWaves * 512];  // 8 KB per wave
    const uint32_t xpose = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float4 *)park + (threadIdx.x >> 6) * 8192;
    const uint64_t first = (uint64_t)blockIdx.x * kBlockThreads + (threadIdx.x & ~63u);
    for (uint64_t t0 = first; t0 < n_blocks; t0 += stride) {
      const uint64_t bi = t0 + (threadIdx.x & 63u);
      mx_block<FMT, KIND, LT>(job, bi, n_blocks, bi < n_blocks, xpose);
    }
  } else {
    for (uint64_t bi = (uint64_t)blockIdx.x * kBlockThreads + threadIdx.x; bi < n_blocks; bi += stride)
      mx_block<FMT, KIND, LT>(job, bi, n_blocks, true, 0u);
  }
}

template <int FMT, Kind KIND, typename LT>
__global__ __launch_bounds__(kBlockThreads) void mx_one(MxJob job) {
  mx_run<FMT, KIND, LT>(job);
}
template <int FMT, Kind KIND, typename LT>
__global__ __launch_bounds__(kBlockThreads) void mx_batch(const MxJob *jobs) {
  const MxJob job = jobs[blockIdx.y];
  mx_run<FMT, KIND, LT>(job);
}

// A whole replay in one launch, as in dq_walk.hip (mx_walk; small and very large ones: mx_quad below): a wave carries 64 blocks of a chunk through all hops of the schedule,
// the pending message in registers (a recursive halving's higher levels in LDS).  A replay of a ring of 8 over 25 MB: 57 us, 4.6 TB/s,
// the rate of a large copy on this card; 94 us in eight launches, bound by the messages' way to memory and back and
// by the launches' fixed parts.  Three waves per SIMD without spills beat four with (57 and 59 us); grids of 3 to 7 blocks
// per CU are within 3 %.
constexpr uint32_t kMxStackLevel = 36 * 64;  // eight code words and the scale per lane
constexpr uint32_t kMxXpose = 8192;

template <bool TREE>
__device__ __forceinline__ uint32_t mx_leaf(const MxWalk &W, uint32_t chunk, uint32_t i) {
  if constexpr (TREE) {
    return chunk ^ (__brev(~i) >> (32u - W.log_n));
  } else {
    const uint32_t x = (W.chain ? 0u : chunk) + i;
    return min(x, x - W.n);
  }
}
template <typename LT>
struct MxSlice {
  u32x4 w[sizeof(LT) == 4 ? 8 : 4];
};
template <typename LT>
__device__ __forceinline__ MxSlice<LT> mx_slice(const MxWalk &W, uint32_t leaf, uint64_t at) {
  typedef __attribute__((address_space(4))) const uint64_t constant_u64;  // a scalar load: nothing here writes the table
  const uint8_t *p = reinterpret_cast<const uint8_t *>(((constant_u64 *)(uintptr_t)W.grads)[leaf]) + at;
  MxSlice<LT> s;
#pragma unroll
  for (int i = 0; i < (sizeof(LT) == 4 ? 8 : 4); ++i) s.w[i] = gld<u32x4>(p + 16 * i);
  return s;
}
template <typename LT>
__device__ __forceinline__ void mx_widen(const MxSlice<LT> &s, float (&v)[32]) {
  if constexpr (sizeof(LT) == 4) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[4 * i] = u2f(s.w[i].x); v[4 * i + 1] = u2f(s.w[i].y); v[4 * i + 2] = u2f(s.w[i].z); v[4 * i + 3] = u2f(s.w[i].w);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w[4] = {s.w[i].x, s.w[i].y, s.w[i].z, s.w[i].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[8 * i + 2 * j] = u2f(w[j] << 16);
        v[8 * i + 2 * j + 1] = u2f(w[j] & 0xFFFF0000u);
      }
    }
  }
}

template <int FMT, typename LT, bool TREE>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(3))) void mx_walk(MxWalk W) {
  extern __shared__ float4 mx_lds[];
  constexpr int cw = Fmt<FMT>::cb;
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t area = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float4 *)mx_lds + wave * W.wave_bytes;
  const uint32_t n_waves = gridDim.x * kBlockWaves, last = W.n - 1;
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  // tile t: blocks [64 k, 64 k + 64) of path p's chunk
  struct Tile {
    uint32_t path, chunk;
    uint64_t first;  // the wave's first block inside the chunk
    uint64_t at;     // this lane's block inside every worker's tensor, in bytes
  };
  auto tile = [&](uint32_t t) {
    Tile x;
    x.path = t / W.tiles_per_path;
    x.chunk = x.path % W.n_chunks;
    x.first = (uint64_t)(t - x.path * W.tiles_per_path) * 64;
    const uint64_t bl = min(x.first + lane, W.chunk_blocks - 1);  // lanes past the end redo the last block
    x.at = ((uint64_t)x.path * W.chunk_blocks + bl) * (32 * sizeof(LT));
    return x;
  };
  uint32_t t = __builtin_amdgcn_readfirstlane(blockIdx.x * kBlockWaves + wave);
  if (t >= W.n_tiles) return;
  Tile x = tile(t);
  MxSlice<LT> s = mx_slice<LT>(W, mx_leaf<TREE>(W, x.chunk, 0u), x.at);
  for (;;) {
    const bool more = W.n_tiles - t > n_waves;
    const Tile next = more ? tile(t + n_waves) : x;
    const uint64_t bl = min(x.first + lane, W.chunk_blocks - 1);
    float v[32];
    MxMsg<FMT> m;
#pragma unroll 1
    for (uint32_t i = 0;; ++i) {
      mx_widen<LT>(s, v);
      if (i < last) s = mx_slice<LT>(W, mx_leaf<TREE>(W, x.chunk, i + 1), x.at);
      else if (more) s = mx_slice<LT>(W, mx_leaf<TREE>(W, next.chunk, 0u), next.at);
      if (TREE ? (i & 1u) : i > 0) mx_decode<FMT, true>(m, v);
      uint32_t stack = area;
      if constexpr (TREE) {
        if (i & 1u) {
#pragma unroll 1
          for (uint32_t q = i >> 1; q & 1u; q >>= 1, stack += kMxStackLevel) {
            MxMsg<FMT> p;
#pragma unroll
            for (int k = 0; k < cw; ++k) p.w[k] = *reinterpret_cast<lds_u32 *>(stack + k * 256 + lane * 4);
            p.e = *reinterpret_cast<lds_u32 *>(stack + 2048 + lane * 4);
            mx_decode<FMT, true>(p, v);
          }
        }
      }
      if (i == W.encodes) break;
      m = mx_encode<FMT>(v);
      if (i == last) {  // all-gather: what every worker decodes from the sink's message
        mx_decode<FMT, false>(m, v);
        break;
      }
      if constexpr (TREE) {
        if (i & 1u) {
#pragma unroll
          for (int k = 0; k < cw; ++k) *reinterpret_cast<lds_u32 *>(stack + k * 256 + lane * 4) = m.w[k];
          *reinterpret_cast<lds_u32 *>(stack + 2048 + lane * 4) = m.e;
        }
      } else if (i >= W.first_kept) {
        mx_store<FMT>(W.msg[i & 1u] + (size_t)x.path * W.msg_stride, W.chunk_blocks, bl, m);
      }
    }
    mx_store_f32(W.out + ((uint64_t)x.path * W.chunk_blocks + x.first) * 32, W.chunk_blocks - x.first, v, area);
    if (!more) break;
    t += n_waves;
    x = next;
  }
}

// The same with four lanes to a block, eight entries each: a tile of 16 blocks per wave, eight leaves requested ahead.
//
// Why: with a lane per block and one leaf ahead a replay of few tiles is a chain of trips to memory, 0.55 us (fp32: 0.95) for each worker
// whatever the size.  Eight entries leave registers for eight leaves (16 or 32 bytes each) on their way, a hop is a quarter as long, and
// there are four times as many waves.  Measured, us, walk -> this:
//   MXFP8 bf16, 2,048 super-groups: ring of 8 7.2 -> 4.9, of 64 34.8 -> 14.8; 4,096: 7.7 -> 5.9, 35.5 -> 24.6, of 256 180 -> 97
//   MXFP8 butterfly of 128 workers, 128 super-groups 73.5 -> 26.4, 4,096 79.8 -> 42.1; fp32, 16 workers, 4,096 18.1 -> 14.3
//   MXFP4 fp32 chain of 174 workers, 1,823 super-groups 166 -> 54.6 (the reads alone, at the rate of a large copy: 66)
//   MXFP8 fp32 ring of 8, 131,072 super-groups 256 -> 230; bf16 142 -> 132
// What bounds it: few tiles, instructions of a hop, one per four cycles and wave; many, memory.
constexpr uint32_t kQuadBlocks = 16;      // blocks per tile
constexpr uint32_t kQuadLevel = 12 * 64;  // two code words and the scale per lane
constexpr int kAhead = 8;                 // leaves on their way

// A lane's eight entries' codes (6-bit ones: in the first 48 bits; 4-bit ones: in the first word) and the block's scale byte.
struct QuadMsg {
  uint32_t w[2], e;
};
template <int FMT, bool ADD>
__device__ __forceinline__ void quad_decode(const QuadMsg &m, float (&v)[8]) {
  constexpr int cw = Fmt<FMT>::cb;
  const float X = u2f(m.e << 23);
  float d[8];
  if constexpr (cw == 8) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const f32x2 lo = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(m.w[i], X, false);
      const f32x2 hi = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(m.w[i], X, true);
      d[4 * i] = lo.x; d[4 * i + 1] = lo.y; d[4 * i + 2] = hi.x; d[4 * i + 3] = hi.y;
    }
  } else if constexpr (cw == 4) {
    const f32x2 b0 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[0], X, 0);
    const f32x2 b1 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[0], X, 1);
    const f32x2 b2 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[0], X, 2);
    const f32x2 b3 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(m.w[0], X, 3);
    d[0] = b0.x; d[1] = b0.y; d[2] = b1.x; d[3] = b1.y; d[4] = b2.x; d[5] = b2.y; d[6] = b3.x; d[7] = b3.y;
  } else {  // the conversion takes 32 entries: a quarter of what it returns is used
    const f32x32 all = __builtin_amdgcn_cvt_scalef32_pk32_f32_bf6(u32x6{m.w[0], m.w[1], 0u, 0u, 0u, 0u}, X);
#pragma unroll
    for (int k = 0; k < 8; ++k) d[k] = all[k];
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = ADD ? d[k] + v[k] : d[k];
}
// The maximum of a block with a NaN among what the workers gave, as mx_encode finds it: the hardware's maximum turns a signalling NaN into a
// quiet one, so that only what comes behind it counts, and the order of all 32 entries does.  (A sum is never signalling.)
template <int CTRL>
__device__ __forceinline__ void quad_lane(const float (&v)[8], float *all) {  // the eight entries of one of the four lanes
#pragma unroll
  for (int k = 0; k < 8; ++k) all[k] = u2f((uint32_t)__builtin_amdgcn_mov_dpp((int)f2u(v[k]), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ uint32_t quad_nan_max(const float (&v)[8]) {
  float all[32], m = 0.0f;
  quad_lane<0x00>(v, all);
  quad_lane<0x55>(v, all + 8);
  quad_lane<0xAA>(v, all + 16);
  quad_lane<0xFF>(v, all + 24);
#pragma unroll
  for (int k = 0; k < 32; ++k) m = fmaxf(m, fabsf(all[k]));
  return f2u(m);
}
// given: v may be what a worker gave, not a sum
template <int FMT>
__device__ __forceinline__ QuadMsg quad_encode(float (&v)[8], bool given) {
  using F = Fmt<FMT>;
  constexpr int cw = F::cb;
  QuadMsg out;
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < 8; ++k) m = fmaxf(m, fabsf(v[k]));
  // bit patterns of values without a sign order as they do, and NaN is gone: the block's maximum over its four lanes
  uint32_t b = f2u(m);
  b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0xB1, 0xF, 0xF, true));  // quad_perm [1, 0, 3, 2]
  b = max(b, (uint32_t)__builtin_amdgcn_mov_dpp((int)b, 0x4E, 0xF, 0xF, true));  // quad_perm [2, 3, 0, 1]
  if (given) {
    const float sum = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    if (__builtin_amdgcn_ballot_w64(sum != sum)) b = quad_nan_max(v);
  }
  int e = (int)(b >> 23) - F::emax;
  e = e < 0 ? 0 : (e > 254 ? 254 : e);
  const float X = u2f((uint32_t)e << 23);
  out.w[1] = 0;
  if constexpr (cw == 8) {
    const float top = 448.0f * X;  // saturated before the conversion, as in mx_encode
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = __builtin_amdgcn_fmed3f(v[k], -top, top);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      s16x2 r = {0, 0};
      r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, v[4 * i], v[4 * i + 1], X, false);
      r = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(r, v[4 * i + 2], v[4 * i + 3], X, true);
      out.w[i] = __builtin_bit_cast(uint32_t, r);
    }
  } else if constexpr (cw == 4) {
    uint32_t r = 0;
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[0], v[1], X, 0);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[2], v[3], X, 1);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[4], v[5], X, 2);
    r = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(r, v[6], v[7], X, 3);
    out.w[0] = r;
  } else {
    f32x16 a, c;
#pragma unroll
    for (int k = 0; k < 16; ++k) { a[k] = v[2 * (k & 3)]; c[k] = v[2 * (k & 3) + 1]; }  // 32 entries: ours four times
    const u32x6 r = to_bf6(a, c, X);
    out.w[0] = r[0];
    out.w[1] = r[1] & 0xFFFFu;
  }
  out.e = (uint32_t)e;
  return out;
}
// lane: of the block, 0 to 3
template <int FMT>
__device__ __forceinline__ void quad_store(uint8_t *packed, uint64_t n_blocks, uint64_t bl, uint32_t lane, const QuadMsg &m) {
  constexpr int cw = Fmt<FMT>::cb;
  uint8_t *dst = packed + (size_t)bl * (cw * 4) + lane * cw;
  if constexpr (cw == 8) {
    gst<u32x2>(dst, u32x2{m.w[0], m.w[1]});
  } else if constexpr (cw == 4) {
    gst<uint32_t>(dst, m.w[0]);
  } else {  // six bytes at an even address
    gst<uint16_t>(dst, (uint16_t)m.w[0]);
    gst<uint16_t>(dst + 2, (uint16_t)(m.w[0] >> 16));
    gst<uint16_t>(dst + 4, (uint16_t)m.w[1]);
  }
  if (lane == 0) gst<uint8_t>(packed + (size_t)n_blocks * (cw * 4) + bl, (uint8_t)m.e);
}
template <typename LT>
struct QuadSlice {
  u32x4 w[sizeof(LT) == 4 ? 2 : 1];
};
template <typename LT>
__device__ __forceinline__ QuadSlice<LT> quad_slice(uint64_t tensor, uint64_t at) {
  const uint8_t *p = reinterpret_cast<const uint8_t *>(tensor) + at;
  QuadSlice<LT> s;
#pragma unroll
  for (int i = 0; i < (sizeof(LT) == 4 ? 2 : 1); ++i) s.w[i] = gld<u32x4>(p + 16 * i);
  return s;
}
template <typename LT>
__device__ __forceinline__ void quad_widen(const QuadSlice<LT> &s, float (&v)[8]) {
  if constexpr (sizeof(LT) == 4) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      v[4 * i] = u2f(s.w[i].x); v[4 * i + 1] = u2f(s.w[i].y); v[4 * i + 2] = u2f(s.w[i].z); v[4 * i + 3] = u2f(s.w[i].w);
    }
  } else {
    const uint32_t w[4] = {s.w[0].x, s.w[0].y, s.w[0].z, s.w[0].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[2 * j] = u2f(w[j] << 16);
      v[2 * j + 1] = u2f(w[j] & 0xFFFF0000u);
    }
  }
}

template <int FMT, typename LT, bool TREE>
__global__ __launch_bounds__(kBlockThreads) void mx_quad(MxWalk W) {
  extern __shared__ float4 mx_lds[];
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  [[maybe_unused]] const uint32_t area = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float4 *)mx_lds + wave * W.wave_bytes;
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  const uint32_t t = __builtin_amdgcn_readfirstlane(blockIdx.x * kBlockWaves + wave), last = W.n - 1, leaves = W.n;
  if (t >= W.n_tiles) return;
  const uint32_t path = t / W.tiles_per_path, chunk = path % W.n_chunks;
  const uint64_t bi = (uint64_t)(t - path * W.tiles_per_path) * kQuadBlocks + (lane >> 2);
  const uint64_t bl = min(bi, W.chunk_blocks - 1);  // lanes past the end redo the last block
  const uint64_t entry = ((uint64_t)path * W.chunk_blocks + bl) * 32 + (lane & 3u) * 8, at = entry * sizeof(LT);
  typedef __attribute__((address_space(4))) const uint64_t constant_u64;  // scalar loads: nothing here writes the table
  auto tensor = [&](uint32_t i) { return ((constant_u64 *)(uintptr_t)W.grads)[mx_leaf<TREE>(W, chunk, i)]; };
  // Behind the last leaf all lanes read the last tensor's first words, which costs next to nothing: with every request made, the wait for a
  // leaf leaves those behind it on their way.
  auto request = [&](uint64_t tensor, uint32_t i) { return quad_slice<LT>(tensor, i < leaves ? at : 0); };
  QuadSlice<LT> s[kAhead];
  uint64_t p[kAhead];
#pragma unroll
  for (uint32_t k = 0; k < kAhead; ++k) p[k] = tensor(min(k, last));
#pragma unroll
  for (uint32_t k = 0; k < kAhead; ++k) s[k] = request(p[k], k);
  float v[8];
  QuadMsg m;
  // leaf i0 + k; false: it was the last
  auto hop = [&](uint32_t i0, uint32_t k, QuadSlice<LT> &mine, auto refill, auto may_end) {
    const uint32_t i = i0 + k;
    quad_widen<LT>(mine, v);
    refill();
    if (TREE ? (i & 1u) : i > 0) quad_decode<FMT, true>(m, v);
    [[maybe_unused]] uint32_t stack = area;
    if constexpr (TREE) {
      if (i & 1u) {
#pragma unroll 1
        for (uint32_t q = i >> 1; q & 1u; q >>= 1, stack += kQuadLevel) {
          QuadMsg x;
          x.w[0] = *reinterpret_cast<lds_u32 *>(stack + lane * 4);
          x.w[1] = *reinterpret_cast<lds_u32 *>(stack + 256 + lane * 4);
          x.e = *reinterpret_cast<lds_u32 *>(stack + 512 + lane * 4);
          quad_decode<FMT, true>(x, v);
        }
      }
    }
    if (may_end && i == W.encodes) return false;
    m = quad_encode<FMT>(v, TREE ? !(k & 1u) : k == 0 && i0 == 0);
    if (may_end && i == last) {  // all-gather: what every worker decodes from the sink's message
      quad_decode<FMT, false>(m, v);
      return false;
    }
    if constexpr (TREE) {
      if (i & 1u) {
        *reinterpret_cast<lds_u32 *>(stack + lane * 4) = m.w[0];
        *reinterpret_cast<lds_u32 *>(stack + 256 + lane * 4) = m.w[1];
        *reinterpret_cast<lds_u32 *>(stack + 512 + lane * 4) = m.e;
      }
    } else if (i >= W.first_kept) {
      quad_store<FMT>(W.msg[i & 1u] + (size_t)path * W.msg_stride, W.chunk_blocks, bl, lane & 3u, m);
    }
    return true;
  };
  uint32_t i0 = 0;
#pragma unroll 1
  for (; i0 + 2 * kAhead <= leaves; i0 += kAhead) {  // eight leaves with eight or more behind them
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) p[k] = tensor(i0 + kAhead + k);
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) hop(i0, k, s[k], [&] { s[k] = quad_slice<LT>(p[k], at); }, std::false_type{});
  }
#pragma unroll 1
  for (;; i0 += kAhead) {
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k) p[k] = tensor(min(i0 + kAhead + k, last));
#pragma unroll
    for (uint32_t k = 0; k < kAhead; ++k)
      if (!hop(i0, k, s[k], [&] { s[k] = request(p[k], i0 + kAhead + k); }, std::true_type{})) goto done;
  }
done:
  if (bi < W.chunk_blocks) {
    float *o = W.out + entry;
    gst<f32x4>(o, f32x4{v[0], v[1], v[2], v[3]});
    gst<f32x4>(o + 4, f32x4{v[4], v[5], v[6], v[7]});
  }
}

// By tiles per CU (512 super-groups are one at 256 CUs); a block of the walk does the work of 16 of them.  Ratios below: this kernel's time over the
// walk's, fp32 and bf16 rings, chains and butterflies of 2 to 128 workers in the three formats (profiles/mx_replay_splits.txt).
//   Up to 16, one block of the walk per CU, whose waves have a SIMD to themselves: the tiles' chains are a quarter as long here, 0.3 to 0.9 at 8, until
// the CU's lanes are full: at 10 in fp32 (8 workers 0.95 to 0.99; 11: 1.04), 12 in bf16 (0.85 to 0.91 of 8, 0.86 to 1.04 of 32), 10 or 11 for rings and chains of 12
// to 23 (15 at 11: 1.04 to 1.06, 12 at 11 0.92 and at 12 1.07).  6-bit codes, whose conversions take 32 entries whether there are or not, end at 8; two or three
// workers, who leave most of the eight requests idle, at 8 in fp32 (0.9; 9: 1.15) and 4 in bf16.
//   Above, most inputs come from memory, and what counts is how many requests are on their way: this kernel's are eight leaves' of each wave, the walk's one or two
// workers' of each of three blocks per CU.  But everyone waits for the CUs that have a block of the walk more than others, where inputs stay in the cache.
// fp32: of 16 workers and more all (0.84 to 1.0); of 8 to 15 all but the second block's last quarter (32 tiles per CU: 1.0 to 1.13; 40: 0.84 to 0.9); 4 to 7
// from 36 on (0.9 to 1.0) and in a quarter of the second (0.78 to 0.92); fewer never (1.05 to 1.3).  6-bit from 45 (16 workers; 0.88 to 1.0) and 75 (8).
// bf16, whose walk moves half the bytes and has less to wait for: 8 to 47 workers from 50 tiles per CU (0.87 to 0.98; 40: 0.95 to 1.05; halvings of 8 from 65), more workers
// from 100 (0.93 to 0.98; 46 to 75: 0.93 to 1.09); 4 to 7 from 165 to 400 (0.87 to 0.96); an eighth of the second block of 64 workers and more
// (0.84 to 0.9; chains of 100 and more 1.05 to 1.07).  6-bit from 100 (16 workers: 0.89 to 0.97) and 150 (8: 0.87 to 0.97).
//   Inputs that are used again and again, or were just written, come from the cache up to some 250 MB, and lose by that: bf16 of 8 to 15 workers between 50 tiles per CU and that size
// 1.03 to 1.18 where from memory it is 0.87 to 1.04; fp32 of 4 to 7 workers 1.0 to 1.16 for 0.9 to 1.0; fp32 of 8 to 15 at 28 and 48 tiles per CU 1.03 and 1.09 for 0.87.  The walk from the
// cache and this kernel from memory cannot both be had, as the library does not know where its inputs are.
//   600 drawn replays from memory against the walk wherever fp32's or a large bf16 ring's shape did not ask for this: 1.00 to 1.06 of their time by format, type and workers; 1.7 % on average.
template <int FMT, typename LT, bool TREE>
bool takes_quad(uint32_t n, uint32_t n_chunks, uint64_t tiles, uint32_t n_cu) {
  constexpr bool six = FMT == DQ_MXFP6_E3M2, wide = sizeof(LT) == 4;
  if (tiles >= 1u << 25) return false;  // threads of a launch: below 2^31
  const uint64_t half_full = TREE || n < 12 || n >= 24 ? 12 : n < 14 ? 11 : 10;
  const uint64_t few = n < 4 ? (wide ? 8 : 4) : six ? 8 : wide ? 10 : half_full;
  if (tiles <= few * n_cu) return true;
  if (tiles <= 16ull * n_cu) return false;
  const uint64_t c = (tiles + 16ull * n_cu - 1) / (16ull * n_cu), slack = 16ull * c * n_cu - tiles;  // slack: tiles that the fullest CUs' last blocks lack
  const uint64_t per_cu = tiles / n_cu;
  const bool last_quarter = c == 2 && slack >= 12ull * n_cu;  // of the second block per CU only a quarter is there
  if (wide) {
    if (six) return n >= 8 && (per_cu >= (n >= 16 ? 45 : 75) || last_quarter);
    if (n >= 16) return true;
    if (n >= 8) return c != 2 || slack >= 4ull * n_cu;
    return n >= 4 && (per_cu >= 36 || last_quarter);
  }
  if (c == 2 && slack >= 14ull * n_cu && !six) return n >= 64 && (n_chunks > 1 || n < 100);
  if (six) return n >= 8 && per_cu >= (n >= 16 ? 100 : 150);
  if (n >= 8) return per_cu >= (n >= 48 ? 100 : TREE && n < 16 ? 65 : 50);
  return n >= 4 && per_cu >= 165 && per_cu < 400;
}

template <int FMT, typename LT, bool TREE>
hipError_t go_mx_quad(MxWalk W, uint32_t n_paths, hipStream_t s) {
  W.tiles_per_path = (uint32_t)((W.chunk_blocks + kQuadBlocks - 1) / kQuadBlocks);
  W.n_tiles = n_paths * W.tiles_per_path;
  W.wave_bytes = TREE && W.log_n > 1 ? (W.log_n - 1) * kQuadLevel : 0;
  const uint32_t blocks = (W.n_tiles + kBlockWaves - 1) / kBlockWaves;
  hipLaunchKernelGGL((mx_quad<FMT, LT, TREE>), dim3(blocks), dim3(kBlockThreads), W.wave_bytes * kBlockWaves, s, W);
  return hipGetLastError();
}

template <int FMT, typename LT, bool TREE>
hipError_t go_mx_walk(MxWalk W, uint32_t n_cu, hipStream_t s) {
  const uint32_t n_paths = W.n_tiles / W.tiles_per_path;
  if (takes_quad<FMT, LT, TREE>(W.n, W.n_chunks, n_paths * ((W.chunk_blocks + kQuadBlocks - 1) / kQuadBlocks), n_cu)) return go_mx_quad<FMT, LT, TREE>(W, n_paths, s);
  const uint32_t levels = TREE && W.log_n > 1 ? W.log_n - 1 : 0;
  W.wave_bytes = levels * kMxStackLevel > kMxXpose ? levels * kMxStackLevel : kMxXpose;
  const uint32_t lds = W.wave_bytes * kBlockWaves;
  uint32_t per_cu = 160u * 1024 / lds;
  // Three blocks fit a CU (168 registers); a fourth begins when one ends and has a last round to itself.  bf16: three and a longer walk each 3 to 10 % faster from 32 tiles
  // per CU on, and for 4 workers and more of the 8- and 4-bit formats from the start (0 to 5 %); 2 workers at 21 to 26 tiles 2 to 7 % slower; fp32 0 to 3 % either way.
  const uint32_t most = sizeof(LT) == 2 && (W.n_tiles >= 32 * n_cu || (FMT != DQ_MXFP6_E3M2 && W.n >= 4)) ? 3 : 4;
  if (per_cu > most) per_cu = most;
  if (per_cu < 1) per_cu = 1;
  uint32_t blocks = (W.n_tiles + kBlockWaves - 1) / kBlockWaves;
  if (blocks > n_cu * per_cu) blocks = n_cu * per_cu;
  hipLaunchKernelGGL((mx_walk<FMT, LT, TREE>), dim3(blocks), dim3(kBlockThreads), lds, s, W);
  return hipGetLastError();
}
template <int FMT>
hipError_t mx_walk_fmt(dq_dtype dtype, bool tree, const MxWalk &W, uint32_t n_cu, hipStream_t s) {
  if (dtype == DQ_F32) return tree ? go_mx_walk<FMT, float, true>(W, n_cu, s) : go_mx_walk<FMT, float, false>(W, n_cu, s);
  return tree ? go_mx_walk<FMT, uint16_t, true>(W, n_cu, s) : go_mx_walk<FMT, uint16_t, false>(W, n_cu, s);
}

template <int FMT, Kind KIND, typename LT>
hipError_t go(const MxJob *one, const MxJob *jobs, uint32_t n_jobs, uint64_t max_entries, uint32_t n_cu, hipStream_t s) {
  const uint64_t blocks_needed = (max_entries / 32 + kBlockThreads - 1) / kBlockThreads;
  if (blocks_needed == 0 || n_jobs == 0) return hipSuccess;
  uint64_t cap = ((uint64_t)n_cu * 8 + n_jobs - 1) / n_jobs;
  if (cap < 1) cap = 1;
  const uint32_t blocks = (uint32_t)(blocks_needed < cap ? blocks_needed : cap);
  if (one) hipLaunchKernelGGL((mx_one<FMT, KIND, LT>), dim3(blocks), dim3(kBlockThreads), 0, s, *one);
  else
    for (uint32_t first = 0; first < n_jobs; first += kMaxGridRows) {  // gridDim.y holds at most 65,535 rows
      const uint32_t rows = n_jobs - first < kMaxGridRows ? n_jobs - first : kMaxGridRows;
      hipLaunchKernelGGL((mx_batch<FMT, KIND, LT>), dim3(blocks, rows), dim3(kBlockThreads), 0, s, jobs + first);
    }
  return hipGetLastError();
}

template <int FMT>
hipError_t dispatch(Kind kind, dq_dtype dtype, bool has_local, const MxJob *one, const MxJob *jobs, uint32_t n_jobs,
                    uint64_t max_entries, uint32_t n_cu, hipStream_t s) {
  const bool f32 = dtype == DQ_F32;
  switch (kind) {
    case kCompress:
      return f32 ? go<FMT, kCompress, float>(one, jobs, n_jobs, max_entries, n_cu, s)
                 : go<FMT, kCompress, uint16_t>(one, jobs, n_jobs, max_entries, n_cu, s);
    case kDar:
      return f32 ? go<FMT, kDar, float>(one, jobs, n_jobs, max_entries, n_cu, s)
                 : go<FMT, kDar, uint16_t>(one, jobs, n_jobs, max_entries, n_cu, s);
    default:
      if (!has_local) return go<FMT, kDecompress, NoLocal>(one, jobs, n_jobs, max_entries, n_cu, s);
      return f32 ? go<FMT, kDecompress, float>(one, jobs, n_jobs, max_entries, n_cu, s)
                 : go<FMT, kDecompress, uint16_t>(one, jobs, n_jobs, max_entries, n_cu, s);
  }
}

hipError_t dispatch_fmt(Kind kind, dq_codec fmt, dq_dtype dtype, bool has_local, const MxJob *one, const MxJob *jobs,
                        uint32_t n_jobs, uint64_t max_entries, uint32_t n_cu, hipStream_t s) {
  switch (fmt) {
    case DQ_MXFP8_E4M3: return dispatch<DQ_MXFP8_E4M3>(kind, dtype, has_local, one, jobs, n_jobs, max_entries, n_cu, s);
    case DQ_MXFP6_E3M2: return dispatch<DQ_MXFP6_E3M2>(kind, dtype, has_local, one, jobs, n_jobs, max_entries, n_cu, s);
    case DQ_MXFP4_E2M1: return dispatch<DQ_MXFP4_E2M1>(kind, dtype, has_local, one, jobs, n_jobs, max_entries, n_cu, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_mx_walk(dq_codec fmt, dq_dtype dtype, bool tree, const MxWalk &W, uint32_t n_cu, hipStream_t s) {
  switch (fmt) {
    case DQ_MXFP8_E4M3: return mx_walk_fmt<DQ_MXFP8_E4M3>(dtype, tree, W, n_cu, s);
    case DQ_MXFP6_E3M2: return mx_walk_fmt<DQ_MXFP6_E3M2>(dtype, tree, W, n_cu, s);
    case DQ_MXFP4_E2M1: return mx_walk_fmt<DQ_MXFP4_E2M1>(dtype, tree, W, n_cu, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t mx_launch_one(Kind kind, dq_codec fmt, dq_dtype dtype, bool has_local, const MxJob &job, uint32_t n_cu,
                         hipStream_t s) {
  return dispatch_fmt(kind, fmt, dtype, has_local, &job, nullptr, 1, job.n_entries, n_cu, s);
}
hipError_t mx_launch_batch(Kind kind, dq_codec fmt, dq_dtype dtype, bool has_local, const MxJob *jobs, uint32_t n_jobs,
                           uint64_t max_entries, uint32_t n_cu, hipStream_t s) {
  return dispatch_fmt(kind, fmt, dtype, has_local, nullptr, jobs, n_jobs, max_entries, n_cu, s);
}

}  // namespace dq

// ---- C ABI ----------------------------------------------------------------------------
namespace {
bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool is_mx_fmt(dq_codec f) { return f == DQ_MXFP8_E4M3 || f == DQ_MXFP6_E3M2 || f == DQ_MXFP4_E2M1; }
int code_bits(dq_codec f) { return f == DQ_MXFP8_E4M3 ? 8 : f == DQ_MXFP6_E3M2 ? 6 : 4; }
uint32_t device_cus() {
  static thread_local int cached = 0;
  if (!cached) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
      cached = prop.multiProcessorCount;
    else
      cached = 256;
  }
  return (uint32_t)cached;
}
}  // namespace

extern "C" {

size_t dq_mx_packed_bytes(dq_codec fmt, uint64_t n_entries) {
  if (!is_mx_fmt(fmt) || n_entries % 256) return 0;
  const uint64_t blocks = n_entries / 32;
  const uint64_t sz = blocks * (uint64_t)(code_bits(fmt) * 4) + blocks;
  return (size_t)((sz + 15) & ~(uint64_t)15);
}

dq_status dq_mx_compress(dq_codec fmt, const void *local, dq_dtype dtype, uint64_t n_entries, void *packed_out,
                         void *hip_stream) {
  if (!is_mx_fmt(fmt) || !local || !packed_out || n_entries % 256 || (dtype != DQ_F32 && dtype != DQ_BF16))
    return DQ_EINVAL;
  if (!al16(local) || !al16(packed_out)) return DQ_EALIGN;
  dq::MxJob j{nullptr, local, packed_out, n_entries};
  return dq::hip_status(dq::mx_launch_one(dq::kCompress, fmt, dtype, true, j, device_cus(), (hipStream_t)hip_stream));
}

dq_status dq_mx_dar_hop(dq_codec fmt, const void *packed_in, const void *local, dq_dtype dtype, uint64_t n_entries,
                        void *packed_out, void *hip_stream) {
  if (!is_mx_fmt(fmt) || !packed_in || !local || !packed_out || n_entries % 256 ||
      (dtype != DQ_F32 && dtype != DQ_BF16))
    return DQ_EINVAL;
  if (!al16(packed_in) || !al16(local) || !al16(packed_out)) return DQ_EALIGN;
  dq::MxJob j{(const uint8_t *)packed_in, local, packed_out, n_entries};
  return dq::hip_status(dq::mx_launch_one(dq::kDar, fmt, dtype, true, j, device_cus(), (hipStream_t)hip_stream));
}

dq_status dq_mx_decompress(dq_codec fmt, const void *packed_in, const void *local_or_null, dq_dtype dtype,
                           uint64_t n_entries, float *out, void *hip_stream) {
  if (!is_mx_fmt(fmt) || !packed_in || !out || n_entries % 256) return DQ_EINVAL;
  if (local_or_null && dtype != DQ_F32 && dtype != DQ_BF16) return DQ_EINVAL;
  if (!al16(packed_in) || !al16(out) || !al16(local_or_null)) return DQ_EALIGN;
  dq::MxJob j{(const uint8_t *)packed_in, local_or_null, out, n_entries};
  return dq::hip_status(dq::mx_launch_one(dq::kDecompress, fmt, dtype, local_or_null != nullptr, j, device_cus(),
                           (hipStream_t)hip_stream));
}

}  // extern "C"
