// A whole replay in one launch: every tile of a chunk is carried through ALL hops of its schedule (first
// compress, every DAR hop, the last decompress-accumulate, optionally the all-gather's compress and
// decompress) by one wave, with the partial sum in registers.
//
// Why: a super-group's hop depends on nothing but the same super-group's hop before it, so the steps of a
// schedule need no synchronisation between waves.  Launched step by step, a replay reads and writes every
// packed partial sum once per hop, reads the fp32 keep-buffers of a recursive halving twice and pays the fixed part
// of a launch (5 us: descriptor, tables, the first tile's trip to memory, the tail) per step.  Here a tile's
// memory traffic is its n local slices and one result.
//   ring / chain : leaf i is worker chunk + i (mod n) / worker i; one message is pending at a time and stays
//                  in registers as signed levels and scale.  The packed messages of the last two steps are
//                  also written, where dq_replay_message finds them.
//   butterfly    : recursive halving of one chunk is a binary tree over the workers; the leaves are visited
//                  depth first, the sending child of a node before the keeping one, so that at most one
//                  message per level is pending.  A message that the next leaf takes stays in registers, the
//                  others wait as packed codes in LDS (20 bytes per lane and level).
// Per hop and tile the random numbers are the same Philox counters as in the step kernels; the per-super-group
// draws of up to 16 hops are made by one wave-wide call (lane = tile of the batch, hop, row).
#include <string.h>

#include "dq_bounds.h"
#include "dq_walk.h"

namespace dq {
namespace {

// Waves per SIMD, as many as the kernel's vector registers allow: 94 for a ring or chain of bf16 tensors, 101 to 127 for the
// others.  (Five are 3 % faster than four where a wave has a few tiles, 25 MB through a ring of eight.)
template <typename LT, bool TREE>
constexpr int kWalkPerSimd = sizeof(LT) == 2 && !TREE ? 5 : 4;
constexpr uint32_t kParkBytes = 1280;   // per wave: 64 scale draws of 16 bytes, 64 permutation slots
constexpr uint32_t kXposeBytes = 2048;  // per wave: half a tile of fp32 results
static_assert(4 * kParkBytes <= (kOffTab4 - kOffDec2) * 4, "a ring's draws lie over the decode tables");

// Per-super-group draws for 2^hops_log hops, starting at hop i, of 16 >> hops_log tiles, starting at `pos`.
template <bool TREE>
__device__ __forceinline__ void park_hops(const Job &job, const Params &P, const Walk &W, uint32_t chunk, const TilePos pos,
                                          uint32_t i, uint32_t area) {
  const uint32_t lane = lane_here();
  const uint32_t idx = lane >> 2, h = idx & ((1u << W.hops_log) - 1u), sub = idx >> W.hops_log;
  const uint32_t sgw = min(pos.tile_first + sub * kWaveSGs + (lane & 3u), pos.n_seg - 1);
  const uint64_t G = job.first_sg + pos.seg_first + sgw;
  const uint32_t rank = leaf_of<TREE>(W, chunk, min(i + h, W.n - 1));  // hops past the last are drawn for nothing
  const U4 shared = philox4x32_10((uint32_t)G, (uint32_t)(G >> 32), P.round, (2u << 16) | 0xFFFFu, P.key0, P.key1);
  const U4 scale = philox4x32_10((uint32_t)G, (uint32_t)(G >> 32), P.round, (1u << 16) | (rank & 0xFFFFu), P.key0, P.key1);
  lds_st4(area + lane * 16, u32x4{scale.x, scale.y, scale.z, scale.w});
  lds_st1(area + 1024 + lane * 4, perm_slot(shared, P, rank));
}

template <typename LT>
struct Slice {
  uint4 w[sizeof(LT) == 4 ? 4 : 2];  // a lane's 16 entries, raw
};
template <typename LT>
__device__ __forceinline__ Slice<LT> load_slice(const Walk &W, uint32_t leaf, uint64_t at) {
  const uint8_t *p = reinterpret_cast<const uint8_t *>(table_entry(reinterpret_cast<const uint64_t *>(W.grads), leaf)) + at;
  Slice<LT> s;
#pragma unroll
  for (int i = 0; i < (sizeof(LT) == 4 ? 4 : 2); ++i) s.w[i] = gld16(p + 16 * i);
  return s;
}
// Byte offset of this lane's 16 entries of the tile at `pos` inside every worker's tensor, and the mean to take off.
template <typename LT, bool MU>
__device__ __forceinline__ uint64_t slice_at(const Job &job, const TilePos pos, float *mu) {
  const uint32_t lane = lane_here();
  const uint32_t sg0 = pos.seg_first + min(pos.tile_first + (lane >> 4), pos.n_seg - 1);
  const uint64_t sg = job.src ? (uint64_t)gld<uint32_t>(job.src + sg0) : (uint64_t)sg0;
  if constexpr (MU) *mu = gld<float>(job.mu + sg0);
  return (uint64_t)reinterpret_cast<uintptr_t>(job.local) + sg * (kSG * sizeof(LT)) + (lane & 15u) * (16 * sizeof(LT));
}

// A tile's results, v[16] per lane, to out[...] like store_tile_f32, two super-groups at a time.
__device__ __forceinline__ void store_result(const Job &job, const Params &P, float (&v)[16], uint32_t xpose, const TilePos pos) {
  const uint32_t lane = lane_here(), l = lane & 31u;
  const uint32_t last_row = min((uint32_t)kWaveSGs - 1, pos.n_seg - 1 - pos.tile_first);
  const size_t sg0 = (size_t)pos.seg_first + pos.tile_first;
  if (job.back) {
    const float back = (float)P.n_workers * gld<float>(job.back + sg0 + min(lane >> 4, last_row));
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = v[k] + back;
  }
  float *out = static_cast<float *>(job.out);
#pragma unroll
  for (uint32_t half = 0; half < 2; ++half) {
    __builtin_amdgcn_wave_barrier();
    if ((lane >> 5) == half) {
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i)
        lds_stf4(xpose + l * 64 + ((i ^ ((l >> 2) & 3u)) * 16), f32x4{v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]});
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q) {
      const uint32_t r = 2 * half + q;
      if (r > last_row) break;
      const uint32_t slot = q * 64 + lane, w = slot >> 2, c = slot & 3u;
      const f32x4 o = lds_ldf4(xpose + w * 64 + ((c ^ ((w >> 2) & 3u)) * 16));
      const size_t sg = job.dest ? (size_t)gld<uint32_t>(job.dest + sg0 + r) : sg0 + r;
      gst_once<f32x4>(reinterpret_cast<float4 *>(out + sg * kSG) + lane, o);
    }
  }
  __builtin_amdgcn_wave_barrier();
}

// Where the LDS areas of a wave sit.
struct Areas {
  uint32_t park, xpose, stack;
};

enum { kNone = 0, kLevels = 1, kCodes = 2, kBoth = 3 };
template <int N>
struct How { static constexpr int value = N; };

// `len` consecutive tiles of width B from `pos` on.
template <int B, typename LT, bool MU, bool TREE>
__device__ __forceinline__ void walk_tiles(const WalkPath &path, const Params &P, const Vec &V, const Walk &W, const Areas A,
                                           TilePos pos, uint32_t len) {
  const Job &job = path.job;
  const uint32_t lane = threadIdx.x & 63u, g = lane & 15u;
  const uint32_t hops = 1u << W.hops_log, tiles = 16u >> W.hops_log;
  float mu = 0.0f, mu_next = 0.0f;
  uint64_t at = slice_at<LT, MU>(job, pos, &mu);
  Slice<LT> s = load_slice<LT>(W, leaf_of<TREE>(W, path.chunk, 0u), at);
  for (uint32_t t = 0; t < len; ++t) {
    TilePos pos_next = pos;
    pos_next.tile_first += kWaveSGs;
    uint64_t at_next = at;
    const bool more = t + 1 < len;
    if (more) at_next = slice_at<LT, MU>(job, pos_next, &mu_next);
    const uint32_t rowc = min(lane >> 4, pos.n_seg - 1 - pos.tile_first);
    const uint64_t gi = (job.first_sg + pos.seg_first + pos.tile_first + rowc) * 16 + g;  // global group index
    float v[16];       // this leaf's entries, then the partial sum, then the message's signed levels
    float level[16];   // the pending message: signed levels ...
    float sfg = 0.0f;  // ... times this
    // One leaf: its entries, plus the pending message (has), plus (tree) `taken` messages of the stack; then the
    // encoding (kNone: it is the last).  The loops below are written so that every encoding variant has a body of its
    // own: behind a branch the compiler computes what the variants share for all 16 entries first and runs
    // out of registers.
    auto leaf = [&](uint32_t i, bool has, uint32_t taken, auto how, auto is_last) {
      constexpr int kHow = decltype(how)::value;
      const uint32_t rank = leaf_of<TREE>(W, path.chunk, i);
      Draws d;
      if constexpr (kHow != kNone) {
        if ((i & (hops - 1u)) == 0 && (t & (tiles - 1u)) == 0) {
          __builtin_amdgcn_wave_barrier();
          park_hops<TREE>(job, P, W, path.chunk, pos, i, A.park);
          __builtin_amdgcn_wave_barrier();
        }
        const uint32_t slot = ((((t & (tiles - 1u)) << W.hops_log) + (i & (hops - 1u))) * 4 + rowc);
        uint64_t index = gi;
        asm volatile("" : "+v"(index));  // the generator's first round is not worth four registers around the loop
        d = draw_group(P, index, rank, lds_ld1(A.park + 1024 + slot * 4), lds_ld1(A.park + slot * 16 + (g >> 2) * 4), g);
        asm volatile("" : "+v"(s.w[0].x) : "v"(d.gam.x), "v"(d.gam.y), "v"(d.gam.z), "v"(d.gam.w), "v"(d.o_pi), "v"(d.us));
      }
      widen_local<LT>(s.w, v);
      if constexpr (MU) {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = v[k] - mu;
      }
      // the next leaf's entries, or the next tile's first.  Where there is none s is nothing, not what it was: to keep that the
      // compiler would load into other registers, and wait for the data at every leaf's end to move it here.
      Slice<LT> next;
      if constexpr (!decltype(is_last)::value) next = load_slice<LT>(W, leaf_of<TREE>(W, path.chunk, i + 1), at);
      else if (more) next = load_slice<LT>(W, leaf_of<TREE>(W, path.chunk, 0u), at_next);
      s = next;
      if (has) {
#pragma unroll
        for (int k = 0; k < 16; ++k) v[k] = __builtin_fmaf(level[k], sfg, v[k]);
      }
      uint32_t stack = A.stack;
      if constexpr (TREE) {
#pragma unroll 1
        for (uint32_t q = 0; q < taken; ++q, stack += kStackCoded) {
          const u32x4 m = lds_ld4(stack + lane * 16);
          const uint32_t ms[4] = {m.x, m.y, m.z, m.w};
          uint32_t cw[Width<B>::words];
#pragma unroll
          for (int k = 0; k < Width<B>::words; ++k) cw[k] = ms[k];
          const float f = u2f(lds_ld1(stack + 1024 + lane * 4));
          each_level<B, HopTables>(cw, [&](int k, float l) { v[k] = __builtin_fmaf(l, f, v[k]); });
        }
      }
      if constexpr (kHow != kNone) {
        const Scales sc = scale_group(v, d.us, kRec0);
        sfg = sc.sfg;
        uint32_t ow[Width<B>::words];
        quantize<B, (kHow & kCodes) != 0, (kHow & kLevels) != 0>(v, sc.inv, d.gam, d.o_pi, V, ow);
        if constexpr (kHow == kCodes) {  // tree: onto the stack
          u32x4 m = {0, 0, 0, 0};
          m.x = ow[0];
          if constexpr (B >= 4) m.y = ow[1];
          if constexpr (B == 8) { m.z = ow[2]; m.w = ow[3]; }
          lds_st4(stack + lane * 16, m);
          lds_st1(stack + 1024 + lane * 4, f2u(sc.sfg));
        } else {
          if constexpr (kHow == kBoth) store_codes<B>(message_of(path, i), TileBase<B>(job, pos), rowc * 16 + g, rowc, ow, sc.rg, sc.sfb);
#pragma unroll
          for (int k = 0; k < 16; ++k) level[k] = v[k];
        }
      }
    };
    const uint32_t last = W.n - 1;
    const bool gathered = W.encodes == W.n;
    uint32_t taken = 0;
    if constexpr (TREE) {
#pragma unroll 1
      for (uint32_t i = 0;; i += 2) {
        leaf(i, false, 0, How<kLevels>(), Is<false>());
        taken = __builtin_ctz(~(i >> 1));  // trailing ones above the lowest bit: the messages this node takes
        if (i + 1 == last) break;
        leaf(i + 1, true, taken, How<kCodes>(), Is<false>());
      }
    } else {
      uint32_t i = 0;
#pragma unroll 1
      for (; i < W.first_kept; ++i) leaf(i, i > 0, 0, How<kLevels>(), Is<false>());
#pragma unroll 1
      for (; i < last; ++i) leaf(i, i > 0, 0, How<kBoth>(), Is<false>());
    }
    if (gathered) {  // what every worker decodes from the sink's message
      leaf(last, true, taken, How<kLevels>(), Is<true>());
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = level[k] * sfg;
    } else {
      leaf(last, true, taken, How<kNone>(), Is<true>());
    }
    store_result(job, P, v, A.xpose, pos);
    pos = pos_next;
    at = at_next;
    mu = mu_next;
  }
}

// The same for raw 16-bit super-groups: the message is the partial sum rounded to bf16.
template <typename LT, bool TREE>
__device__ __forceinline__ void walk_tile16(const WalkPath &path, const Params &P, const Walk &W, const Areas A, const TilePos pos) {
  const Job &job = path.job;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t rowc = min(lane >> 4, pos.n_seg - 1 - pos.tile_first), lg = rowc * 16 + (lane & 15u);
  float mu = 0.0f;
  const uint64_t at = job.mu ? slice_at<LT, true>(job, pos, &mu) : slice_at<LT, false>(job, pos, &mu);
  Slice<LT> s = load_slice<LT>(W, leaf_of<TREE>(W, path.chunk, 0u), at);
  float v[16];
  uint32_t m[8];  // the pending message
#pragma unroll
  for (int k = 0; k < 8; ++k) m[k] = 0;
  auto take = [&](const uint32_t (&w)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[2 * j] = u2f(w[j] << 16) + v[2 * j];
      v[2 * j + 1] = u2f(w[j] & 0xFFFF0000u) + v[2 * j + 1];
    }
  };
#pragma unroll 1
  for (uint32_t i = 0; i < W.n; ++i) {
    widen_local<LT>(s.w, v);
    if (job.mu) {
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = v[k] - mu;
    }
    if (i + 1 < W.n) s = load_slice<LT>(W, leaf_of<TREE>(W, path.chunk, i + 1), at);
    if (TREE ? (i & 1u) : i > 0) take(m);
    uint32_t up = i >> 1, stack = A.stack;
    if constexpr (TREE) {
      if (i & 1u) {
#pragma unroll 1
        for (; up & 1u; up >>= 1, stack += kStackRaw) {
          const u32x4 a = lds_ld4(stack + lane * 16), b = lds_ld4(stack + 1024 + lane * 16);
          const uint32_t w[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
          take(w);
        }
      }
    }
    if (i < W.encodes) {
#pragma unroll
      for (int k = 0; k < 8; ++k) m[k] = bf16_rne_pair(v[2 * k], v[2 * k + 1]);
      if constexpr (TREE) {
        if ((i & 1u) && i + 1 < W.n) {
          lds_st4(stack + lane * 16, u32x4{m[0], m[1], m[2], m[3]});
          lds_st4(stack + 1024 + lane * 16, u32x4{m[4], m[5], m[6], m[7]});
        }
      } else if (i >= W.first_kept && i + 1 < W.n) {
        uint8_t *dst = message_of(path, i) + TileBase<16>(job, pos).code_off + lg * 32;
        gst<u32x4>(dst, u32x4{m[0], m[1], m[2], m[3]});
        gst<u32x4>(dst + 16, u32x4{m[4], m[5], m[6], m[7]});
      }
    }
  }
  if (W.encodes == W.n) {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = 0.0f;
    take(m);
  }
  store_result(job, P, v, A.xpose, pos);
}

template <typename LT, bool MU, bool TREE>
__device__ __forceinline__ void walk_range(const WalkPath &path, const Params &P, const Vec &V, const Walk &W, const Areas A,
                                           uint32_t lo, uint32_t hi) {
  while (lo < hi) {
    const TilePos p = locate(path.job, lo);
    const uint32_t left = (p.n_seg - p.tile_first + kWaveSGs - 1) / kWaveSGs;
    const uint32_t len = min(hi - lo, left);
    if (p.wi == 0) walk_tiles<2, LT, MU, TREE>(path, P, V, W, A, p, len);
    else if (p.wi == 1) walk_tiles<4, LT, MU, TREE>(path, P, V, W, A, p, len);
    else if (p.wi == 2) walk_tiles<8, LT, MU, TREE>(path, P, V, W, A, p, len);
    else {
      TilePos q = p;
      for (uint32_t i = 0; i < len; ++i, q.tile_first += kWaveSGs) walk_tile16<LT, TREE>(path, P, W, A, q);
    }
    lo += len;
  }
}

// Wave w takes the tiles from S.shares[w] up to S.shares[w + 1] of the paths laid end to end (split_walk).
template <typename LT, bool MU, bool TREE>
__global__ __launch_bounds__((TREE ? 512 : 256)) __attribute__((amdgpu_waves_per_eu((kWalkPerSimd<LT, TREE>)))) void k_walk(
    const WalkPath *paths, const WalkShare *shares, Walk W, Params P) {
  extern __shared__ uint4 lds_raw[];
  uint32_t *lds = reinterpret_cast<uint32_t *>(lds_raw);
  const uint32_t waves = blockDim.x / 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t v = __builtin_amdgcn_readfirstlane(share_of<TREE>(W, wave, waves));
  const WalkShare from = table_entry(shares, v), to = table_entry(shares, v + 1);
  copy_tables(lds, P.blob, P, TREE ? kOffDec2 : kOffTab4);  // a ring or chain never decodes from codes
  __syncthreads();
  Areas A;
  const uint32_t end = P.blob_dwords * 4;
  A.park = (TREE ? end : kOffDec2 * 4) + wave * kParkBytes;  // ring, chain: over the decode tables, which they do not copy
  A.stack = end + (TREE ? waves * kParkBytes : 0u) + wave * (TREE ? W.stack_bytes : kXposeBytes);
  A.xpose = A.stack;  // the stack is empty when a tile's result is stored
  const Vec V(P);
  for (uint32_t p = from.path, lo = from.tile; p < to.path || (p == to.path && lo < to.tile); ++p, lo = 0) {
    const WalkPath path = table_entry(paths, p);
    uint32_t hi = to.tile;
    if (p < to.path) {
      hi = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) hi += (path.job.n_sg[w] + kWaveSGs - 1) / kWaveSGs;
    }
    walk_range<LT, MU, TREE>(path, P, V, W, A, lo, hi);
  }
}

uint32_t walk_lds(const Params &P, bool tree, uint32_t stack_bytes, uint32_t waves) {
  return P.blob_dwords * 4 + waves * (tree ? kParkBytes + stack_bytes : kXposeBytes);
}

template <typename LT, bool MU, bool TREE>
hipError_t go_walk(const WalkPath *paths, const WalkShare *shares, const Walk &W, const Params &P, hipStream_t s) {
  hipLaunchKernelGGL((k_walk<LT, MU, TREE>), dim3(W.blocks), dim3(W.waves * 64), walk_lds(P, TREE, W.stack_bytes, W.waves), s, paths,
                     shares, W, P);
  return hipGetLastError();
}

template <typename LT>
hipError_t static_lds_of(size_t *bytes) {
  hipError_t e = add_static_lds(k_walk<LT, false, false>, bytes);
  if (e == hipSuccess) e = add_static_lds(k_walk<LT, false, true>, bytes);
  if (e == hipSuccess) e = add_static_lds(k_walk<LT, true, false>, bytes);
  return e != hipSuccess ? e : add_static_lds(k_walk<LT, true, true>, bytes);
}

}  // namespace

hipError_t walk_static_lds(size_t *bytes) {
  const hipError_t e = static_lds_of<float>(bytes);
  return e != hipSuccess ? e : static_lds_of<uint16_t>(bytes);
}

// The launch of W's schedule with tiles of W->tile_sgs super-groups.  *resident: waves that a CU holds at once.  False: no block fits.
static bool grid_of_tiles(const Params &P, bool f32, bool tree, uint32_t n_cu, uint64_t tiles, WalkGrid *W, uint32_t *resident) {
  constexpr uint32_t kLds = 160u * 1024, kGranule = 1280;  // LDS is given out in 128 pieces
  uint32_t lds, most;  // most: waves that fit a CU's registers
  if (W->tile_sgs < kWaveSGs) {
    W->stack_bytes = thin_stack(W->tile_sgs, W->levels);
    W->waves = 4;
    lds = thin_lds(P, W->stack_bytes);
    most = f32 && W->tile_sgs == 2 ? 12 : 16;
  } else {
    // the stack area also stages half a tile's result
    W->stack_bytes = W->levels * (W->raw ? kStackRaw : kStackCoded);
    if (W->stack_bytes < kXposeBytes) W->stack_bytes = kXposeBytes;
    // A butterfly's two blocks per CU share a copy of the tables each; where there are fewer tiles than two waves for every
    // SIMD, blocks of four reach all CUs.  Rings and chains always take blocks of four, 29 KB at the levels of 25 MB and n = 8: five per CU.
    // (Blocks of ten waves put three waves on two of the SIMDs, and the CU has no room for the second one: 97 us, not 75.)
    W->waves = tree && tiles >= (uint64_t)n_cu * 8 ? 8 : 4;
    if (walk_lds(P, tree, W->stack_bytes, W->waves) > kLds) W->waves = 4;  // raw chunks of 1,024 workers and more
    lds = walk_lds(P, tree, W->stack_bytes, W->waves);
    most = 4 * (tree ? kWalkPerSimd<float, true> : (f32 ? kWalkPerSimd<float, false> : kWalkPerSimd<uint16_t, false>));
  }
  if (lds > kLds) return false;
  uint32_t per_cu = kLds / ((lds + kGranule - 1) / kGranule * kGranule);
  const uint32_t held = per_cu < most / W->waves ? per_cu : most / W->waves;
  *resident = held * W->waves;
  if (W->tile_sgs == kWaveSGs) per_cu = held;
  const uint64_t needed = (tiles + W->waves - 1) / W->waves, blocks = (uint64_t)n_cu * per_cu;
  W->blocks = (uint32_t)(needed < blocks ? needed : blocks);
  W->most_blocks = (uint32_t)blocks;
  W->full = W->blocks * W->waves > 8 * n_cu;
  return true;
}

// Tiles of 1, 2 (dq_thin.hip) or 4 super-groups: the narrower, the shorter a hop's chain and the more hops' worth of
// instructions there are in all, so narrow ones pay where wide ones would leave SIMDs idle or with a wave or two each.
// us per replay, tiles of 1 / 2 / 4 super-groups, 256 CUs, by super-groups per CU (profiles/replay_tile_sizes.txt has all that was measured):
//                 12              16              20              24              28              32
//   ring bf16 4   6.7/8.5/7.8     7.8/9.6/7.9     10.1/10.8/8.2   11.4/11.4/8.7   13.1/12.8/9.2   14.7/14.0/9.5
//   ring bf16 16  13.6/15.9/20.7  15.6/17.6/20.9  19.6/18.7/20.9  21.4/21.9/22.2  26.4/23.2/23.2  29.8/27.2/23.5
//   ring bf16 128 75.5/95.3/142   92.7/102/145    120/110/149     134/136/158     170/147/169     186/171/166
//   ring f32  4   7.9/8.9/7.9     9.3/9.7/8.1     11.2/11.0/8.5   12.2/12.8/9.1   14.0/14.5/9.6   15.6/15.8/10.0
//   ring f32  32  23.4/27.7/37.9  29.2/32.2/38.7  38.2/39.5/38.8  42.8/50.2/41.5  53.2/59.6/46.0  62.1/62.8/50.5
//   tree bf16 8   9.1/11.1/13.4   10.3/11.8/13.7  13.0/12.5/13.8  15.4/14.6/14.5  16.1/16.8/15.1  17.1/19.9/16.4
//   tree f32  16  14.1/15.5/23.6  16.8/17.1/23.8  22.2/18.0/23.8  27.6/23.4/24.8  28.9/29.9/26.3  32.6/36.2/38.5
//   tree bf16 64  42.9/52.3/88.6  69.0/65.5/88.0  75.7/95.1/86.7  84.1/104/90.2   94.9/105/93.3   112/108/105
// Rings and short trees: one super-group while four waves per SIMD hold them all (a little longer where a wave's start counts more than its hops,
// less with two workers, whose waves have no more than a start: 12 per CU, but 20 and 16 with an all-gather behind it, halving over 2 at 16 on the original tensors
// 6.2/7.1/7.0 with and 5.7/6.6/6.0 without); two, for fp32 rings of 11 to 16 (16 at 17 19.5/19.4/21.5) and fp32 halvings over 2 and 4 with an all-gather (2 at 18 8.2/7.2/7.8) up to 21, for bf16 rings of nine workers and more and short trees, up to 24 or 32
// per CU; then four.  What the CUs hold of a wider butterfly falls with the levels of its stack, differently for each
// tile size, so there the time is estimated, up to 48 super-groups per CU: beyond, the three are within 20 % of each other with no order.
// Of the 252 rows (two mixtures of widths each) the rule's choice is on average 0.6 % behind the best.  LDS is counted in the pieces it is given out in, and tiles of
// one and two without those that the widths' ends add, which the last waves take beside cheap ones: without that 128 workers' tree
// of 4,096 took 219 us with tiles of one for 109 with two.
static uint64_t tree_time(uint32_t n, uint32_t n_cu, uint32_t sgs, uint64_t tiles, uint32_t resident) {
  // in 0.01 us, fitted to the measurement: the launch, a tile's start, a hop alone and by the waves of the same SIMD
  struct Cost { uint32_t launch, start, hop, wave; };
  const Cost c = sgs == 1 ? Cost{640, 200, 31, 12} : sgs == 2 ? Cost{600, 240, 34, 25} : Cost{670, 0, 122, 18};
  const uint64_t at_once = (uint64_t)n_cu * resident, full = tiles / at_once, rest = tiles % at_once;
  const uint64_t rounds = full + (rest != 0), waves = full * resident / 4 + (rest + 4 * n_cu - 1) / (4 * n_cu);
  return c.launch + rounds * c.start + n * (rounds * c.hop + waves * c.wave);
}
// Super-groups of a tile, or 0: by tree_time.
static uint32_t tile_for(uint32_t n, bool f32, bool tree, bool all_gather, uint32_t n_cu, uint64_t super_groups) {
  const uint32_t per_cu = (uint32_t)((super_groups + n_cu - 1) / n_cu);
  if (tree && n >= 32) return per_cu <= 48 ? 0 : kWaveSGs;
  uint32_t one = 16, two = 16;  // up to so many per CU
  if (f32) {
    if (tree) {
      two = n > 4 ? 24 : all_gather ? 21 : 16;
    } else {
      one = n <= 4 ? 12 : n <= 16 ? 16 : 20;
      two = n <= 10 ? one : n <= 16 ? 21 : 20;
    }
  } else if (n <= 8) {
    one = two = n <= 2 ? (!all_gather ? 12 : tree ? 20 : 16) : tree ? (n <= 4 ? 22 : 24) : n <= 4 ? 16 : 20;
  } else {
    two = !tree && n >= 32 ? 32 : 24;
  }
  return per_cu <= one ? 1 : per_cu <= two ? 2 : kWaveSGs;
}

bool grid_walk(const Params &P, dq_dtype dtype, bool tree, uint32_t n_cu, const uint64_t tiles_of[3], WalkGrid *W) {
  const bool f32 = dtype == DQ_F32;
  const uint64_t super_groups = tiles_of[0];
  if (super_groups == 0) return false;
  const uint32_t wanted = tile_for(W->n, f32, tree, W->encodes == W->n, n_cu, super_groups);
  WalkGrid best = *W;
  uint64_t best_time = 0;
  bool found = false;
  for (uint32_t sgs = kWaveSGs; sgs >= (wanted ? wanted : 1); sgs /= 2) {  // the wanted one, or the next wider that fits
    WalkGrid w = *W;
    w.tile_sgs = sgs;
    uint32_t resident = 0;
    const uint64_t tiles = tiles_of[sgs / 2];
    if (!grid_of_tiles(P, f32, tree, n_cu, tiles, &w, &resident)) continue;
    const uint64_t time = wanted ? 0 : tree_time(W->n, n_cu, sgs, sgs == kWaveSGs ? tiles : (super_groups + sgs - 1) / sgs, resident);
    if (!found || time <= best_time) {
      best = w;
      best_time = time;
      found = true;
    }
  }
  if (!found) return false;
  *W = best;
  const uint64_t tiles = tiles_of[W->tile_sgs / 2], waves = (uint64_t)W->blocks * W->waves;
  // Halvings over few workers: what counts is each CU's tiles, as memory's time is most of it.  With bounded shares in path order the waves of a CU hold
  // two or three of one width while another's hold one (over 4 in bf16, 7,433/0/15,439: 23.6 us, 19.3 so, 20.9 with equal counts; 300 schedules over 2 and 4 6.4 instead
  // of 5.2 % faster than with equal shares); but where no wave has more than one tile, or over 2 workers two, path order is the better one (1 to 3 % on average, some 16 %).
  const bool several = tiles > (W->n == 2 ? 2 : 1) * waves;
  const bool spread = tree && (W->n > 4 || several) && W->tile_sgs == kWaveSGs && tiles < 8 * waves;
  // (Not with 16-bit tiles, the cheapest, at the end: ring of 6, three buckets of 4,476, a quarter of them 16-bit, 15.0 us and 15.8 reversed.)
  W->order = spread ? n_cu : tiles <= waves && !W->raw ? kReversed : 0;
  return true;
}

// Where every wave's share of the tiles begins.  All waves of tiles of four are resident at once (of narrower ones mostly, too) and a SIMD's waves share its issue, so what counts is how much the
// fullest waves hold: one with three tiles where the others have two works on alone for a third of the launch, and shares of equal cost (or equal
// count) leave that to chance.  Here every width gets a most, the tiles of it that a wave may hold, such that the fullest wave costs as little as
// possible and then each most, the dearest first, is as small as the waves allow; and the costs are raised just so far that equal shares keep to it.
// us, equal cost (below two tiles per wave: equal count) -> this, passes in turn over three sets of tensors; super-groups by width:
//   ring of 8, 51,200 in bf16: 17,608/33,584/8  60.5 -> 59.6;  a quarter, a quarter, a half  69.1 -> 61.4;  of 11, 25,322  57.5 -> 49.5
//   recursive halving in bf16 over 8, 18,504  36.8 -> 23.8;  over 32, 20,128  119 -> 91;  over 16, 8 x 51,200 at 3 bits  833 -> 831
//   in fp32: ring of 6, 8 x 44,976  687 -> 573;  halving over 2, 8 x 40,450  269 -> 214
// The geometric mean of 240 schedules of 2 to 100 workers and 1,000 to 40,700 super-groups: rings in bf16 and fp32 4.8 and 1.5 % faster, halvings
// 8.2 and 4.1 (of 14,000 and more 7.4, 1.2, 9.6 and 8.3); ten of the 240 lose more than 3 %, three more than 5 (profiles/replay_shares.txt).
// A tile's costs: what its instructions take beside the memory's time, which all widths have alike, measured as the ratios that are fastest: 1.8 to 2.2 with
// bf16 tensors of five workers and more, 1.1 to 1.25 where a hop moves more bytes (fp32, or a result of 4 bytes per two or three workers).  (12/15/16
// instead of 12/24/26 for the first ring above: 64.2.  58 schedules over 4 in bf16 with 12/20/22 1.2 % faster than with 12/14/15, halving of 9,872/24,561/2,107 25.6 -> 23.1; 92 over 2
// and 3 1.2 % slower.)  A raw tile has the fewest instructions but waits for every slice: as dear as a 2-bit one it came four
// to a wave where others held one (bf16 ring of 24, 5,354/9,868/5,525/10,261: 111 to 116 us, 95 so, 98 with equal counts).  It is no dearer in bf16 halvings
// over 16 workers and more, whose stack it hardly uses (55 schedules at 2 to 4 tiles per wave 1 % faster so), and in tiles of one and two, where it is the shortest (halving over 8 of
// 1,126/427/565/2,058 12.6 us, 14.1 at 15; 110 schedules the same or faster).
Costs costs_of(dq_dtype dtype, bool tree, uint32_t n, uint32_t tile_sgs) {
  const uint32_t raw = tile_sgs < kWaveSGs || (dtype != DQ_F32 && tree && n > 12) ? 12 : 15;
  if (dtype == DQ_F32 || n <= 3) return Costs{{12, 14, 15, raw}};
  return tree || n == 4 ? Costs{{12, 20, 22, raw}} : Costs{{12, 24, 26, raw}};
}
namespace {
// The most tiles per wave of every width (0: there is none of it), at most `waves` waves.
void most_per_wave(const uint64_t tiles[4], const uint32_t cost[4], uint32_t waves, uint64_t most[4]) {
  auto fits = [&] {
    double need = 0;
    for (int w = 0; w < 4; ++w)
      if (tiles[w]) {
        if (most[w] == 0) return false;
        need += (double)tiles[w] / (double)most[w];
      }
    return need <= (double)waves;
  };
  auto within = [&](uint64_t s) {
    for (int w = 0; w < 4; ++w) most[w] = !tiles[w] ? 0 : s >> 32 ? s / cost[w] : (uint32_t)s / cost[w];
    return fits();
  };
  // the least cost of the fullest wave, which is at least the mean
  uint64_t all = 0, lo, hi, by = cost[0];
  for (int w = 0; w < 4; ++w) all += tiles[w] * cost[w];
  lo = all / waves ? all / waves - 1 : 0;
  for (hi = lo + by; !within(hi); hi += by *= 2) lo = hi;
  while (hi - lo > 1) {
    const uint64_t mid = lo + (hi - lo) / 2;
    if (within(mid)) hi = mid; else lo = mid;
  }
  within(hi);
  for (bool less = true; less;) {
    less = false;
    int order[4] = {0, 1, 2, 3};
    for (int i = 1; i < 4; ++i)
      for (int k = i; k > 0 && most[order[k]] * cost[order[k]] > most[order[k - 1]] * cost[order[k - 1]]; --k) {
        const int t = order[k];
        order[k] = order[k - 1];
        order[k - 1] = t;
      }
    for (int i = 0; i < 4 && !less; ++i) {
      const int w = order[i];
      if (most[w] < 2) continue;
      --most[w];
      less = fits();
      if (!less) ++most[w];
    }
  }
}
}  // namespace

void split_walk(const WalkPath *paths, dq_dtype dtype, bool tree, const Walk &W, std::vector<WalkShare> *shares) {
  const uint32_t sgs = W.tile_sgs, n = W.blocks * W.waves;
  uint64_t tiles[4] = {0, 0, 0, 0}, most[4], cost[4], total = 0;
  for (uint32_t p = 0; p < W.n_paths; ++p)
    for (int w = 0; w < 4; ++w) tiles[w] += (paths[p].job.n_sg[w] + sgs - 1) / sgs;
  const Costs c = costs_of(dtype, tree, W.n, sgs);
  most_per_wave(tiles, c.of, n, most);
  // Equal shares of cost total / n hold at most `most` tiles of a width that costs at least that over `most`.  The costs rise until that is so, each
  // round by less; where the waves are just enough it is so at the cost of the fullest.
  constexpr uint64_t kUnit = 1u << 20;
  uint64_t fullest = 0;
  for (int w = 0; w < 4; ++w) {
    cost[w] = c.of[w] * kUnit;
    fullest = most[w] * cost[w] > fullest ? most[w] * cost[w] : fullest;
  }
  for (int round = 0;; ++round) {
    total = 0;
    for (int w = 0; w < 4; ++w) total += tiles[w] * cost[w];
    const uint64_t share = round < 8 ? (total + n - 1) / n : fullest;
    bool raised = false;
    for (int w = 0; w < 4; ++w)
      if (most[w] && cost[w] * most[w] < share) {
        cost[w] = (share + most[w] - 1) / most[w];
        raised = true;
      }
    if (!raised || round > 8) break;
  }
  shares->resize((size_t)n + 1);
  // Share v begins with the first tile whose cost before it reaches want = floor(v * total / n); over = that division's remainder.
  WalkShare *share = shares->data(), *const end = share + n;
  const uint64_t step = total / n, rest = total % n;
  uint64_t tiles_on[4], part_on[4];  // step in tiles
  for (int w = 0; w < 4; ++w) {
    tiles_on[w] = step / cost[w];
    part_on[w] = step % cost[w];
  }
  uint64_t want = 0, over = 0, before = 0;  // before: cost of all runs of one width before this one
  for (uint32_t p = 0; p < W.n_paths; ++p) {
    uint32_t first = 0;  // tile of this run
    for (int w = 0; w < 4; ++w) {
      const uint32_t count = (paths[p].job.n_sg[w] + sgs - 1) / sgs;
      if (count == 0) continue;
      const uint64_t each = cost[w], last = before + (count - 1) * each;
      // The shares that begin in this run: at = tile * each + part.  (With a division per share 2,049 shares took the host 15 us of a
      // plan's 17.)
      uint64_t tile = 0, part = 0;
      bool inside = false;
      while (share != end && want <= last) {
        if (!inside && want >= before) {
          tile = (want - before) / each;
          part = (want - before) % each;
          inside = true;
        }
        *share++ = WalkShare{p, first + (uint32_t)(inside ? tile + (part != 0) : 0)};
        over += rest;
        const uint64_t carry = over >= n ? 1 : 0;
        over -= n & (0 - carry);
        want += step + carry;
        if (inside) {
          tile += tiles_on[w];
          part += part_on[w] + carry;
          if (part >= each) {
            part -= each;
            ++tile;
          }
        }
      }
      before += count * each;
      first += count;
    }
  }
  while (share != end + 1) *share++ = WalkShare{W.n_paths, 0};
}

hipError_t launch_walk(dq_dtype dtype, bool tree, bool means, const WalkPath *paths, const WalkShare *shares, const WalkGrid &W,
                       const Params &P, hipStream_t s) {
  if (W.tile_sgs < kWaveSGs) return launch_thin(dtype, tree, paths, shares, W, P, s);
  const bool f32 = dtype == DQ_F32;
#define DQ_WALK(T, M) (tree ? go_walk<T, M, true>(paths, shares, W, P, s) : go_walk<T, M, false>(paths, shares, W, P, s))
  if (means) return f32 ? DQ_WALK(float, true) : DQ_WALK(uint16_t, true);
  return f32 ? DQ_WALK(float, false) : DQ_WALK(uint16_t, false);
#undef DQ_WALK
}

}  // namespace dq

// The shares of a launch, for the tests: n_sg[p][4] super-groups by width of every path; shares[2 * (blocks * waves + 1)].
extern "C" void dqx_split(const uint32_t *n_sg, uint32_t n_paths, uint32_t n_workers, int f32, int tree, uint32_t tile_sgs, uint32_t blocks,
                          uint32_t waves, uint32_t *shares) {
  std::vector<dq::WalkPath> paths(n_paths, dq::WalkPath{});
  for (uint32_t p = 0; p < n_paths; ++p) memcpy(paths[p].job.n_sg, n_sg + 4 * (size_t)p, 16);
  dq::WalkGrid W = {};
  W.n = n_workers;
  W.n_paths = n_paths;
  W.tile_sgs = tile_sgs;
  W.blocks = blocks;
  W.waves = waves;
  std::vector<dq::WalkShare> s;
  dq::split_walk(paths.data(), f32 ? DQ_F32 : DQ_BF16, tree != 0, W, &s);
  memcpy(shares, s.data(), s.size() * sizeof(dq::WalkShare));
}
