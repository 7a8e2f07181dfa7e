// A whole replay in one launch, as dq_walk.hip, for schedules with few super-groups: a lane holds E = 4 or 8 entries of
// a group, not all 16, so a wave's tile is E / 4 super-groups and there are 16 / E times as many waves.
//
// Why: a tile's hops are a serial chain.  With a tile of four super-groups per wave, a schedule of fewer than some 4,000
// super-groups leaves most SIMDs with one wave or none, and a hop takes 1.1 us whatever the size: the instructions of 16
// entries one after the other, then the next slice's trip from memory.  With 4 entries per lane the chain of a hop is a
// quarter of it, and the slices are requested four hops ahead (they are two registers each): 0.45 to 0.5 us per hop.  Measured, bf16, wide
// tile to E = 8 to E = 4: ring of 100, 1,000 super-groups, 114 -> 68 -> 50 us; 64 workers' recursive halving 94 -> 48 -> 34;
// ring of 256, 4,096 super-groups of 2 to 16 bits, 284 -> 209 -> 222 (profiles/replay_tile_sizes.txt).  grid_walk (dq_walk.hip) says which
// schedules come here.
//
// What bounds it is how much of a hop's chain four waves per SIMD cover: two vector instructions can go per four cycles, from two waves,
// and about half of that is reached (256 workers, 4,096 super-groups: 93 instructions per hop, 159 to 169 us from card to card; 88 would be their issue).  So all
// instructions count, on the path or beside it, scalar ones and waits too.  Earlier states against each other, in turn on one card, as are the pairs further down: both super-group
// draws made by one generator call, the next four tensors by one scalar load and the group scale left in fp32 took 188 us there to 184, four workers' fp32 ring of 4,096 with
// all-gather from 9.9 to 9.1; the super-group's maximum and scale in scalar registers and the rounding of the group scale in two instructions 185 to 177.
// (All comparisons of a hop before its selections, which saves the waits between them: 192.)
//
// What differs from the wide tile:
//   draws    : a lane draws the group's 16 bytes for ONE of the next 16 / E hops, and the group's lanes exchange them through
//              LDS: per hop and group one generator call, as before.  Per-super-group draws cover 128 / E hops at a time.
//   maxima   : within a group by quad permutes, within a super-group by row rotates and row / half-wave swaps.
//   rounding : levels are looked up with 1 / maximum while the stored scales are still being worked out.  A group whose
//              scale rounds to zero then has levels that are not zero, but they are multiplied by zero.
//   messages : pending ones are signed levels and scale, also those of a recursive halving in LDS: nothing is decoded.
//   result   : a lane's entries are whole 16-byte pieces, stored as they are.
#include "dq_walk.h"

namespace dq {
namespace {

constexpr uint32_t kAhead = 4;  // hops a slice is requested ahead of its use
constexpr uint32_t kThinPark = 656;    // per wave: 32 scale draws of 16 bytes, 32 permutation slots, 16 bytes of zero
constexpr uint32_t kThinDraws = 1536;  // per wave: 64 groups' (of some hop) 16 bytes, their rounding offset and scale dither
constexpr uint32_t kThinWaves = 4;     // per block
static_assert(kThinWaves * kThinDraws <= (kOffTab4 - kOffDec2) * 4, "the draws lie over the decode tables, which are not copied");

template <int E>
constexpr uint32_t kThinStack = E * 256 + 256;  // per wave and level: signed levels and scale

__device__ __forceinline__ void lds_st2(uint32_t a, u32x2 v) {
  *reinterpret_cast<__attribute__((address_space(3))) u32x2 *>(a) = v;
}
__device__ __forceinline__ void lds_turn() {  // the wave's LDS writes before here, its reads after
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename LT, int E>
struct Bit {
  uint32_t w[E * sizeof(LT) / 4];  // a lane's E entries, raw
};
template <typename LT, int E>
__device__ __forceinline__ Bit<LT, E> load_bit(uint64_t tensor, uint64_t at) {
  constexpr int kWords = E * sizeof(LT) / 4;
  const uint8_t *p = reinterpret_cast<const uint8_t *>(tensor) + at;
  Bit<LT, E> s;
  if constexpr (kWords == 2) {
    const u32x2 t = gld<u32x2>(p);
    s.w[0] = t.x; s.w[1] = t.y;
  } else {
#pragma unroll
    for (int i = 0; i < kWords / 4; ++i) {
      const u32x4 t = gld<u32x4>(p + 16 * i);
      s.w[4 * i] = t.x; s.w[4 * i + 1] = t.y; s.w[4 * i + 2] = t.z; s.w[4 * i + 3] = t.w;
    }
  }
  return s;
}

// Address of the i-th tensor a chunk meets.  (The table holds every tensor twice: a ring's leaves are consecutive entries.)
template <bool TREE>
__device__ __forceinline__ uint64_t tensor_of(const Walk &W, uint32_t chunk, uint32_t i) {
  return table_entry(reinterpret_cast<const uint64_t *>(W.grads), TREE ? leaf_of<TREE>(W, chunk, i) : (W.chain ? 0u : chunk) + i);
}

// Maximum over a super-group of which every lane of the wave has its group's maximum.  (As one block, as the compiler makes three instructions of each of the
// last two maxima.  A maximum reads what the one before it wrote from other lanes: two wait states between them.)
__device__ __forceinline__ uint32_t wave_max(uint32_t x) {
  asm("s_nop 1\n\t"
      "v_max_u32_dpp %0, %0, %0 row_ror:4 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_max_u32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_max_u32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"  // row 0 into 1, row 2 into 3
      "s_nop 1\n\t"
      "v_max_u32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"  // row 1 into 2 and 3
      "s_nop 1"
      : "+v"(x));
  return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);  // outside: the compiler knows what has to stand between it and a vector instruction's read
}

// What the search leads to: a level, the next one, and the step between them.  As 16 bytes, or as 8, T and the next T, with the step a subtraction.
template <bool SHORT>
struct Level {
  u32x4 w;  // T, step, next T, index << (32 - width)
  __device__ __forceinline__ void load(uint32_t sign, uint32_t pair) { w = lds_ld4(or_and(sign, 16u, pair)); }
  __device__ __forceinline__ uint32_t here() const { return w.x; }
  __device__ __forceinline__ uint32_t next() const { return w.z; }
  __device__ __forceinline__ float step() const { return u2f(w.y); }
  template <int B>
  __device__ __forceinline__ uint32_t index() const { return w.w >> (32 - B); }
};
template <>
struct Level<true> {
  u32x2 w;
  uint32_t at;
  __device__ __forceinline__ void load(uint32_t sign, uint32_t pair) {
    at = or_and(sign >> 1, 8u, pair);
    w = lds_ld2(at);
  }
  __device__ __forceinline__ uint32_t here() const { return w.x; }
  __device__ __forceinline__ uint32_t next() const { return w.y; }
  __device__ __forceinline__ float step() const { return u2f(w.y) - u2f(w.x); }
  template <int B>
  __device__ __forceinline__ uint32_t index() const {  // pair r has the entries of r + 1 and r
    return ((at - (B == 4 ? kOffTab4 : kOffTab8) * 4) >> 4) + 1 - (at >> 3 & 1u);
  }
};

// What a wave holds of a tile before it walks it: where it is and the slices of its first hops.
template <typename LT, int E>
struct Start {
  TilePos pos;
  uint64_t at;  // byte offset of the lane's entries inside every worker's tensor
  float mu;
  uint32_t dest;  // with one super-group per wave: where its result goes, and what is added to it
  float back;
  Bit<LT, E> s[kAhead];
};

template <typename LT, bool TREE, int E>
__device__ __forceinline__ Start<LT, E> start_tile(const WalkPath &path, const Walk &W, uint32_t t) {
  constexpr uint32_t kSgs = E / 4;
  const Job &job = path.job;
  Start<LT, E> x;
  uint32_t first = 0, w = 0;
#pragma unroll
  for (; w < 3; ++w) {
    const uint32_t tiles = (job.n_sg[w] + kSgs - 1) / kSgs;
    if (t < tiles) break;
    t -= tiles;
    first += job.n_sg[w];
  }
  x.pos = TilePos{first, w == 0 ? job.n_sg[0] : w == 1 ? job.n_sg[1] : w == 2 ? job.n_sg[2] : job.n_sg[3], t * kSgs, (int)w};
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t row = min(lane * kSgs / 64u, x.pos.n_seg - 1 - x.pos.tile_first);
  const uint32_t sg0 = first + x.pos.tile_first + row;
  const uint64_t sg = job.src ? (uint64_t)gld<uint32_t>(job.src + sg0) : (uint64_t)sg0;
  x.mu = job.mu ? gld<float>(job.mu + sg0) : 0.0f;  // taking off 0 changes nothing
  if constexpr (E == 4) {  // on the index's trip, not one of their own behind the last hop
    x.dest = sg0;
    x.back = 0.0f;
    if (job.dest) x.dest = (uint32_t)__builtin_amdgcn_readfirstlane((int)(job.dest == job.src ? (uint32_t)sg : gld<uint32_t>(job.dest + sg0)));
    if (job.back) x.back = u2f((uint32_t)__builtin_amdgcn_readfirstlane((int)f2u(job.back == job.mu ? x.mu : gld<float>(job.back + sg0))));
  }
  x.at = (uint64_t)reinterpret_cast<uintptr_t>(job.local) + sg * (kSG * sizeof(LT)) + (lane & (64u / kSgs - 1u)) * (E * (uint32_t)sizeof(LT));
#pragma unroll
  for (uint32_t j = 0; j < kAhead; ++j) {
    x.s[j] = load_bit<LT, E>(tensor_of<TREE>(W, path.chunk, min(j, W.n - 1)), x.at);
  }
  return x;
}

// Places of the tile in a packed chunk, worked out here and now: the compiler would otherwise keep them in registers around
// the hops of which only two write a message.
template <int B>
__device__ __forceinline__ TileBase<B> tile_base_here(const Job &job, const TilePos &pos) {
  Job j = job;
  TilePos p = pos;
  asm volatile("" : "+s"(j.n_sg[0]), "+s"(j.n_sg[1]), "+s"(j.n_sg[2]), "+s"(j.n_sg[3]), "+s"(p.seg_first), "+s"(p.tile_first));
  return TileBase<B>(j, p);
}

// B: 2, 4, 8, or 16 (raw: the message is the partial sum rounded to bf16)
template <int B, typename LT, bool TREE, int E, int SHORT>
__device__ __forceinline__ void walk_thin(const WalkPath &path, const Params &P, const Vec &V, const Walk &W, uint32_t park, uint32_t draws,
                                          uint32_t stack0, Start<LT, E> &x) {
  constexpr uint32_t kLanes = 16 / E, kSgs = E / 4, kHops = 32 / kSgs;  // lanes per group, super-groups per tile, hops per park
  const Job &job = path.job;
  const TilePos pos = x.pos;
  const uint32_t lane = threadIdx.x & 63u, q = lane & (kLanes - 1u), g = (lane / kLanes) & 15u;
  const uint32_t row = min(lane * kSgs / 64u, pos.n_seg - 1 - pos.tile_first);
  const uint64_t gi = (job.first_sg + pos.seg_first + pos.tile_first + row) * 16 + g;  // global group index
  const uint32_t last = W.n - 1, zeros = park + 640;
  float v[E], level[E], sfg = 0.0f;  // the pending message: level * sfg
#pragma unroll
  for (int k = 0; k < E; ++k) level[k] = -0.0f;  // nothing pending: adding -0 changes nothing
  auto widen = [&](const Bit<LT, E> &b, float (&y)[E]) {
    if constexpr (sizeof(LT) == 4) {
#pragma unroll
      for (int k = 0; k < E; ++k) y[k] = u2f(b.w[k]) - x.mu;
    } else {
#pragma unroll
      for (int k = 0; k < E / 2; ++k) {
        y[2 * k] = u2f(b.w[k] << 16) - x.mu;
        y[2 * k + 1] = u2f(b.w[k] & 0xFFFF0000u) - x.mu;
      }
    }
  };
  // Whether a hop's steps stand in the order in which the next needs them: the searches, beside their trip to LDS the scale of the super-group; the levels,
  // beside theirs all that does not depend on them: the group's scale, the random numbers, the next hop's entries.  Where a wave is alone or in
  // throughput, bf16 rings are faster so (256 workers 172.8 -> 171.0 us, 100 of 2,000 super-groups 47.3 -> 46.3); in fp32, whose entries then wait
  // for memory a hop earlier, slower (32 of 4,096 30.3 -> 32.9), and recursive halvings (128 of 384 53.6 -> 54.8).
  constexpr bool kEarly = !TREE && E == 4 && sizeof(LT) == 2;
  float next[E];  // kEarly: the next hop's entries
  if constexpr (kEarly) widen(x.s[0], next);

  // kAhead hops from i0 on.  PLAIN: all of them encode, none writes its message, and the slices to request exist.
  auto some_hops = [&](uint32_t i0, auto plain) {
    constexpr bool PLAIN = decltype(plain)::value;
    uint64_t tensor[kAhead];
    if constexpr (PLAIN && !TREE) {  // a run of the table: one scalar load
      struct Run { uint64_t at[kAhead]; };
      const Run run = table_entry(reinterpret_cast<const Run *>(W.grads + (W.chain ? 0u : path.chunk) + i0 + kAhead), 0u);
#pragma unroll
      for (uint32_t j = 0; j < kAhead; ++j) tensor[j] = run.at[j];
    } else
#pragma unroll
    for (uint32_t j = 0; j < kAhead; ++j) tensor[j] = tensor_of<TREE>(W, path.chunk, PLAIN ? i0 + kAhead + j : min(i0 + kAhead + j, last));
#pragma unroll
    for (uint32_t j = 0; j < kAhead; ++j) {
      // A hop past the last (the last four may be fewer) does nothing but load: behind a condition, or a way out of the loop, the
      // compiler would load into other registers and wait at every hop's end to move the data.
      const uint32_t i = i0 + j;
      __builtin_amdgcn_sched_barrier(0);
      float y[E];
      if constexpr (!kEarly) widen(x.s[j], y);
      x.s[j] = load_bit<LT, E>(tensor[j], x.at);  // past the last hop: the last slice again, out of the cache
      if (PLAIN || i <= last) {
        if constexpr (B != 16) {
          if (j % kLanes == 0) {
            if (j == 0 && (i & (kHops - 1u)) == 0) {  // the super-groups' draws of the next kHops hops: lane = stream, hop, super-group
              const uint32_t l = lane & 31u, r = min(l & (kSgs - 1u), pos.n_seg - 1 - pos.tile_first);
              const uint64_t G = job.first_sg + pos.seg_first + pos.tile_first + r;
              const uint32_t rank = leaf_of<TREE>(W, path.chunk, min(i + l / kSgs, last));
              const U4 w = philox4x32_10((uint32_t)G, (uint32_t)(G >> 32), P.round, lane < 32 ? (1u << 16) | (rank & 0xFFFFu) : (2u << 16) | 0xFFFFu,
                                         P.key0, P.key1);
              const uint32_t slot = perm_slot(w, P, rank);  // of the shared draw; nothing in the other half
              lds_turn();
              if (lane < 32) lds_st4(park + l * 16, u32x4{w.x, w.y, w.z, w.w});
              else lds_st1(park + 512 + l * 4, slot);
              lds_turn();
            }
            // the groups' draws of the next kLanes hops: lane q of a group draws for hop i + q
            const uint32_t slot = ((i + q) & (kHops - 1u)) * kSgs + row;
            const Draws d = draw_group(P, gi, leaf_of<TREE>(W, path.chunk, min(i + q, last)), lds_ld1(park + 512 + slot * 4),
                                       lds_ld1(park + slot * 16 + (g >> 2) * 4), g);
            lds_turn();
            lds_st4(draws + q * (64 * E) + (lane / kLanes) * 16, u32x4{d.gam.x, d.gam.y, d.gam.z, d.gam.w});
            lds_st2(draws + 1024 + q * (512 / kLanes) + (lane / kLanes) * 8, u32x2{f2u(d.o_pi), f2u(d.us)});
            lds_turn();
          }
        }
        uint32_t gam[E / 4];
        u32x2 offset = {0, 0};
        if constexpr (B != 16) {
          constexpr uint32_t kHop = 64 * E;
          const uint32_t jj = j % kLanes;
          if constexpr (E == 4) {
            gam[0] = lds_ld1(draws + jj * kHop + lane * 4);
          } else {
            const u32x2 t = lds_ld2(draws + jj * kHop + lane * 8);
            gam[0] = t.x; gam[1] = t.y;
          }
          offset = lds_ld2(draws + 1024 + jj * (512 / kLanes) + (lane / kLanes) * 8);
        }
#pragma unroll
        for (int k = 0; k < E; ++k) v[k] = kEarly ? next[k] : y[k];
        if constexpr (B == 16 && kEarly) widen(x.s[(j + 1) % kAhead], next);
        if (!TREE || (j & 1)) {
#pragma unroll
          for (int k = 0; k < E; ++k) v[k] = B == 16 ? level[k] + v[k] : __builtin_fmaf(level[k], sfg, v[k]);
        }
        uint32_t stack = stack0;
        if constexpr (TREE) {
          if (j == 3) {
#pragma unroll 1
            for (uint32_t up = i >> 1; up & 1u; up >>= 1, stack += kThinStack<E>) {
              const float f = u2f(lds_ld1(stack + E * 256 + lane * 4));
#pragma unroll
              for (int h = 0; h < E / 4; ++h) {
                const f32x4 t = lds_ldf4(stack + h * 1024 + lane * 16);
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * h + k] = B == 16 ? t[k] + v[4 * h + k] : __builtin_fmaf(t[k], f, v[4 * h + k]);
              }
            }
          }
        }
        if (PLAIN || i < W.encodes) {
          const bool keep = !TREE && !PLAIN && i >= W.first_kept && i < last;  // the message is written
          if constexpr (B == 16) {
            uint32_t w[E / 2];
#pragma unroll
            for (int k = 0; k < E / 2; ++k) {
              w[k] = bf16_rne_pair(v[2 * k], v[2 * k + 1]);
              level[2 * k] = u2f(w[k] << 16);
              level[2 * k + 1] = u2f(w[k] & 0xFFFF0000u);
            }
            if (keep) {
              uint8_t *dst = message_of(path, i) + tile_base_here<16>(job, pos).code_off + (row * 16 + g) * 32 + q * (2 * E);
              if constexpr (E == 4) gst<u32x2>(dst, u32x2{w[0], w[1]});
              else gst<u32x4>(dst, u32x4{w[0], w[1], w[2], w[3]});
            }
          } else {
            float m = 0.0f;
#pragma unroll
            for (int k = 0; k < E; ++k) m = fmaxf(m, fabsf(v[k]));
            const uint32_t mg = group_max<E>(f2u(m));
            m = u2f(mg);
            // Levels: a stored scale above zero implies m > 2^-118 (the super-group's is at least 2^-100, and the dither at least
            // 1/512), so the bound only keeps the quotient finite where the levels do not count.
            const float inv = TREE ? (m >= 0x1p-120f ? 1.0f / m : 0.0f) : reciprocal(u2f(max(mg, f2u(0x1p-120f))));
            // The scales, as in scale_group.  With one super-group per wave its maximum and what follows from it are scalar, and a
            // super-group that is encoded as zero finds zeros for its reciprocals.  With two such a one has its groups' maxima taken as zero instead
            // of its results: as conditional results the compiler puts the chain behind a branch, after the levels' lookups.
            uint32_t sfb, ex;
            u32x2 rec;
            auto look_up_scale = [&] {
              const uint32_t top = (E == 4 ? wave_max(mg) : sg_max<E>(mg)) + 0xFFFFu;
              const bool tiny = top < 0x0D800000u;
              const uint32_t b = tiny ? 0u : top;
              sfb = b >> 16;
              ex = b & 0x7F800000u;
              rec = lds_ld2(E == 4 && tiny ? zeros : kRec0 + ((b >> 13) & 0x3F8u));
              if (E != 4 && tiny) m = 0.0f;
            };
            if constexpr (!kEarly) look_up_scale();
            float xs[E], u[E];
            u32x2 e[E];
            constexpr bool kShort = B == 8 ? SHORT >= 1 : SHORT == 2;
            Level<kShort> t[E];
#pragma unroll
            for (int k = 0; k < E; ++k) {
              xs[k] = v[k] * inv;
              if constexpr (B != 2) e[k] = lds_ld2(f2u(fabsf(xs[k]) + (B == 4 ? V.magic4 : V.magic8)) & 0x1FFF8u);
            }
            if constexpr (B != 2 || kEarly) __builtin_amdgcn_sched_barrier(0);  // all searches, then all levels: two trips to LDS, not eight
            if constexpr (kEarly) {  // beside the searches
              look_up_scale();
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (B != 2) {
#pragma unroll
              for (int k = 0; k < E; ++k) t[k].load(f2u(fabsf(xs[k]) - u2f(e[k].x)) >> 27, e[k].y);
            }
            __builtin_amdgcn_sched_barrier(0);
            auto uniform = [&](int k) { return __builtin_fmaf((float)((gam[k >> 2] >> (8 * (k & 3))) & 0xFFu), V.s_n, u2f(offset.x)); };
            if constexpr (kEarly) {  // beside the levels
#pragma unroll
              for (int k = 0; k < E; ++k) u[k] = uniform(k);
              widen(x.s[(j + 1) % kAhead], next);
            }
            // floor(ts) + [us < ts - floor(ts)] is the ceiling of ts - us: that difference is exact, or lies between -1 and 0
            const float ts = fminf(m * u2f(rec.y - ex), 255.0f), rg = fabsf(ceilf(ts - u2f(offset.y)));
            sfg = rg * fabsf(u2f(rec.x + ex));  // (without an exponent to add, the table's pattern has the sign bit)
            if constexpr (kEarly) __builtin_amdgcn_sched_barrier(0);
            bool up[E];
#pragma unroll
            for (int k = 0; k < E; ++k) {
              const float ax = fabsf(xs[k]);
              if constexpr (!kEarly) u[k] = uniform(k);
              if constexpr (B == 2) {
                up[k] = u[k] < ax;
                level[k] = u2f(or_and(f2u(xs[k]), V.top, f2u(up[k] ? 1.0f : 0.0f)));
              } else {
                up[k] = __builtin_fmaf(u[k], t[k].step(), u2f(t[k].here())) < ax;
                level[k] = u2f(or_and(f2u(xs[k]), V.top, up[k] ? t[k].next() : t[k].here()));
              }
            }
            // A level's fourth word counts as read here: the compiler would take its register for another purpose while the read is under way, and wait
            // for the first entry's level before it asks for the others' (ring of 16, 496 super-groups, 10.0 us instead of 9.5; a chain of 100 of 600 in fp32
            // 43.4 and 39.9).  With eight entries per lane there are no registers for that: halving over 8 of 5,600 in fp32 14.8 instead of 13.1.
            if constexpr (B != 2 && !kShort && E == 4) {
#pragma unroll
              for (int k = 0; k < E; ++k) asm volatile("" ::"v"(t[k].w.w));
            }
            if (keep) {
              const TileBase<B> tb = tile_base_here<B>(job, pos);
              uint8_t *out = message_of(path, i);
              const uint32_t lg = row * 16 + g;
              uint64_t word = 0;
#pragma unroll
              for (int k = E - 1; k >= 0; --k) {
                const uint32_t index = B == 2 ? 0u : t[k].template index<B>();
                word = (word << B) | (f2u(xs[k]) >> 31 << (B - 1)) | (rg != 0.0f ? index + (up[k] ? 1u : 0u) : 0u);
              }
              uint8_t *cp = out + tb.code_off + lg * (2 * B) + q * (E * B / 8);
              if constexpr (E * B == 8) gst<uint8_t>(cp, (uint8_t)word);
              else if constexpr (E * B == 16) gst<uint16_t>(cp, (uint16_t)word);
              else if constexpr (E * B == 32) gst<uint32_t>(cp, (uint32_t)word);
              else gst<u32x2>(cp, u32x2{(uint32_t)word, (uint32_t)(word >> 32)});
              gst<uint8_t>(out + tb.gs_off + lg, (uint8_t)rg);  // all lanes of a group, of a super-group: the same value
              gst<uint16_t>(out + tb.sf_off + row * 2, (uint16_t)sfb);
            }
          }
          if constexpr (TREE) {
            if ((j & 1) && (PLAIN || i < last)) {
#pragma unroll
              for (int h = 0; h < E / 4; ++h)
                lds_stf4(stack + h * 1024 + lane * 16, f32x4{level[4 * h], level[4 * h + 1], level[4 * h + 2], level[4 * h + 3]});
              lds_st1(stack + E * 256 + lane * 4, f2u(sfg));
            }
          }
        }
      }
    }
  };
  uint32_t i0 = 0;
  for (; i0 + 2 * kAhead <= W.n && (TREE || i0 + kAhead <= W.first_kept); i0 += kAhead) some_hops(i0, Is<true>());
  for (; i0 < W.n; i0 += kAhead) some_hops(i0, Is<false>());
  if (W.encodes == W.n) {  // what every worker decodes from the sink's message
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = B == 16 ? level[k] + 0.0f : level[k] * sfg;
  }
  const size_t sg0 = (size_t)pos.seg_first + pos.tile_first + row;
  if (job.back) {
    const float back = (float)P.n_workers * (E == 4 ? x.back : gld<float>(job.back + sg0));
#pragma unroll
    for (int k = 0; k < E; ++k) v[k] = v[k] + back;
  }
  const size_t sg = E == 4 ? (size_t)x.dest : job.dest ? (size_t)gld<uint32_t>(job.dest + sg0) : sg0;
  float *out = static_cast<float *>(job.out) + sg * kSG + (lane & (64u / kSgs - 1u)) * E;
#pragma unroll
  for (int h = 0; h < E / 4; ++h) gst_once<f32x4>(out + 4 * h, f32x4{v[4 * h], v[4 * h + 1], v[4 * h + 2], v[4 * h + 3]});
}

// SHORT: which levels are 8 bytes, by the number of the tables behind the blob: 1 the 8-bit ones, 2 both.
//   8-bit : a wave's lanes read as many of the set's 254 entries at a time as the LDS has room for; with four waves per SIMD it was busy two thirds of the time
//           (256 workers, 4,096 super-groups of 2 to 16 bits 164.5 -> 159.4 us; 32 of 8,000 at 6 bits 39.6 -> 38.9, in fp32 64 of 4,992 65.9 ->
//           64.4).  Not in bf16 rings and chains of up to two waves per SIMD, where the subtraction is on the one wave's way (100 of 2,000 41.0 -> 41.7), nor in
//           any of up to eight workers, which have too few hops for the fewer conflicts to count (us of a ring, long -> short: bf16, 4 of 3,584 8.2 -> 8.3, 8 of them
//           10.6 -> 10.8; fp32, 3 of 1,024 5.27 -> 5.36.  Means over three mixtures and up to 16 super-groups per CU, over 4, 8, 12 and 16 workers: bf16 with more than two
//           waves per SIMD 1.5 and 0.8 % longer, 0.2 and 1.1 % less; fp32 0.6 and 0.3 longer, 0.3 and 0.8 less).
//   4-bit : 14 entries, read by many lanes at once whatever their size; but halvings with tiles of two need no scratch memory so (over 16 of 5,600 23.1 -> 19.5, over
//           32 of 4,096 27.0 -> 23.5, over 64 62.0 -> 56.5), and bf16 rings with tiles of two less of it (100 of 6,000 at 5 bits 86.5, with the 8-bit ones alone 87.8).
//   fp32 rings with tiles of two have neither (16 of 4,992 20.0; 20.3 with any).
template <typename LT, bool TREE, int E, int SHORT>
__global__ __launch_bounds__(kThinWaves * 64) __attribute__((amdgpu_waves_per_eu((E == 4 || sizeof(LT) == 2 ? 4 : 3)))) void k_thin(
    const WalkPath *paths, const WalkShare *shares, Walk W, Params P) {
  extern __shared__ uint4 lds_raw[];
  uint32_t *lds = reinterpret_cast<uint32_t *>(lds_raw);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t share = __builtin_amdgcn_readfirstlane(share_of<false>(W, wave, kThinWaves));
  WalkShare at = table_entry(shares, share);
  const WalkShare to = table_entry(shares, share + 1);
  const bool any = at.path < to.path || (at.path == to.path && at.tile < to.tile);
  WalkPath path;
  Start<LT, E> x;
  if (any) {  // the first tile's entries are on their way while the tables are copied
    path = table_entry(paths, at.path);
    x = start_tile<LT, TREE, E>(path, W, at.tile);
  }
  copy_tables(lds, P.blob + SHORT * P.blob_dwords, P, kOffTab4);  // nothing is decoded from codes
  __syncthreads();
  if (!any) return;
  const uint32_t draws = kOffDec2 * 4 + wave * kThinDraws, park = P.blob_dwords * 4 + wave * kThinPark;
  const uint32_t stack = P.blob_dwords * 4 + kThinWaves * kThinPark + wave * W.stack_bytes;
  lds_st4(park + 640, u32x4{0, 0, 0, 0});
  const Vec V(P);
  for (;;) {
    if (x.pos.wi == 0) walk_thin<2, LT, TREE, E, SHORT>(path, P, V, W, park, draws, stack, x);
    else if (x.pos.wi == 1) walk_thin<4, LT, TREE, E, SHORT>(path, P, V, W, park, draws, stack, x);
    else if (x.pos.wi == 2) walk_thin<8, LT, TREE, E, SHORT>(path, P, V, W, park, draws, stack, x);
    else walk_thin<16, LT, TREE, E, SHORT>(path, P, V, W, park, draws, stack, x);
    ++at.tile;
    uint32_t tiles = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) tiles += (path.job.n_sg[w] + E / 4 - 1) / (E / 4);
    if (at.tile == tiles) { ++at.path; at.tile = 0; }
    if (at.path > to.path || (at.path == to.path && at.tile >= to.tile)) break;
    path = table_entry(paths, at.path);
    x = start_tile<LT, TREE, E>(path, W, at.tile);
  }
}

template <typename LT, bool TREE>
constexpr int kShortPairs = TREE || sizeof(LT) == 2 ? 2 : 0;  // tiles of two
template <bool TREE>
constexpr int kShortSingles = TREE ? 2 : 1;
constexpr uint32_t kFewHops = 8;  // of a ring or chain whose levels all have 16 bytes
template <typename LT, bool TREE>
hipError_t go_thin(const WalkPath *paths, const WalkShare *shares, const WalkGrid &W, const Params &P, hipStream_t s) {
  const uint32_t lds = thin_lds(P, W.stack_bytes);
  auto kernel = k_thin<LT, TREE, 8, kShortPairs<LT, TREE>>;
  if (W.tile_sgs == 1) kernel = k_thin<LT, TREE, 4, kShortSingles<TREE>>;
  if constexpr (!TREE)
    if (W.tile_sgs == 1 && (W.n <= kFewHops || (sizeof(LT) == 2 && !W.full))) kernel = k_thin<LT, TREE, 4, 0>;
  hipLaunchKernelGGL(kernel, dim3(W.blocks), dim3(kThinWaves * 64), lds, s, paths, shares, W, P);
  return hipGetLastError();
}

template <typename LT>
hipError_t static_lds_of(size_t *bytes) {
  hipError_t e = add_static_lds(k_thin<LT, false, 4, kShortSingles<false>>, bytes);
  if (e == hipSuccess) e = add_static_lds(k_thin<LT, false, 4, 0>, bytes);
  if (e == hipSuccess) e = add_static_lds(k_thin<LT, false, 8, kShortPairs<LT, false>>, bytes);
  if (e == hipSuccess) e = add_static_lds(k_thin<LT, true, 4, kShortSingles<true>>, bytes);
  return e != hipSuccess ? e : add_static_lds(k_thin<LT, true, 8, kShortPairs<LT, true>>, bytes);
}

}  // namespace

hipError_t thin_static_lds(size_t *bytes) {
  const hipError_t e = static_lds_of<float>(bytes);
  return e != hipSuccess ? e : static_lds_of<uint16_t>(bytes);
}

uint32_t thin_lds(const Params &P, uint32_t stack_bytes) { return P.blob_dwords * 4 + kThinWaves * (kThinPark + stack_bytes); }
uint32_t thin_stack(uint32_t tile_sgs, uint32_t levels) { return levels * (tile_sgs == 1 ? kThinStack<4> : kThinStack<8>); }

hipError_t launch_thin(dq_dtype dtype, bool tree, const WalkPath *paths, const WalkShare *shares, const WalkGrid &W, const Params &P, hipStream_t s) {
  if (dtype == DQ_F32) return tree ? go_thin<float, true>(paths, shares, W, P, s) : go_thin<float, false>(paths, shares, W, P, s);
  return tree ? go_thin<uint16_t, true>(paths, shares, W, P, s) : go_thin<uint16_t, false>(paths, shares, W, P, s);
}

}  // namespace dq
