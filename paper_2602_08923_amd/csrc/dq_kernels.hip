// DynamiQ hot-path kernels for gfx950: compress, decompress-accumulate-recompress (DAR)
// and decompress(+accumulate)  (paper Section 3.3 for the quantizer, Section 3.4 "Fused
// kernels" / Section 4 for which node runs which kernel).
//
// Mapping.  One lane owns one group of 16 entries; a DPP row of 16 lanes is one super-group
// (SG), so the group maximum is in-lane and the SG maximum is four row-rotate DPP steps; a
// wave64 processes 4 SGs per tile and a run of consecutive tiles per launch.  Codes travel as
// one 32/64/128-bit access per lane (2/4/8-bit widths), the local slice as 128-bit accesses.
// Level tables live in LDS from byte 0 on:
//   dec[byte]      the 8/b signed levels (+-T[r]) one byte of packed codes holds  -> decode
//   lut[q]         {T[rc+1], address of rc's pair} for q = round(x' * 2^m): rc is the level index
//                  at the lower edge of the bin, and bins are narrower than any gap, so the
//                  level at or below x' is rc or rc+1 -- one compare settles it
//   tab[rc]        the entries {T[r], D[r], T[r+1], code} of r = rc+1 and r = rc   -> rounding
// The stochastic rounding follows the division-free form  T + u*D < x'  with
// u = (pi + gamma)/n built from one Philox byte per entry (Section 3.3 "Correlated rounding").
// The per-SG random numbers (group-scale bytes, shared permutation) of up to 8 tiles are
// drawn by ONE wave-wide Philox call (each lane a different counter) and parked in LDS; a block
// with few tiles draws for all its waves at once.  A chunk may end in a run of 16-bit
// super-groups (raw bf16 values, Section 3.2): those tiles only add and round.
// Three options ride on the job: per-super-group means taken off the local entries in fp32 where
// they enter (Section 3.1), the local super-groups gathered from the original tensor through an
// index (the reorder of Section 3.5 done by addressing), and, for decompress, every super-group
// stored to its original place with the mean added back (the restore of Section 3.4, fused in).
//
// All arithmetic that decides a code is IEEE binary32 with explicit fused multiply-adds
// only where written (this file is compiled with -ffp-contract=off and correctly rounded
// division), so the results do not depend on the launch shape.
#include "dq_bounds.h"
#include "dq_codec.h"

namespace dq {
namespace {

// What one lane fetches for one tile of compress / DAR: raw words only.
template <int B, Kind KIND, typename LT>
struct Fetch {
  uint4 loc[sizeof(LT) == 4 ? 4 : 2];  // the lane's 16 local entries
  float mu;                            // the mean to take off them (if the job has means)
  uint32_t cw[B / 2];                  // DAR: their incoming codes
  uint32_t rg_in, sf_in;               // DAR: incoming group scale (u8) and SG scale (bf16 pattern)
};

template <int B, Kind KIND, typename LT, bool MU>
__device__ __forceinline__ Fetch<B, KIND, LT> fetch(const Job &job, const TilePos pos) {
  const TileBase<B> tb(job, pos);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t rowc = min(lane >> 4, tb.last_row);  // idle rows redo the last SG and store nothing
  const uint32_t lg = rowc * 16 + (lane & 15u);       // group index inside the tile
  Fetch<B, KIND, LT> f;
  if constexpr (KIND == kDar) {  // the incoming words first: with job.src the local loads wait for an index
    const uint8_t *cp = job.in + tb.code_off + lg * (2 * B);
    load_codes<B>(cp, f.cw);
    f.rg_in = gld<uint8_t>(job.in + tb.gs_off + lg);
    f.sf_in = gld<uint16_t>(job.in + tb.sf_off + rowc * 2);
  }
  if constexpr (MU) f.mu = local_mean(job, tb.first_entry, rowc);
  else f.mu = 0.0f;
  load_local<LT>(job, tb.first_entry, rowc, lane & 15u, f.loc);
  return f;
}

// A tile's encoded output.
template <int B>
struct Encoded {
  uint32_t ow[Width<B>::words], rg, sfb;
};

// One wave tile of compress / DAR after the fetch: up to 4 super-groups of width B.
//   stage    : LDS byte address of this tile's 8 parked draws (row r: [2r] = permutation
//              stream, [2r+1] = group-scale stream), 16 bytes each
//   ahead    : called once the tile's loaded data is used up, before the per-entry work: from there the
//              next tile's loads have the longest time to arrive without holding two tiles' data at once
template <int B, Kind KIND, typename LT, bool MU, typename Ahead>
__device__ __forceinline__ Encoded<B> compute(const Job &job, const Params &P, const Vec &V, uint32_t stage,
                                              const TilePos pos, const Fetch<B, KIND, LT> &f, Ahead ahead) {
  static_assert(KIND != kDecompress, "decompress has its own tile function");
  const TileBase<B> tb(job, pos);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t g = lane & 15u;
  const uint32_t rowc = min(lane >> 4, tb.last_row);

  // random numbers first: they need nothing from memory, so a wave that still waits for its tile has them done;
  // the empty asm ties the tile's first use to them, or the scheduler would sink them below the wait
  const Draws d = draw_group(P, (tb.G0 + rowc) * 16 + g, job.rank, lds_ld1(stage + rowc * 32),
                             lds_ld1(stage + rowc * 32 + 16 + (g >> 2) * 4), g);
  uint4 loc[sizeof(LT) == 4 ? 4 : 2];
#pragma unroll
  for (int i = 0; i < (sizeof(LT) == 4 ? 4 : 2); ++i) loc[i] = f.loc[i];
  asm volatile("" : "+v"(loc[0].x) : "v"(d.gam.x), "v"(d.gam.y), "v"(d.gam.z), "v"(d.gam.w), "v"(d.o_pi), "v"(d.us));
  float v[16];
  widen_local<LT>(loc, v);
  if constexpr (MU) {
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = v[k] - f.mu;
  }
  if constexpr (KIND == kDar) {
    // decode: sf_G = r_G * (sf_SG / 255); estimate = +-T[r] * sf_G, accumulated by one fma
    const float sfg = (float)f.rg_in * sf_over_255(f.sf_in, kRec0);
    each_level<B, HopTables>(f.cw, [&](int k, float t) { v[k] = __builtin_fmaf(t, sfg, v[k]); });
  }
  const Scales s = scale_group(v, d.us, kRec0);
  ahead();
  Encoded<B> e;
  e.rg = s.rg;
  e.sfb = s.sfb;
  quantize<B, true, false>(v, s.inv, d.gam, d.o_pi, V, e.ow);
  return e;
}
template <int B>
__device__ __forceinline__ void put(const Job &job, const TilePos pos, const Encoded<B> &e) {
  const TileBase<B> tb(job, pos);
  const uint32_t lane = threadIdx.x & 63u, rowc = min(lane >> 4, tb.last_row);
  store_codes<B>(static_cast<uint8_t *>(job.out), tb, rowc * 16 + (lane & 15u), rowc, e.ow, e.rg, e.sfb);
}

// One wave tile of decompress(+accumulate).  Lanes fetch and decode like the DAR tile (a lane
// owns a group of 16 entries, few wide loads), then the 4 KB of fp32 results are transposed
// through a per-wave LDS area so that every store instruction writes 1 KB of contiguous memory.
//   xpose : LDS byte address of this wave's 4 KB transpose area
template <int B, typename LT>
__device__ __forceinline__ void tile_da(const Job &job, const Params &P, uint32_t xpose,
                                        const TilePos pos) {
  using W = Width<B>;
  constexpr bool kHasLocal = !__is_same(LT, NoLocal);
  const TileBase<B> tb(job, pos);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t rowc = min(lane >> 4, tb.last_row);
  const uint32_t lg = rowc * 16 + (lane & 15u);
  constexpr uint32_t rec0 = kRec0;

  // the incoming words first: with job.src the local loads wait for an index
  uint32_t cw[W::words];
  const uint8_t *cp = job.in + tb.code_off + lg * (2 * B);
  load_codes<B>(cp, cw);
  const uint32_t rg_in = gld<uint8_t>(job.in + tb.gs_off + lg);
  const uint32_t sf_in = gld<uint16_t>(job.in + tb.sf_off + rowc * 2);
  float v[16];
  float mu = 0.0f;
  if constexpr (kHasLocal) {
    uint4 loc[sizeof(LT) == 4 ? 4 : 2];
    mu = local_mean(job, tb.first_entry, rowc);
    load_local<LT>(job, tb.first_entry, rowc, lane & 15u, loc);
    widen_local<LT>(loc, v);
  }
  const float sfg = (float)rg_in * sf_over_255(sf_in, rec0);
  // after every load of the tile has been issued: the branch would otherwise hold the later loads back
  if constexpr (kHasLocal) subtract_mean(job, mu, v);
  each_level<B, HopTables>(cw, [&](int k, float t) {
    if constexpr (kHasLocal) v[k] = __builtin_fmaf(t, sfg, v[k]);
    else v[k] = t * sfg;
  });
  store_tile_f32(job, P, v, xpose, tb.first_entry, tb.last_row);
}

// Decompress-accumulate over `len` consecutive tiles of width B: the tile's operands are those of a DAR
// hop (fetch<.., kDar, ..>); the next tile is requested before the current one's transpose and stores.
template <int B, typename LT, bool MU>
__device__ __forceinline__ void run_tiles_da(const Job &job, const Params &P, uint32_t xpose, TilePos pos, uint32_t len, uint32_t step) {
  constexpr uint32_t rec0 = kRec0;
  Fetch<B, kDar, LT> f = fetch<B, kDar, LT, MU>(job, pos);
  for (uint32_t i = 0; i < len; ++i) {
    const TileBase<B> tb(job, pos);
    float v[16];
    widen_local<LT>(f.loc, v);
    if constexpr (MU) {
#pragma unroll
      for (int k = 0; k < 16; ++k) v[k] = v[k] - f.mu;
    }
    const float sfg = (float)f.rg_in * sf_over_255(f.sf_in, rec0);
    each_level<B, HopTables>(f.cw, [&](int k, float t) { v[k] = __builtin_fmaf(t, sfg, v[k]); });
    TilePos pos_next = pos;
    pos_next.tile_first += step;
    Fetch<B, kDar, LT> next;
    if (i + 1 < len) next = fetch<B, kDar, LT, MU>(job, pos_next);
    store_tile_f32(job, P, v, xpose, tb.first_entry, tb.last_row);
    f = next;
    pos = pos_next;
  }
}

// One wave tile of uncompressed (16-bit) super-groups: the packed values are raw bf16
// ("16 bits corresponds to uncompressed values", Section 3.2).  Compress rounds the local entries
// to bf16 (nearest even); a DAR hop adds the local entry to the widened incoming value in fp32
// and rounds the sum back; decompress widens (and adds).  No scales, no random numbers.
template <Kind KIND, typename LT>
__device__ __forceinline__ void tile16(const Job &job, const Params &P, uint32_t xpose, const TilePos pos) {
  constexpr bool kHasLocal = !__is_same(LT, NoLocal);
  const TileBase<16> tb(job, pos);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t row = lane >> 4;
  const uint32_t rowc = min(row, tb.last_row);
  const uint32_t lg = rowc * 16 + (lane & 15u);
  uint4 in[2];
  if constexpr (KIND != kCompress) {  // the incoming words first: with job.src the local loads wait for an index
    const uint4 *p = reinterpret_cast<const uint4 *>(job.in + tb.code_off) + lg * 2;
    in[0] = gld16(p);
    in[1] = gld16(p + 1);
  }
  float v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = 0.0f;
  float mu = 0.0f;
  if constexpr (kHasLocal) {
    uint4 loc[sizeof(LT) == 4 ? 4 : 2];
    mu = local_mean(job, tb.first_entry, rowc);
    load_local<LT>(job, tb.first_entry, rowc, lane & 15u, loc);
    widen_local<LT>(loc, v);
  }
  if constexpr (kHasLocal) subtract_mean(job, mu, v);  // after every load of the tile has been issued
  if constexpr (KIND != kCompress) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint4 x = in[i];
      const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[8 * i + 2 * j] = u2f(w[j] << 16) + v[8 * i + 2 * j];
        v[8 * i + 2 * j + 1] = u2f(w[j] & 0xFFFF0000u) + v[8 * i + 2 * j + 1];
      }
    }
  }
  if constexpr (KIND == kDecompress) {
    store_tile_f32(job, P, v, xpose, tb.first_entry, tb.last_row);
  } else if (row <= tb.last_row) {
    uint8_t *dst = static_cast<uint8_t *>(job.out) + tb.code_off + lg * 32;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      gst<u32x4>(dst + 16 * i, u32x4{bf16_rne_pair(v[8 * i], v[8 * i + 1]), bf16_rne_pair(v[8 * i + 2], v[8 * i + 3]),
                                     bf16_rne_pair(v[8 * i + 4], v[8 * i + 5]), bf16_rne_pair(v[8 * i + 6], v[8 * i + 7])});
  }
}

// `len` consecutive tiles of width B starting at `pos` (their parked draws 128 bytes apart).
template <int B, Kind KIND, typename LT, bool MU>
__device__ __forceinline__ void run_tiles(const Job &job, const Params &P, const Vec &V, uint32_t stage, uint32_t stage_step,
                                          TilePos pos, uint32_t len, uint32_t step) {
  // The next tile of the run is requested from inside the current one (see compute's `ahead`): with five waves
  // per SIMD a wave's own wait for its tile is no longer covered by the others (measured: 3-7 % on the 25 MB
  // and the 100-bucket configurations, nothing on the largest launches).
  Fetch<B, KIND, LT> f = fetch<B, KIND, LT, MU>(job, pos);
  for (uint32_t i = 0; i < len; ++i) {
    Fetch<B, KIND, LT> next;  // nothing where there is no next tile, not f: see walk_tiles
    TilePos pos_next = pos;
    pos_next.tile_first += step;
    const Encoded<B> e = compute<B, KIND, LT, MU>(job, P, V, stage + i * stage_step, pos, f, [&] {
      if (i + 1 < len) next = fetch<B, KIND, LT, MU>(job, pos_next);
    });
    put<B>(job, pos, e);
    f = next;
    pos = pos_next;
  }
}

// Per-SG draws of nb <= 8 tiles, tile(0) to tile(nb - 1), made by one wave-wide
// Philox call and parked at `area` (128 bytes per tile: row r at [32r] this worker's slot of the
// shared permutation, at [32r+16] the worker's group-scale stream).  Lane l draws for tile l/8, row (l%8)/2.
template <typename F>
__device__ __forceinline__ void park_draws(const Job &job, const Params &P, uint32_t nb, uint32_t area, F tile) {
  const uint32_t lane = threadIdx.x & 63u;
  const TilePos p = locate(job, tile(min(lane >> 3, nb - 1)));
  const uint32_t sgw = min(p.tile_first + ((lane >> 1) & 3u), p.n_seg - 1);
  const uint64_t G = job.first_sg + p.seg_first + sgw;
  const uint32_t c3 = (lane & 1u) ? ((1u << 16) | (job.rank & 0xFFFFu)) : ((2u << 16) | 0xFFFFu);
  const U4 d = philox4x32_10((uint32_t)G, (uint32_t)(G >> 32), P.round, c3, P.key0, P.key1);
  // even lanes hold the shared draw: they park the slot it gives this job's worker in word 0
  const uint32_t w0 = (lane & 1u) ? d.x : perm_slot(d, P, job.rank);
  lds_st4(area + lane * 16, u32x4{w0, d.y, d.z, d.w});
}

// A wave's tiles: first, first + stride, ... (n of them).
struct Tiles {
  uint32_t first, stride, n;
};
// How many of them, from the one at `p` on, are of its width, at most n
__device__ __forceinline__ uint32_t same_width(const TilePos &p, uint32_t stride, uint32_t n) {
  const uint32_t left = (p.n_seg - p.tile_first + kWaveSGs - 1) / kWaveSGs;  // tiles to the segment's end
  return min(n, (left + stride - 1) / stride);
}

// Tiles T of the job, the draws of the first parked at `area`, the others' stage_step bytes apart.
template <Kind KIND, typename LT>
__device__ __forceinline__ void run_range(const Job &job, const Params &P, const Vec &V, uint32_t area, uint32_t stage_step, Tiles T) {
  const uint32_t step = T.stride * kWaveSGs;
  while (T.n) {
    const TilePos p = locate(job, T.first);
    const uint32_t len = same_width(p, T.stride, T.n);
    // two builds of the tile loop, with and without means: a branch on job.mu inside a tile makes the
    // path without means wait, at the branch's join, for the loads issued before it
    if (job.mu) {
      if (p.wi == 0) run_tiles<2, KIND, LT, true>(job, P, V, area, stage_step, p, len, step);
      else if (p.wi == 1) run_tiles<4, KIND, LT, true>(job, P, V, area, stage_step, p, len, step);
      else if (p.wi == 2) run_tiles<8, KIND, LT, true>(job, P, V, area, stage_step, p, len, step);
    } else {
      if (p.wi == 0) run_tiles<2, KIND, LT, false>(job, P, V, area, stage_step, p, len, step);
      else if (p.wi == 1) run_tiles<4, KIND, LT, false>(job, P, V, area, stage_step, p, len, step);
      else if (p.wi == 2) run_tiles<8, KIND, LT, false>(job, P, V, area, stage_step, p, len, step);
    }
    if (p.wi > 2) {
      TilePos q = p;
      for (uint32_t i = 0; i < len; ++i, q.tile_first += step) tile16<KIND, LT>(job, P, 0u, q);
    }
    T.first += len * T.stride;
    T.n -= len;
    area += len * stage_step;
  }
}

// Decompress(+accumulate) over the tiles T of the job: tile by tile without a local slice, in
// runs of one width (the next tile requested ahead) with one.
template <typename LT>
__device__ __forceinline__ void da_range(const Job &job, const Params &P, uint32_t xpose, Tiles T) {
  if constexpr (__is_same(LT, NoLocal)) {
    for (; T.n; --T.n, T.first += T.stride) {
      const TilePos p = locate(job, T.first);
      if (p.wi == 0) tile_da<2, LT>(job, P, xpose, p);
      else if (p.wi == 1) tile_da<4, LT>(job, P, xpose, p);
      else if (p.wi == 2) tile_da<8, LT>(job, P, xpose, p);
      else tile16<kDecompress, LT>(job, P, xpose, p);
    }
  } else {
    const uint32_t step = T.stride * kWaveSGs;
    while (T.n) {  // runs of one width, as in run_range
      const TilePos p = locate(job, T.first);
      const uint32_t len = same_width(p, T.stride, T.n);
      if (job.mu) {
        if (p.wi == 0) run_tiles_da<2, LT, true>(job, P, xpose, p, len, step);
        else if (p.wi == 1) run_tiles_da<4, LT, true>(job, P, xpose, p, len, step);
        else if (p.wi == 2) run_tiles_da<8, LT, true>(job, P, xpose, p, len, step);
      } else {
        if (p.wi == 0) run_tiles_da<2, LT, false>(job, P, xpose, p, len, step);
        else if (p.wi == 1) run_tiles_da<4, LT, false>(job, P, xpose, p, len, step);
        else if (p.wi == 2) run_tiles_da<8, LT, false>(job, P, xpose, p, len, step);
      }
      if (p.wi > 2) {
        TilePos q = p;
        for (uint32_t i = 0; i < len; ++i, q.tile_first += step) tile16<kDecompress, LT>(job, P, xpose, q);
      }
      T.first += len * T.stride;
      T.n -= len;
    }
  }
}

// The tables on their way into a block's LDS: 16-byte words requested together before anything else is, put down after the draws are
// made.  All the tables, whatever widths the block meets (decompress: what lies before the search tables); a level set with larger ones
// takes further trips.  Only the tables of the widths that a block met, a trip for each of their six
// ranges beyond its first 4 KB, took longer at every size, us per call, bf16, 2- to 8-bit super-groups, ranges -> together:
//                 12,288         20,000         40,000          100,000
//   hop           6.9 -> 6.2     8.3 -> 7.2     11.5 -> 10.3    20.2 -> 18.8
//   compress      6.7 -> 5.9     7.9 -> 6.8     10.3 -> 9.1     17.9 -> 16.8
//   sink          5.9 -> 5.1     6.8 -> 6.0     10.7 -> 9.7     27.8 -> 27.0
// A ring of eight step by step: 384 super-groups 4.9 -> 4.3 per step, 4,096 5.75 -> 4.85, 48,832 13.8 -> 12.5.
template <Kind KIND>
struct BlockTables {
  // Words per thread: the default sets' 21 KB; decompress's 12.5 KB in two trips, as with all four words at once the restore of 488,282
  // gathered super-groups took 192 us instead of 186.5, where it was 187.4 range by range (and smaller ones the same).
  static constexpr uint32_t kTogether = KIND == kDecompress ? 2 : 6;
  uint4 part[kTogether];
  uint32_t words;
  __device__ __forceinline__ explicit BlockTables(const Params &P) : words(KIND == kDecompress ? kOffLut4 / 4 : P.blob_dwords / 4) {
#pragma unroll
    for (uint32_t k = 0; k < kTogether; ++k) part[k] = gld16(&P.blob[min(threadIdx.x + k * kBlockThreads, words - 1) * 4]);
  }
  __device__ __forceinline__ void put_down(uint32_t *lds, const Params &P) const {
#pragma unroll
    for (uint32_t k = 0; k < kTogether; ++k)
      *reinterpret_cast<uint4 *>(&lds[min(threadIdx.x + k * kBlockThreads, words - 1) * 4]) = part[k];
    for (uint32_t i = threadIdx.x + kTogether * kBlockThreads; i < words; i += kBlockThreads)
      *reinterpret_cast<uint4 *>(&lds[i * 4]) = gld16(&P.blob[i * 4]);
  }
};

// The job's tiles go round the waves of the grid row (4 * gridDim.x waves): wave w takes w, w + W, w + 2W, ...  What the
// waves read and write at one time is then one window of each stream, in the order of its addresses, and not W places in
// it; and every wave meets the widths in about the same shares, so that they end together (2-bit tiles are cheaper).  The
// launcher sizes the grid to what the GPU holds at once, so a wave lives for the whole launch and the table copy is paid
// once.  Measured against shares of consecutive tiles: the sink of 125 M entries 191 -> 187.5 us, a hop of as many the
// same with half the blocks that consecutive shares needed to even the widths out, 6400 super-groups' compress 5.6 -> 5.4 us.
template <Kind KIND, typename LT>
__device__ __forceinline__ void run_job(const Job &job, const Params &P) {
  extern __shared__ uint4 lds_raw[];
  uint32_t *lds = reinterpret_cast<uint32_t *>(lds_raw);
  const uint32_t n0 = job.n_sg[0], n1 = job.n_sg[1], n2 = job.n_sg[2];
  const uint32_t t0 = (n0 + kWaveSGs - 1) / kWaveSGs, t1 = (n1 + kWaveSGs - 1) / kWaveSGs,
                 t2 = (n2 + kWaveSGs - 1) / kWaveSGs, t3 = (job.n_sg[3] + kWaveSGs - 1) / kWaveSGs;
  const uint32_t total = t0 + t1 + t2 + t3;
  const uint32_t n_waves = gridDim.x * kBlockWaves, q = total / n_waves, r = total - q * n_waves;
  const uint32_t bw = blockIdx.x * kBlockWaves;
  if (q == 0 && bw >= r) return;
  constexpr uint32_t lds0 = kLds0;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t mine = q + (bw + wave < r ? 1u : 0u);
  // parking area for per-SG draws: 1 KB (8 tiles) per wave, the four areas contiguous
  // (decompress needs no search tables: its blocks leave them out and are small enough for six per CU)
  const uint32_t park0 = lds0 + (KIND == kDecompress ? kOffLut4 : P.blob_dwords) * 4;
  // a block with at most 32 tiles makes all its draws up front, 8 tiles per wave-wide call,
  // instead of one call per wave (waves of a small job hold only a tile or two each): the block's tile k is wave k % 4's
  const uint32_t in_block = q * kBlockWaves + min(r - min(r, bw), (uint32_t)kBlockWaves);
  const bool block_draws = KIND != kDecompress && in_block <= 8u * kBlockWaves;

  BlockTables<KIND> tables(P);
  if constexpr (KIND != kDecompress) {
    if (block_draws && 8u * wave < in_block)
      park_draws(job, P, min(8u, in_block - 8u * wave), park0 + wave * 1024, [&](uint32_t j) {
        const uint32_t k = 8u * wave + j;
        return (k / kBlockWaves) * n_waves + bw + k % kBlockWaves;
      });
  }
  tables.put_down(lds, P);
  __syncthreads();

  [[maybe_unused]] const uint32_t area = park0 + wave * 1024;     // compress, DAR: this wave's parked draws
  [[maybe_unused]] const uint32_t xpose = park0 + wave * (64 * 64);  // decompress: its transpose area, 64 lanes x 64 bytes
  const Vec V(P);
  Tiles T = {bw + wave, n_waves, mine};
  if constexpr (KIND == kDecompress) {
    da_range<LT>(job, P, xpose, T);
  } else if (block_draws) {
    __builtin_amdgcn_wave_barrier();
    run_range<KIND, LT>(job, P, V, park0 + wave * 128, kBlockWaves * 128, T);
  } else {
    for (uint32_t left = mine; left; left -= T.n, T.first += T.n * n_waves) {
      T.n = min((uint32_t)kBatch, left);
      park_draws(job, P, T.n, area, [&](uint32_t j) { return T.first + j * n_waves; });
      __builtin_amdgcn_wave_barrier();
      run_range<KIND, LT>(job, P, V, area, 128u, T);
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// Five blocks of four waves are resident per CU (the launcher's grid): at most 96 vector registers (they use 73 to 95).
template <Kind KIND, typename LT>
__global__ __launch_bounds__(kBlockThreads) void k_one(Job job, Params P) {
  if (P.guard && gld<uint32_t>(P.guard) == P.guard_call) return;
  run_job<KIND, LT>(job, P);
}
template <Kind KIND, typename LT>
__global__ __launch_bounds__(kBlockThreads) void k_batch(const Job *jobs, Params P) {
  const Job job = jobs[blockIdx.y];
  run_job<KIND, LT>(job, P);
}
// Launches of thousands of jobs of at most kBatch tiles each (a replay of thousands of simulated workers:
// a tile or two per chunk): one job per WAVE, so that a block's table copy and its place on a CU serve
// four jobs instead of one wave's worth of one.
template <Kind KIND, typename LT>
__global__ __launch_bounds__(kBlockThreads) void k_batch_small(const Job *jobs, uint32_t n_jobs, Params P) {
  extern __shared__ uint4 lds_raw[];
  uint32_t *lds = reinterpret_cast<uint32_t *>(lds_raw);
  BlockTables<KIND>(P).put_down(lds, P);
  __syncthreads();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t j = __builtin_amdgcn_readfirstlane(blockIdx.x * kBlockWaves + wave);
  if (j >= n_jobs) return;
  const Job job = jobs[j];
  const uint32_t tiles = (job.n_sg[0] + kWaveSGs - 1) / kWaveSGs + (job.n_sg[1] + kWaveSGs - 1) / kWaveSGs +
                         (job.n_sg[2] + kWaveSGs - 1) / kWaveSGs + (job.n_sg[3] + kWaveSGs - 1) / kWaveSGs;
  if (tiles == 0) return;
  const uint32_t park0 = kLds0 + (KIND == kDecompress ? kOffLut4 : P.blob_dwords) * 4;
  if constexpr (KIND == kDecompress) {
    da_range<LT>(job, P, park0 + wave * (64 * 64), Tiles{0u, 1u, tiles});
  } else {
    const Vec V(P);
    const uint32_t area = park0 + wave * 1024;
    park_draws(job, P, tiles, area, [](uint32_t j) { return j; });
    __builtin_amdgcn_wave_barrier();
    run_range<KIND, LT>(job, P, V, area, 128u, Tiles{0u, 1u, tiles});
  }
}

// Copy of a packed block in 16-byte words; the bytes from `valid` on (the padding at the block's end,
// which the codec kernels never write) are put down as zero.
__global__ void __launch_bounds__(256) k_wire_copy(const uint4 *src, uint4 *dst, uint64_t words, uint64_t valid) {
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (uint64_t)gridDim.x * 256) {
    uint4 w = src[i];
    if ((i + 1) * 16 > valid) {
      uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint64_t at = i * 16 + 4 * k;  // first byte of this dword
        const uint32_t keep = at >= valid ? 0u : (valid - at >= 4 ? 0xFFFFFFFFu : (1u << (8 * (uint32_t)(valid - at))) - 1u);
        x[k] &= keep;
      }
      w = uint4{x[0], x[1], x[2], x[3]};
    }
    dst[i] = w;
  }
}

uint32_t job_tiles(const Job &j) {
  return (j.n_sg[0] + kWaveSGs - 1) / kWaveSGs + (j.n_sg[1] + kWaveSGs - 1) / kWaveSGs +
         (j.n_sg[2] + kWaveSGs - 1) / kWaveSGs + (j.n_sg[3] + kWaveSGs - 1) / kWaveSGs;
}

// Grid shape: `grid_blocks` (what the GPU holds at once: CUs x blocks per CU, fixed when the
// context is made) shared between the jobs of the launch (one block holds 4 waves; a wave
// then walks its share of the job's tiles).
uint32_t blocks_per_job(uint32_t max_tiles, uint32_t n_jobs, uint32_t grid_blocks) {
  uint32_t blocks = (grid_blocks + n_jobs - 1) / n_jobs;
  const uint32_t needed = (max_tiles + kBlockWaves - 1) / kBlockWaves;
  if (blocks > needed) blocks = needed;
  return blocks < 1 ? 1 : blocks;
}

// blob + per-wave area: 1 KB of parked draws (compress, DAR) or 4 KB for the transpose (decompress)
size_t lds_bytes(const Params &p, Kind kind) {
  return kind == kDecompress ? (size_t)kOffLut4 * 4 + kBlockWaves * 64 * 64 : (size_t)p.blob_dwords * 4 + kBlockWaves * 64 * 16;
}

template <Kind KIND, typename LT>
hipError_t go_one(const Job &job, const Params &p, uint32_t grid_blocks, hipStream_t s) {
  const uint32_t tiles = job_tiles(job);
  const uint32_t blocks = blocks_per_job(tiles, 1, grid_blocks);
  hipLaunchKernelGGL((k_one<KIND, LT>), dim3(blocks), dim3(kBlockThreads), lds_bytes(p, KIND), s, job, p);
  return hipGetLastError();
}
template <Kind KIND, typename LT>
hipError_t go_batch(const Job *jobs, uint32_t n_jobs, uint32_t max_tiles, Params p,
                    uint32_t grid_blocks, hipStream_t s) {
  if (n_jobs == 0 || max_tiles == 0) return hipSuccess;
  if (max_tiles <= (uint32_t)kBatch && n_jobs >= grid_blocks) {  // so many small jobs that a block per job would queue up
    hipLaunchKernelGGL((k_batch_small<KIND, LT>), dim3((n_jobs + kBlockWaves - 1) / kBlockWaves), dim3(kBlockThreads),
                       lds_bytes(p, KIND), s, jobs, n_jobs, p);
    return hipGetLastError();
  }
  const uint32_t blocks = blocks_per_job(max_tiles, n_jobs, grid_blocks);
  // the grid's y dimension (one row per job) holds at most 65,535 rows: more jobs take more launches
  for (uint32_t first = 0; first < n_jobs; first += kMaxGridRows) {
    const uint32_t rows = n_jobs - first < kMaxGridRows ? n_jobs - first : kMaxGridRows;
    hipLaunchKernelGGL((k_batch<KIND, LT>), dim3(blocks, rows), dim3(kBlockThreads), lds_bytes(p, KIND), s, jobs + first, p);
  }
  return hipGetLastError();
}

}  // namespace

// LT for a local of `dtype`, gathered through job.src or not
#define DQ_DISPATCH_LOCAL(CALL, KINDV)                                                        \
  (gather ? (f32 ? CALL<KINDV, Gathered<float>> ARGS : CALL<KINDV, Gathered<uint16_t>> ARGS) \
          : (f32 ? CALL<KINDV, float> ARGS : CALL<KINDV, uint16_t> ARGS))

hipError_t launch_one(Kind kind, dq_dtype dtype, bool has_local, const Job &job, const Params &params, uint32_t n_cu, uint32_t grid_blocks,
                      hipStream_t s) {
  if (job_tiles(job) == 0) return hipSuccess;
  Params p = params;
  if (takes_few(kind, job, p, n_cu)) return launch_few(kind, dtype, has_local, job, p, s);
  Guard guard;
  const hipError_t armed = armed_guard(s, &guard);
  if (armed != hipSuccess) return armed;
  p.guard = guard.word;
  p.guard_call = guard.call;
  const bool f32 = dtype == DQ_F32, gather = job.src != nullptr;
#define ARGS (job, p, grid_blocks, s)
  switch (kind) {
    case kCompress: return DQ_DISPATCH_LOCAL(go_one, kCompress);
    case kDar: return DQ_DISPATCH_LOCAL(go_one, kDar);
    default:
      if (!has_local) return go_one<kDecompress, NoLocal>(job, p, grid_blocks, s);
      return DQ_DISPATCH_LOCAL(go_one, kDecompress);
  }
#undef ARGS
}

hipError_t launch_batch(Kind kind, dq_dtype dtype, bool has_local, bool gather, const Job *jobs, uint32_t n_jobs,
                        uint32_t max_tiles, const Params &p, uint32_t grid_blocks, hipStream_t s) {
  const bool f32 = dtype == DQ_F32;
#define ARGS (jobs, n_jobs, max_tiles, p, grid_blocks, s)
  switch (kind) {
    case kCompress: return DQ_DISPATCH_LOCAL(go_batch, kCompress);
    case kDar: return DQ_DISPATCH_LOCAL(go_batch, kDar);
    default:
      if (!has_local) return go_batch<kDecompress, NoLocal>(jobs, n_jobs, max_tiles, p, grid_blocks, s);
      return DQ_DISPATCH_LOCAL(go_batch, kDecompress);
  }
#undef ARGS
}
#undef DQ_DISPATCH_LOCAL

namespace {
template <Kind KIND, typename LT>
hipError_t add_static_lds_of(size_t *bytes) {
  hipError_t e = add_static_lds(k_one<KIND, LT>, bytes);
  if (e == hipSuccess) e = add_static_lds(k_batch<KIND, LT>, bytes);
  return e != hipSuccess ? e : add_static_lds(k_batch_small<KIND, LT>, bytes);
}
}  // namespace

hipError_t static_lds_bytes(size_t *bytes) {
  *bytes = 0;
  hipError_t e = add_static_lds_of<kDecompress, NoLocal>(bytes);
#define DQ_ONE_KIND(KINDV)                                                             \
  if (e == hipSuccess) e = add_static_lds_of<KINDV, float>(bytes);                     \
  if (e == hipSuccess) e = add_static_lds_of<KINDV, uint16_t>(bytes);                  \
  if (e == hipSuccess) e = add_static_lds_of<KINDV, Gathered<float>>(bytes);           \
  if (e == hipSuccess) e = add_static_lds_of<KINDV, Gathered<uint16_t>>(bytes);
  DQ_ONE_KIND(kCompress)
  DQ_ONE_KIND(kDar)
  DQ_ONE_KIND(kDecompress)
#undef DQ_ONE_KIND
  if (e == hipSuccess) e = few_static_lds(bytes);
  if (e == hipSuccess) e = walk_static_lds(bytes);
  return e != hipSuccess ? e : thin_static_lds(bytes);
}

hipError_t wire_copy(void *dst, const void *src, size_t bytes, size_t valid, hipStream_t s) {
  const uint64_t words = bytes / 16;
  if (words == 0) return hipSuccess;
  const uint64_t want = (words + 1023) / 1024;  // four words per thread
  const uint32_t blocks = (uint32_t)(want < 2048 ? want : 2048);
  hipLaunchKernelGGL(k_wire_copy, dim3(blocks), dim3(256), 0, s, static_cast<const uint4 *>(src), static_cast<uint4 *>(dst),
                     words, (uint64_t)valid);
  return hipGetLastError();
}

}  // namespace dq
