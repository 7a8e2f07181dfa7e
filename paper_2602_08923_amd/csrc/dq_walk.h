// Device code shared by the two kernels that carry a tile through all hops of a schedule (dq_walk.hip, dq_thin.hip).
#pragma once
#include "dq_codec.h"

namespace dq {
namespace {

// The lane's number, opaque to the compiler: what is derived from it is computed where it is used, once in many hops,
// and not held in registers around the loops (a spilled register's reload waits for the tile's loads in flight).
__device__ __forceinline__ uint32_t lane_here() {
  uint32_t lane = threadIdx.x & 63u;
  asm volatile("" : "+v"(lane));
  return lane;
}

template <bool B>
struct Is { static constexpr bool value = B; };

// Which share a wave takes (the order goes from narrow to wide).  Where no wave has more than a tile the wide ones go first, so that the blocks that are
// dispatched last, beside another on their CU or after it, have the narrow ones.  With more, a ring's four or five blocks of four waves per CU take
// shares from as many places of the order.  A recursive halving has two blocks of eight: there the i-th waves of all CUs take the i-th
// stretch of the shares, so that every CU has some of all widths, and CUs with a block more have the cheapest in it: the first shares, of two bits, or
// the last, if there are more raw tiles (over 16 in bf16, 385/376/4,981/3,570: 28.3 us; with the few 2-bit ones there 38.8, in path order 30.8).
// (The number of blocks is read with the other arguments: gridDim is a trip of its own, 0.2 us.)
template <bool TREE>
__device__ __forceinline__ uint32_t share_of(const Walk &W, uint32_t wave, uint32_t waves) {
  const uint32_t b = blockIdx.x;
  if (W.order == kReversed) return (W.blocks - 1 - b) * waves + wave;
  if (TREE && W.order) {
    const uint32_t cus = W.order, row = b / cus, rows = W.blocks / cus, rest = W.blocks - rows * cus;
    const uint32_t beside = W.raw_beside ? rows * cus * waves : 0, all = W.raw_beside ? 0 : rest * waves;
    return row < rows ? all + (row * waves + wave) * cus + b % cus : beside + wave * rest + b % cus;
  }
  return b * waves + wave;
}

// Worker whose entries are the i-th a chunk meets.
template <bool TREE>
__device__ __forceinline__ uint32_t leaf_of(const Walk &W, uint32_t chunk, uint32_t i) {
  if constexpr (TREE) {
    return chunk ^ (__brev(~i) >> (32u - W.log_n));
  } else {
    const uint32_t x = (W.chain ? 0u : chunk) + i;
    return min(x, x - W.n);
  }
}

// Where leaf i's message goes.  (A choice between two registers: as an array indexed at run time the path lived in scratch
// memory, 120 bytes of it per lane, which every wave of a ring wrote: 39 MB written and about as much read of 368 MB for 25 MB through a
// ring of eight, 74.6 us; 61.6 without.  A ring of fp32 tensors 115 -> 104, of 8,192 super-groups 23.3 -> 20.2.)
__device__ __forceinline__ uint8_t *message_of(const WalkPath &path, uint32_t i) { return i & 1u ? path.msg[1] : path.msg[0]; }

// The launch's tables (tensors, paths, shares) are read through the constant address space, as nothing in the kernel
// writes to them: scalar loads into scalar registers.  As global loads they are vector loads, and the one of the next
// tensor's address waits in every hop for everything the wave has in flight.
template <typename T>
__device__ __forceinline__ T table_entry(const T *table, uint32_t i) {
  constexpr uint32_t kWords = sizeof(T) / 4;
  typedef __attribute__((address_space(4))) const uint32_t constant_u32;
  constant_u32 *p = (constant_u32 *)(uintptr_t)table + (uint64_t)i * kWords;
  struct Words { uint32_t w[kWords]; } words;
#pragma unroll
  for (uint32_t k = 0; k < kWords; ++k) words.w[k] = p[k];
  return __builtin_bit_cast(T, words);
}

// The tables from dword `first` on, and the reciprocals in front, to their places in LDS, in one trip to memory: whatever widths the
// chunks have.  (Range by range, those of widths that some chunk has, it was a trip each: 8 workers' ring of 8,192 super-groups 19.2 us
// instead of 17.4, 4 workers' fp32 ring of 4,096 9.1 instead of 8.3, 25 MB through a ring of eight 53 instead of 52.)
__device__ __forceinline__ void copy_tables(uint32_t *lds, const uint32_t *blob, const Params &P, uint32_t first) {
  constexpr uint32_t kTogether = 4, kRec = kOffDec2 / 4;  // 16-byte words per thread requested at once; of the reciprocals
  const uint32_t words = P.blob_dwords / 4, lo = first / 4 + threadIdx.x;
  uint4 rec, part[kTogether];
  if (threadIdx.x < kRec) rec = gld16(&blob[threadIdx.x * 4]);
#pragma unroll
  for (uint32_t k = 0; k < kTogether; ++k) part[k] = gld16(&blob[min(lo + k * blockDim.x, words - 1) * 4]);
  if (threadIdx.x < kRec) *reinterpret_cast<uint4 *>(&lds[threadIdx.x * 4]) = rec;
#pragma unroll
  for (uint32_t k = 0; k < kTogether; ++k) *reinterpret_cast<uint4 *>(&lds[min(lo + k * blockDim.x, words - 1) * 4]) = part[k];
  for (uint32_t i = lo + kTogether * blockDim.x; i < words; i += blockDim.x) *reinterpret_cast<uint4 *>(&lds[i * 4]) = gld16(&blob[i * 4]);
}

}  // namespace
}  // namespace dq
