// Internal declarations shared by the HIP translation units of libdq (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <vector>

#include "dq.h"

namespace dq {

constexpr int kGroup = 16;        // entries per group (Section 5 "configuration")
constexpr int kSG = 256;          // entries per super-group
constexpr int kGroupsPerSG = 16;
constexpr int kWaveSGs = 4;       // one wave64 = 64 groups = 4 super-groups per tile
constexpr int kBlockThreads = 256;
constexpr int kBlockWaves = kBlockThreads / 64;
constexpr uint32_t kMaxGridRows = 65535;  // documented limit of gridDim.y

// One unit of work: a chunk of one simulated worker.
struct Job {
  const uint8_t *in;   // packed partial sum (DAR, decompress) or nullptr (compress)
  const void *local;   // local slice, may be nullptr for decompress
  const float *mu;     // one mean per super-group of the chunk, taken off the local entries, or nullptr
  const uint32_t *src; // per super-group of the chunk: which super-group of `local` holds its entries
                       // (nullptr: `local` holds the chunk's super-groups in chunk order)
  void *out;           // packed (compress, DAR) or fp32 (decompress)
  const uint32_t *dest; // decompress: per super-group of the chunk, the super-group index in `out` it is written to
                        // (nullptr: the chunk's own order, from out[0])
  const float *back;    // decompress: per super-group, the mean added back n_workers times, or nullptr
  uint64_t first_sg;   // global index of the chunk's first super-group
  uint32_t n_sg[4];    // super-groups at 2, 4, 8 and 16 bits
  uint32_t rank;       // worker doing the compression (feeds the random streams)
};

inline Job make_job(const uint8_t *in, const void *local, const float *mu, void *out, uint64_t first_sg,
                    const uint32_t n_sg[4], uint32_t rank) {
  Job j;
  j.in = in; j.local = local; j.mu = mu; j.src = nullptr; j.out = out; j.dest = nullptr; j.back = nullptr;
  j.first_sg = first_sg;
  for (int w = 0; w < 4; ++w) j.n_sg[w] = n_sg[w];
  j.rank = rank;
  return j;
}

// Table blob (dword offsets).  The tables whose size does not depend on the level sets come
// first, at constant places, so that the kernels address them with immediate offsets; the two
// search tables, whose size follows the level sets, come last.  The kernels take LDS byte address
// 0 for the start of the blob: they use dynamic LDS only, which starts at 0 when a kernel has no
// static LDS (checked once per context, see static_lds_bytes).
constexpr uint32_t kOffRec = 0;        // 128 pairs {bits((1+m/128)/255) - bias, bits(255/(1+m/128)) + bias}, bias = 127 << 23
constexpr uint32_t kOffDec2 = 256;     // 2-bit decode: 256 bytes x 4 signed levels
constexpr uint32_t kOffDec4 = 1280;    // 4-bit decode: 256 bytes x 2 signed levels
constexpr uint32_t kOffTab4 = 1792;    // 4-bit levels: 7 pairs of entries {T[r], D[r], T[r+1], r << 28}, of r+1 and of r
constexpr uint32_t kOffDec8 = 1848;    // 8-bit decode: 256 signed levels
constexpr uint32_t kOffTab8 = 2104;    // 8-bit levels: 127 pairs of entries {T[r], D[r], T[r+1], r << 24}
constexpr uint32_t kOffLut4 = 3120;    // search table of the 4-bit set: (2^m + 1) pairs {next level, address of the candidate's pair}

// Behind the blob lie two more of the same layout for dq_thin.hip, with level entries {T[r], T[r+1]} of 8 bytes: of the 8-bit set, and of both.

// Everything the kernels need besides the job: PRNG key, worker count, table blob.
struct Params {
  const uint32_t *guard; // null, or a word the single-chunk kernels read first: if it is guard_call they do nothing (dq_bounds.hip)
  const uint32_t *blob;  // device copy of the table blob
  uint32_t blob_dwords;  // multiple of 4
  float magic[3];        // 2^(20-m) plus the search table's LDS address in units of its last bit (see quantize_codes)
  uint32_t key0, key1, round;
  uint32_t n_workers;
  uint32_t perm_bits;    // ceil(log2 n): width of the integers the rounding permutation mixes
  uint32_t n_slots;      // intervals the rounding divides [0,1) into: n, or 1 for independent rounding
  uint32_t slot_keep;    // all ones, or 0 for independent rounding: every slot is 0
  uint32_t guard_call;   // (here, where alignment leaves four bytes: in front of the tables' fields it cost a small hop 0.2 us of 4.9)
  uint64_t g_mod;        // nibble g: g mod n_slots (g itself above 16)
  float inv_n;           // 1 / n_slots
  float inv_n512;        // inv_n / 512
  float s_n;             // inv_n / 256: one step of an entry's random byte
};

enum Kind { kCompress = 0, kDar = 1, kDecompress = 2 };

// One chunk of one bucket on its way through a whole schedule (dq_walk.hip).
struct WalkPath {
  Job job;          // `local` is the chunk's byte offset inside every worker's tensor; `in` and `rank` are not used
  uint8_t *msg[2];  // ring, chain: where the packed messages of even and odd steps go (the last two are written)
  uint32_t chunk;
};
struct Walk {
  const void *const *grads;  // device: the workers' tensors, all twice
  uint32_t n, log_n;         // workers (log_n: butterfly)
  uint32_t encodes;          // how many leaves are followed by an encoding: n - 1, or n with the all-gather
  uint32_t first_kept;       // ring, chain: first step whose message is written
  uint32_t chain;            // 1: leaf i is worker i
  uint32_t hops_log;         // log2 of the hops one call of the per-super-group draws covers
  uint32_t levels, raw;      // butterfly: messages that can be pending beside the one in registers; whether some chunk has 16-bit super-groups
  uint32_t stack_bytes;      // LDS per wave for them
  uint32_t tile_sgs;         // super-groups of a wave's tile: 4 (dq_walk.hip), 2 or 1 (dq_thin.hip)
  uint32_t n_paths;
  uint32_t blocks, waves;    // grid, waves per block
  uint32_t order;            // which share a wave takes (share_of): 0, kReversed, or the CUs that the shares are spread over
  uint32_t raw_beside;       // spread: CUs with a block more have the last shares in it, raw ones, not the first
};
// With what only the host needs.  (In the kernels' arguments two words more in front of Params cost a small replay 0.2 us of 5.3.)
struct WalkGrid : Walk {
  uint32_t most_blocks;      // of such a grid
  bool full;                 // whether SIMDs have more than two waves
};
constexpr uint32_t kReversed = 0xFFFFFFFFu;
struct WalkShare {
  uint32_t path, tile;
};
constexpr uint32_t kStackCoded = 1280, kStackRaw = 2048;  // bytes of a pending message per wave: codes and scale, or raw bf16
uint32_t thin_lds(const Params &P, uint32_t stack_bytes);           // per block
uint32_t thin_stack(uint32_t tile_sgs, uint32_t levels);            // per wave
hipError_t launch_thin(dq_dtype dtype, bool tree, const WalkPath *paths_dev, const WalkShare *shares_dev, const WalkGrid &W, const Params &P,
                       hipStream_t stream);
// tiles: of one, two and four super-groups.  False: no launch fits
bool grid_walk(const Params &P, dq_dtype dtype, bool tree, uint32_t n_cu, const uint64_t tiles[3], WalkGrid *W);
struct Costs { uint32_t of[4]; };
Costs costs_of(dq_dtype dtype, bool tree, uint32_t n, uint32_t tile_sgs);  // of a tile, by width
void split_walk(const WalkPath *paths_host, dq_dtype dtype, bool tree, const Walk &W, std::vector<WalkShare> *shares);
hipError_t launch_walk(dq_dtype dtype, bool tree, bool means, const WalkPath *paths_dev, const WalkShare *shares_dev, const WalkGrid &W,
                       const Params &P, hipStream_t stream);

// Class counts that a search tells the host as soon as it has them (dq_bounds.hip): per bucket one word in pinned memory, counts of
// 17 bits with a tag above them.  Null: not told.  No ticket for more buckets than a workspace holds.
struct Announce {
  uint64_t *host;
  uint32_t tag;
};
// The tables of a whole replay on the original tensors, made on the device from the allocation's class counts (pp_kernels.hip).
struct Tables {
  WalkPath *paths;
  WalkShare *shares;
  float *out;
  const uint32_t *origin;
  const float *mu;          // in reordered order, or null
  uint32_t n_chunks, n_buckets, chunk_sgs, bucket_sgs;
  uint32_t by_chunk;        // paths of the same chunk number next to each other
  uint32_t entry_bytes;
  uint32_t waves, tile_log;  // shares; log2 of a tile's super-groups
  uint32_t slots;            // waves of every path, one tile at most for each; 0: shares by cost
  Costs cost;
};
constexpr uint32_t kMostTablePaths = 1024;  // a thread each
constexpr uint32_t kMostTensors = 256;      // whose addresses travel in a launch's arguments
// dq_sg_stats of all workers and dq_stats_combine in one launch; grads (or null): the tensors' addresses, all twice, are put down there
dq_status stats_all(const void *const *tensors, uint32_t n_workers, dq_dtype dtype, uint64_t n_sg, float *mu, float *F, const void **grads,
                    hipStream_t stream);
// The search of an allocation alone: counts, and every row's first places in `places`.  Buckets of at most kMostSearched super-groups.
constexpr uint32_t kMostSearched = 65536;
dq_status search(const float *F, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint64_t max_code_bits, uint32_t max_width, uint32_t *places,
                 uint32_t *counts, Announce announce, hipStream_t stream);
// Both in one launch, for one bucket; the places hold the rows' lists, where it takes them, and are not results.
bool takes_search_arrange(uint32_t n_sg_per_bucket, uint32_t n_buckets, const Tables &tables);
dq_status search_arrange(const float *F, const float *mu, uint32_t n_sg, uint64_t max_code_bits, uint32_t max_width, uint32_t *places, float *mu_main,
                         uint32_t *origin, Announce announce, const Tables &tables, hipStream_t stream);
// Behind it: the means in reordered order (mu and mu_main, or both null), the origins, and the tables.
dq_status arrange(const float *F, const float *mu, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint32_t max_width, const uint32_t *counts,
                  const uint32_t *places, float *mu_main, uint32_t *origin, const Tables &tables, hipStream_t stream);

// kernel launchers (dq_kernels.hip); grid_blocks = thread blocks the GPU keeps resident at once
hipError_t launch_one(Kind kind, dq_dtype dtype, bool has_local, const Job &job, const Params &p, uint32_t n_cu, uint32_t grid_blocks,
                      hipStream_t stream);
// the same for chunks of few super-groups (dq_few.hip), and whether a call is one
hipError_t launch_few(Kind kind, dq_dtype dtype, bool has_local, const Job &job, const Params &p, hipStream_t stream);  // makes an armed check itself
bool takes_few(Kind kind, const Job &job, const Params &p, uint32_t n_cu);
// gather: some job of the batch has a `src` (jobs without one still take the contiguous path)
hipError_t launch_batch(Kind kind, dq_dtype dtype, bool has_local, bool gather, const Job *jobs_dev, uint32_t n_jobs,
                        uint32_t max_tiles_per_job, const Params &p, uint32_t grid_blocks,
                        hipStream_t stream);

constexpr uint32_t kAnnounced = 511;  // buckets
hipError_t announce_begin(uint32_t n_buckets, hipStream_t stream, Announce *announce, void **ticket);
void announce_drop(void *ticket);  // nothing has been enqueued

// The check that this thread has armed (dq_bounds.h), enqueued now if it has not been: what the call's kernel reads first
struct Guard;
hipError_t armed_guard(hipStream_t stream, Guard *guard);

// 16 zero bytes at a 16-byte aligned device address, written by a kernel
// dst[0..bytes) = src[0..bytes) in 16-byte words (bytes a multiple of 16), except that the bytes from `valid`
// on are written as zero: the copy that stands in for the wire puts a packed block's padding down itself
hipError_t wire_copy(void *dst, const void *src, size_t bytes, size_t valid, hipStream_t stream);

// Largest static LDS size over the kernels that address their tables from LDS byte 0 (must be 0): all kernels
// of dq_kernels.hip that take a table, of dq_few.hip, of dq_walk.hip and of dq_thin.hip
hipError_t static_lds_bytes(size_t *bytes);
hipError_t walk_static_lds(size_t *bytes);  // raise *bytes to what their kernels have
hipError_t thin_static_lds(size_t *bytes);
hipError_t few_static_lds(size_t *bytes);
template <typename K>
hipError_t add_static_lds(K kernel, size_t *bytes) {
  hipFuncAttributes attr;
  const hipError_t e = hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(kernel));
  if (e == hipSuccess && attr.sharedSizeBytes > *bytes) *bytes = attr.sharedSizeBytes;
  return e;
}

// streaming probe (probe_kernels.hip): reads in_bytes, writes out_bytes (multiples of 16, out <= in)
hipError_t stream_probe(const void *in, size_t in_bytes, void *out, size_t out_bytes, uint32_t n_cu, hipStream_t stream);

// Whether work enqueued on s goes into a graph.  (The null stream is never captured; asked while another stream is, the runtime may
// answer with an error.)
inline hipError_t is_captured(hipStream_t s, bool *yes) {
  *yes = false;
  if (!s) return hipSuccess;
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  const hipError_t e = hipStreamIsCapturing(s, &status);
  *yes = status != hipStreamCaptureStatusNone;
  return e;
}

// DQ_OK, or DQ_EHIP after recording the error's text for dq_last_hip_error (dq_api.cpp)
dq_status hip_status(hipError_t e);

struct MxJob {
  const uint8_t *in;
  const void *local;
  void *out;
  uint64_t n_entries;
};
hipError_t mx_launch_one(Kind kind, dq_codec fmt, dq_dtype dtype, bool has_local, const MxJob &job, uint32_t n_cu,
                         hipStream_t stream);
hipError_t mx_launch_batch(Kind kind, dq_codec fmt, dq_dtype dtype, bool has_local, const MxJob *jobs_dev,
                           uint32_t n_jobs, uint64_t max_entries_per_job, uint32_t n_cu, hipStream_t stream);

// A whole replay of an MX codec in one launch: all chunks have the same size, so a path (bucket, chunk) is found by arithmetic.
struct MxWalk {
  const void *const *grads;  // device: the workers' tensors
  float *out;
  uint8_t *msg[2];           // ring, chain: messages of even and odd steps, one every msg_stride bytes
  size_t msg_stride;
  uint64_t chunk_blocks;     // blocks of 32 entries per chunk
  uint32_t n_chunks, n_tiles, tiles_per_path;  // a tile: 64 blocks of one chunk
  uint32_t n, log_n, encodes, first_kept, chain;  // as in Walk
  uint32_t wave_bytes;       // set by the launcher: LDS per wave
};
hipError_t launch_mx_walk(dq_codec fmt, dq_dtype dtype, bool tree, const MxWalk &W, uint32_t n_cu, hipStream_t stream);

}  // namespace dq

// context internals shared between dq_api.cpp and dq_replay.cpp
struct dq_ctx {
  dq_config cfg;
  dq::Params params;
  void *tables;          // the level tables it shares with other contexts (dq_api.cpp)
  uint32_t n_cu;
  uint32_t grid_blocks;  // n_cu x blocks per CU (5, or the DQ_BLOCKS_PER_CU environment variable at dq_create)
  int device;
  hipEvent_t pipe_event[2];  // block pipeline: fork (0) and join (1) of its two streams; made and destroyed with the context
  bool have_event[2];        // which of the two exist
  bool have_events;          // both
  void *static_stage;  // this device's copy of the library's static staging array (dq_dar_hop_pipelined_static), or null
};
