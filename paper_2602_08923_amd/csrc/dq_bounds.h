// Between libdq and its Python binding and tests (not part of the C ABI): see dq_bounds.hip.
#pragma once
#include <stdint.h>

#include "dq.h"

namespace dq {
struct Bound {
  const uint32_t *index;  // device
  uint32_t n, limit;      // every index must be below limit
};
#ifdef __HIPCC__
__host__ __device__
#endif
inline bool same_array(const Bound &a, const Bound &b) { return a.index == b.index && a.n == b.n; }
constexpr uint32_t kFetchWords = 1023;
struct Guard {
  const uint32_t *word;  // device, or null: the call's kernels do nothing if it holds `call`
  uint32_t call;
};
// A check made by the blocks of the call's own kernel.
struct OwnCheck {
  Bound a, b;
  uint32_t *host;       // where the verdict goes, with the call's number
  uint32_t call;
  uint32_t src_limit;   // of the indices that the kernel reads through before it knows the verdict
};
// Of the check that this thread has armed: how many indices a kernel that makes it itself would look at (0: none is armed; all ones: it is
// to be a launch of its own, as a tensor smaller than a super-group leaves no index that may be used meanwhile) ...
uint64_t own_check_due();
// ... to be made by the kernel itself (false: there is none, or not so) ...
bool take_own_check(const uint32_t *src, OwnCheck *check);
// ... or enqueued in front of it: armed_guard (dq_device.h)
}  // namespace dq

extern "C" {
// Arm a check of one or two index arrays (not under capture) for the one call that this thread makes until
// dqx_bounds_end, which waits for the verdict (bit k: array k has an index out of bounds).  The call in between does nothing
// if a bit is set.
dq_status dqx_bounds_begin(const dq::Bound *bounds, int n_bounds, void *hip_stream);
dq_status dqx_bounds_end(void *hip_stream, int *out_of_bounds);
// n <= kFetchWords words of device memory as the stream's work so far leaves them (waits for it; not under capture): a copy of a few words by
// hipMemcpy costs 13 us on top of the wait.
dq_status dqx_fetch(const uint32_t *src, uint32_t n, uint32_t *dst_host, void *hip_stream);
// dq_allocate, with the class counts sent to the host as soon as the search has them, while the rest of the call and what is enqueued after
// it run (not under capture); dqx_allocate_end waits for them: rows of four.  A null ticket: not so (buckets above 65,536 super-groups,
// more than 500 of them); dqx_fetch of the counts then.  No place for a ticket: they are not asked for.
// lists: dqx_allocate_lists words of memory that the call's kernels may write to (0: it needs none), or null, which costs some large buckets a launch more.
// beside: for a call on a stream of its own beside work that has the chip: few blocks rather than a short call.  The same results.
uint64_t dqx_allocate_lists(uint32_t n_sg_per_bucket, uint32_t n_buckets, uint32_t max_width);
dq_status dqx_allocate_begin(const float *F, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint64_t max_code_bits, uint32_t max_width,
                             uint8_t *widths, uint32_t *pos, uint32_t *counts, uint32_t *lists, int beside, void *hip_stream, void **ticket);
dq_status dqx_allocate_end(void *ticket, uint32_t n_sg_per_bucket, uint32_t n_buckets, uint32_t *rows, void *hip_stream);
// dq_replay_create for a scratch that belongs to a stream (memory that its earlier work may still be using): the tables are
// uploaded as work of that stream, nothing is waited for.  Not while the stream is captured.
dq_status dqx_replay_create(dq_ctx *ctx, const dq_replay_desc *desc, const void *const *worker_grads, void *scratch, size_t scratch_bytes,
                            float *out, dq_replay **plan, void *hip_stream);
// A whole simulated all-reduce of n_workers (the context's) tensors in their original order, ring or recursive halving, codec DynamiQ: dq_sg_stats,
// dq_stats_combine, dq_allocate, dq_reorder_mean and a replay with origin and inputs_in_original_order, the same bits, without waiting (not under
// capture).  The class counts come with the ticket (dqx_allocate_end).  0 bytes: not such a call, or too large for it.
struct dqx_whole {
  dq_topology topology;
  dq_dtype dtype;
  uint32_t n_sg_bucket, n_buckets;
  uint64_t max_code_bits;
  uint32_t max_width, all_gather, means;
  uint32_t n_tensors;  // as many as the context has workers
};
size_t dqx_whole_scratch_bytes(const dq_ctx *ctx, const dqx_whole *desc);
dq_status dqx_whole_run(const dq_ctx *ctx, const dqx_whole *desc, const void *const *tensors, void *scratch, float *out, void *hip_stream, void **ticket);
// Where its scratch holds the shares of the replay's waves, blocks * waves and an end, {path, tile} each; for the tests.
struct dqx_tables {
  size_t shares;
  uint32_t blocks, waves, tile_sgs, by_chunk;  // by_chunk: paths of the same chunk next to each other, not of the same bucket
};
dq_status dqx_whole_tables(const dq_ctx *ctx, const dqx_whole *desc, dqx_tables *tables);
// Whether its search and what the replay needs of it are one launch, on this device, for a replay of so many waves; for the tests.
int dqx_searches_and_arranges(uint32_t n_sg_per_bucket, uint32_t n_buckets, uint32_t waves);
// Adds to *wrong (device) how many results of the codec's reciprocal differ from the division's.
dq_status dqx_reciprocals(uint32_t *wrong, void *hip_stream);
// Where the waves of a replay of n_paths paths begin (dq_walk.hip), {path, tile} each and an end.
void dqx_split(const uint32_t *n_sg, uint32_t n_paths, uint32_t n_workers, int f32, int tree, uint32_t tile_sgs, uint32_t blocks, uint32_t waves,
               uint32_t *shares);
// dq_sg_stats of n_workers (at most 256) tensors and dq_stats_combine in one launch.
dq_status dqx_stats_all(const void *const *tensors, uint32_t n_workers, dq_dtype dtype, uint64_t n_sg, float *mu, float *F,
                        void *hip_stream);
}
