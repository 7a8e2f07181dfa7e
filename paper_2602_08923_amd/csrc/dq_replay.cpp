// Hop replay: the reduce-scatter schedules of Section 3.4 ("Reduce-scatter", "Fused
// kernels") and Appendix B run for N simulated workers whose gradients all sit in this
// GPU's HBM.  A transfer between workers is a pointer hand-off: the buffer one worker's
// kernel writes at step t is the packed_in of the receiving worker's kernel at step t+1.
// Every step is one launch (two where a node both forwards and keeps) whose grid covers
// all (worker, chunk) jobs of that step; the job tables are built once, here, on the host.
#include <string.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

#include "dq_bounds.h"
#include "dq_device.h"

namespace {

struct HostJob {
  const uint8_t *in;
  const void *local;
  const float *mu;
  const uint32_t *src = nullptr;
  const uint32_t *dest = nullptr;
  const float *back = nullptr;
  void *out;
  uint64_t first_sg;
  uint32_t n_sg[4];
  uint32_t rank;
};

struct Launch {
  dq::Kind kind;
  dq_dtype dtype;  // dtype of `local`
  bool has_local = true;  // false: decompress without accumulation
  bool gather = false;    // some job reads its local super-groups through an index
  std::vector<HostJob> jobs;  // freed once the table is on the device
  uint32_t n_jobs = 0;
  size_t table_off = 0;  // byte offset of this launch's job table in scratch
  uint32_t max_tiles = 0;
  uint64_t max_entries = 0;
  uint64_t entries = 0;
};

struct Step {
  std::vector<Launch> launches;
};

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct Plan {
  std::vector<Step> steps;
  size_t scratch_bytes = 0;
  // ring and chain only: where the message of (bucket, chunk) sits inside a message set, its size, and
  // the two sets' starts (step t writes set t & 1); what dq_replay_message answers from
  std::vector<size_t> ring_slot, ring_bytes;
  uint8_t *ring_msg[2] = {nullptr, nullptr};
  uint32_t ring_chunks = 0;   // chunks per bucket (0: not a ring or chain)
  uint32_t ring_message_steps = 0;  // steps 0 .. this-1 write messages
  // the whole schedule as one launch (dq_walk.hip): one path per (bucket, chunk), the workers' tensors
  bool walk = false, tree = false;
  dq::WalkGrid w = {};
  dq::MxWalk mx = {};
  std::vector<dq::WalkPath> paths;  // freed once they are on the device
  std::vector<dq::WalkShare> shares;
  size_t paths_off = 0, shares_off = 0, grads_off = 0;
};

bool is_mx(dq_codec c) { return c == DQ_MXFP8_E4M3 || c == DQ_MXFP6_E3M2 || c == DQ_MXFP4_E2M1; }

size_t chunk_bytes(dq_codec codec, const uint32_t n_sg[4]) {
  if (is_mx(codec)) return dq_mx_packed_bytes(codec, ((uint64_t)n_sg[0] + n_sg[1] + n_sg[2] + n_sg[3]) * 256);
  dq_chunk ch{0, {n_sg[0], n_sg[1], n_sg[2], n_sg[3]}};
  return dq_packed_bytes(&ch);
}

size_t elt_size(dq_dtype t) { return t == DQ_F32 ? 4 : 2; }

// Width counts of chunk c (of n equal chunks) of a reordered bucket: 2-bit SGs first,
// then 4-bit, 8-bit and 16-bit.
void chunk_widths(const uint32_t by_width[4], uint64_t m, uint32_t c, uint32_t out[4]) {
  uint64_t edges[5] = {0, 0, 0, 0, 0};
  for (int w = 0; w < 4; ++w) edges[w + 1] = edges[w] + by_width[w];
  const uint64_t lo = (uint64_t)c * m, hi = lo + m;
  for (int w = 0; w < 4; ++w) {
    const uint64_t a = lo > edges[w] ? lo : edges[w], b = hi < edges[w + 1] ? hi : edges[w + 1];
    out[w] = b > a ? (uint32_t)(b - a) : 0;
  }
}

struct ChunkInfo {
  uint32_t n_sg[4];
  uint64_t first_sg;
  size_t bytes;
};

// Few tiles per wave: the buckets' chunks of the same place, which have about the same widths, one after the other.  The order of all tiles
// goes from narrow to wide once, and the waves that share a CU take them from different places of it, not from the same place of several
// buckets.  (From some eight tiles per wave on they meet all widths anyway, and the order of the memory is the better one: recursive halving
// over 16, eight buckets of 51,200 super-groups, 825 us against 838.  Up to four workers, whose tiles cost memory's time and not their width's, it is no
// better either, 0.4 % either way on average of 146 schedules, but in some: halving over 2 in fp32, 3 x 11,456 at 4 bits, 20.0 against 20.8.)
bool by_chunk_number(const dq::Walk &w, uint32_t n_buckets, uint64_t n_sg_bucket) {
  return n_buckets > 1 && w.n > 4 && n_buckets * n_sg_bucket < 8ull * w.tile_sgs * w.blocks * w.waves;
}

// The schedule's part of W.
void describe(uint32_t n, dq_topology topology, bool all_gather, dq::Walk *w) {
  w->n = n;
  while ((1u << w->log_n) < n) ++w->log_n;
  w->encodes = all_gather ? n : n - 1;
  w->first_kept = n > 3 ? n - 3 : 0;
  w->chain = topology == DQ_CHAIN;
  while ((1u << w->hops_log) < w->encodes && w->hops_log < 4) ++w->hops_log;
  w->levels = topology == DQ_BUTTERFLY && w->log_n > 1 ? w->log_n - 1 : 0;
}

// The same schedule as one launch that carries every tile through all its hops (dq_walk.hip).
void plan_walk(const dq_ctx *ctx, const dq_replay_desc *d, const ChunkInfo *ci, uint32_t n_chunks, uint64_t m, float *out, Plan *plan,
               size_t *off) {
  const uint32_t n = ctx->cfg.n_workers;
  const size_t es = elt_size(d->dtype);
  const uint64_t bucket_bytes = d->n_sg_bucket * 256 * es;
  dq::WalkGrid &w = plan->w;
  describe(n, d->topology, d->all_gather != 0, &w);
  plan->tree = d->topology == DQ_BUTTERFLY;
  bool raw = false;
  w.n_paths = d->n_buckets * n_chunks;
  plan->paths.resize(w.n_paths);
  for (uint32_t b = 0; b < d->n_buckets; ++b)
    for (uint32_t c = 0; c < n_chunks; ++c) {
      const size_t i = (size_t)b * n_chunks + c;
      const ChunkInfo &x = ci[i];
      dq::WalkPath &p = plan->paths[i];
      const uint64_t sg = x.first_sg - d->first_sg;  // place in the reordered bucket set
      const uint64_t local = (uint64_t)b * bucket_bytes + (d->inputs_in_original_order ? 0 : (uint64_t)c * m * 256 * es);
      float *o = out + (uint64_t)b * d->n_sg_bucket * 256;
      p.job = dq::make_job(nullptr, reinterpret_cast<const void *>((uintptr_t)local), d->mu ? d->mu + sg : nullptr,
                           d->origin ? o : o + (uint64_t)c * m * 256, x.first_sg, x.n_sg, 0);
      if (d->inputs_in_original_order) p.job.src = d->origin + sg;
      if (d->origin) {
        p.job.dest = d->origin + sg;
        p.job.back = d->mu ? d->mu + sg : nullptr;
      }
      for (int k = 0; k < 2; ++k) p.msg[k] = plan->ring_chunks ? plan->ring_msg[k] + plan->ring_slot[i] : nullptr;
      p.chunk = c;
      raw = raw || x.n_sg[3] != 0;
    }
  w.raw = raw;
  uint64_t tiles[3] = {0, 0, 0}, two = 0, sixteen = 0;
  for (const dq::WalkPath &p : plan->paths) {
    two += p.job.n_sg[0];
    sixteen += p.job.n_sg[3];
    for (uint32_t k : p.job.n_sg) {
      tiles[0] += k;
      tiles[1] += (k + 1) / 2;
      tiles[2] += (k + 3) / 4;
    }
  }
  w.raw_beside = sixteen > two;
  plan->walk = dq::grid_walk(ctx->params, d->dtype, plan->tree, ctx->n_cu, tiles, &w);
  if (!plan->walk) {
    plan->paths.clear();
    return;
  }
  if (by_chunk_number(w, d->n_buckets, d->n_sg_bucket)) {
    std::vector<dq::WalkPath> by_chunk;
    by_chunk.reserve(plan->paths.size());
    for (uint32_t c = 0; c < n_chunks; ++c)
      for (uint32_t b = 0; b < d->n_buckets; ++b) by_chunk.push_back(plan->paths[(size_t)b * n_chunks + c]);
    plan->paths.swap(by_chunk);
  }
  *off = align_up(*off, 256);
  plan->paths_off = *off;
  *off += plan->paths.size() * sizeof(dq::WalkPath);
  *off = align_up(*off, 256);
  plan->shares_off = *off;
  *off += ((size_t)w.blocks * w.waves + 1) * sizeof(dq::WalkShare);
  *off = align_up(*off, 256);
  plan->grads_off = *off;
  *off += 2 * (size_t)n * sizeof(void *);
}

void plan_mx_walk(const dq_ctx *ctx, const dq_replay_desc *d, uint32_t n_chunks, uint64_t m, float *out, Plan *plan, size_t *off) {
  const uint32_t n = ctx->cfg.n_workers;
  dq::MxWalk &w = plan->mx;
  w.n = n;
  while ((1u << w.log_n) < n) ++w.log_n;
  w.encodes = d->all_gather ? n : n - 1;
  w.first_kept = n > 3 ? n - 3 : 0;
  w.chain = d->topology == DQ_CHAIN;
  plan->tree = d->topology == DQ_BUTTERFLY;
  w.out = out;
  w.chunk_blocks = m * 8;
  w.n_chunks = n_chunks;
  const uint64_t per_path = (w.chunk_blocks + 63) / 64, tiles = per_path * d->n_buckets * n_chunks;
  if (tiles >= (1ull << 31)) return;  // tile numbers are 32-bit: step by step
  w.tiles_per_path = (uint32_t)per_path;
  w.n_tiles = (uint32_t)tiles;
  if (plan->ring_chunks) {
    w.msg[0] = plan->ring_msg[0];
    w.msg[1] = plan->ring_msg[1];
    w.msg_stride = align_up(plan->ring_bytes[0], 256);  // equal chunks: slot i starts at i * msg_stride
  }
  plan->walk = true;
  *off = align_up(*off, 256);
  plan->grads_off = *off;
  *off += 2 * (size_t)n * sizeof(void *);
}

// Builds the whole schedule.  With base == nullptr only sizes are computed (pointers are
// offsets from zero); grads may then be null.
dq_status build_plan(const dq_ctx *ctx, const dq_replay_desc *d, const void *const *grads, uint8_t *base, float *out,
                     Plan *plan) {
  if (!ctx || !d) return DQ_EINVAL;
  const uint32_t n = ctx->cfg.n_workers;
  const bool mx = is_mx(d->codec);
  if (!mx && d->codec != DQ_DYNAMIQ) return DQ_EINVAL;
  if (d->dtype != DQ_F32 && d->dtype != DQ_BF16) return DQ_EINVAL;
  if (n < 2 || d->n_buckets < 1 || d->n_sg_bucket < 1) return DQ_EINVAL;
  if (!mx && !d->n_sg_by_width) return DQ_EINVAL;
  if (mx && d->mu) return DQ_EINVAL;  // the MX codec has no normalization
  if (mx && d->origin) return DQ_EINVAL;
  if (d->inputs_in_original_order && (!d->origin || d->topology == DQ_CHAIN)) return DQ_EINVAL;
  if ((reinterpret_cast<uintptr_t>(d->mu) & 3u) || (reinterpret_cast<uintptr_t>(d->origin) & 3u)) return DQ_EALIGN;
  if (d->topology == DQ_CHAIN) {
    if (d->n_buckets != 1) return DQ_EINVAL;
  } else if (d->topology == DQ_RING || d->topology == DQ_BUTTERFLY) {
    if (d->n_sg_bucket % n) return DQ_EINVAL;
    if (d->topology == DQ_BUTTERFLY && (n & (n - 1))) return DQ_EINVAL;
  } else {
    return DQ_EINVAL;
  }
  if (d->n_sg_bucket >= (1ull << 31)) return DQ_EUNSUPPORTED;
  const size_t es = elt_size(d->dtype);
  const uint64_t bucket_entries = d->n_sg_bucket * 256;
  const uint32_t n_chunks = d->topology == DQ_CHAIN ? 1 : n;
  const uint64_t m = d->n_sg_bucket / n_chunks;  // SGs per chunk
  const uint64_t chunk_entries = m * 256;

  // per (bucket, chunk): widths, packed size
  std::vector<ChunkInfo> ci((size_t)d->n_buckets * n_chunks);
  for (uint32_t b = 0; b < d->n_buckets; ++b) {
    uint32_t bw[4] = {(uint32_t)d->n_sg_bucket, 0, 0, 0};
    if (!mx) {
      memcpy(bw, d->n_sg_by_width + 4 * (size_t)b, sizeof(bw));
      if ((uint64_t)bw[0] + bw[1] + bw[2] + bw[3] != d->n_sg_bucket) return DQ_EINVAL;
    }
    for (uint32_t c = 0; c < n_chunks; ++c) {
      ChunkInfo &x = ci[(size_t)b * n_chunks + c];
      chunk_widths(bw, m, c, x.n_sg);
      x.first_sg = d->first_sg + (uint64_t)b * d->n_sg_bucket + (uint64_t)c * m;
      x.bytes = chunk_bytes(d->codec, x.n_sg);
    }
  }
  auto grad_ptr = [&](uint32_t w, uint32_t b, uint32_t c) -> const void * {
    const uint8_t *g = grads ? (const uint8_t *)grads[w] : nullptr;
    return g + ((uint64_t)b * bucket_entries + (uint64_t)c * chunk_entries) * es;
  };
  auto out_ptr = [&](uint32_t b, uint32_t c) -> float * {
    return out + (uint64_t)b * bucket_entries + (uint64_t)c * chunk_entries;
  };
  // raw: `local` is a worker's own gradient (its means are still to be taken off), not an fp32
  // buffer of sums that already had them taken off
  auto mk = [&](const ChunkInfo &x, const uint8_t *in, const void *local, bool raw, void *o, uint32_t rank) {
    HostJob j;
    j.in = in;
    j.local = local;
    j.mu = (raw && d->mu) ? d->mu + (x.first_sg - d->first_sg) : nullptr;
    if (raw && d->inputs_in_original_order) {
      // `local` points at the chunk's place in a reordered bucket: step back to the bucket's start (the chunk
      // begins (first_sg - first of the bucket) super-groups in) and let the kernel gather through origin
      const uint64_t in_bucket = (x.first_sg - d->first_sg) % d->n_sg_bucket;
      j.local = static_cast<const uint8_t *>(local) - in_bucket * 256 * es;
      j.src = d->origin + (x.first_sg - d->first_sg);
    }
    j.out = o;
    j.first_sg = x.first_sg;
    memcpy(j.n_sg, x.n_sg, sizeof(j.n_sg));
    j.rank = rank;
    return j;
  };
  // The launch that writes the final result: with d->origin every super-group goes straight to its
  // original place in its bucket and gets its mean back (the restore, fused into the last kernel).
  auto finish = [&](HostJob j, const ChunkInfo &x, uint32_t b) {
    if (d->origin) {
      j.out = out + (uint64_t)b * bucket_entries;
      j.dest = d->origin + (x.first_sg - d->first_sg);
      j.back = d->mu ? d->mu + (x.first_sg - d->first_sg) : nullptr;
    }
    return j;
  };

  size_t off = 0;  // running scratch offset (job tables are appended at the end)
  plan->steps.clear();
  const bool sizes_only = base == nullptr;
  auto add = [&](Launch &L, const HostJob &j) {
    ++L.n_jobs;
    if (!sizes_only) L.jobs.push_back(j);
  };

  if (d->topology == DQ_CHAIN || d->topology == DQ_RING) {
    // two message sets (ping-pong), each with one slot per (bucket, chunk)
    std::vector<size_t> slot(ci.size());
    size_t set_bytes = 0;
    for (size_t i = 0; i < ci.size(); ++i) {
      slot[i] = set_bytes;
      set_bytes += align_up(ci[i].bytes, 256);
    }
    uint8_t *msg[2] = {base + off, base + off + set_bytes};
    off += 2 * set_bytes;
    plan->ring_slot = slot;
    plan->ring_bytes.resize(ci.size());
    for (size_t i = 0; i < ci.size(); ++i) plan->ring_bytes[i] = ci[i].bytes;
    plan->ring_msg[0] = msg[0];
    plan->ring_msg[1] = msg[1];
    plan->ring_chunks = n_chunks;
    plan->ring_message_steps = n - 1;
    const uint32_t hops = n;  // steps 0 .. n-1
    for (uint32_t t = 0; t < hops; ++t) {
      Step st;
      Launch L;
      L.dtype = d->dtype;
      L.kind = t == 0 ? dq::kCompress : (t == n - 1 ? dq::kDecompress : dq::kDar);
      for (uint32_t b = 0; b < d->n_buckets; ++b)
        for (uint32_t c = 0; c < n_chunks; ++c) {
          const size_t i = (size_t)b * n_chunks + c;
          // ring: chunk c is at worker c+t at step t; chain: slice t of the one chunk
          const uint32_t w = d->topology == DQ_CHAIN ? t : (c + t) % n;
          const void *local = d->topology == DQ_CHAIN ? grad_ptr(w, 0, 0) : grad_ptr(w, b, c);
          const uint8_t *in = t == 0 ? nullptr : msg[(t - 1) & 1] + slot[i];
          void *o = t == n - 1 ? (void *)out_ptr(b, c) : (void *)(msg[t & 1] + slot[i]);
          HostJob j = mk(ci[i], in, local, true, o, w);
          if (t == n - 1 && !d->all_gather) j = finish(j, ci[i], b);
          add(L, j);
        }
      st.launches.push_back(std::move(L));
      plan->steps.push_back(std::move(st));
    }
  } else {  // butterfly: recursive halving
    uint32_t Lg = 0;
    while ((1u << Lg) < n) ++Lg;
    // message region written at step k for receiver p: the chunks of p's keep range at step k
    // keep_lo(p, k): the chunks worker p still owns after step k
    auto keep_lo = [&](uint32_t p, uint32_t k) { return p & ~((n >> k) - 1); };
    // message sets: parity by step; region offsets per (bucket, receiver, chunk)
    std::vector<std::vector<size_t>> moff(Lg + 1);  // [k][(b*n + p)*half + (c - keep_lo)]
    size_t set_bytes[2] = {0, 0};
    for (uint32_t k = 1; k <= Lg; ++k) {
      const uint32_t half = n >> k;
      moff[k].resize((size_t)d->n_buckets * n * half);
      size_t o = 0;
      for (uint32_t b = 0; b < d->n_buckets; ++b)
        for (uint32_t p = 0; p < n; ++p)
          for (uint32_t j = 0; j < half; ++j) {
            moff[k][((size_t)b * n + p) * half + j] = o;
            o += align_up(ci[(size_t)b * n + keep_lo(p, k) + j].bytes, 256);
          }
      if (o > set_bytes[k & 1]) set_bytes[k & 1] = o;
    }
    uint8_t *msg[2] = {base + off, base + off + set_bytes[0]};
    off += set_bytes[0] + set_bytes[1];
    // fp32 keep-buffers: worker w, bucket b: the n/4 chunks it owns after step 2
    const uint32_t keep_chunks = n >= 4 ? n / 4 : 0;
    off = align_up(off, 256);
    float *acc = reinterpret_cast<float *>(base + off);
    off += (size_t)d->n_buckets * n * keep_chunks * chunk_entries * 4;
    auto acc_ptr = [&](uint32_t w, uint32_t b, uint32_t c) -> float * {
      return acc + (((uint64_t)b * n + w) * keep_chunks + (c - keep_lo(w, 2))) * chunk_entries;
    };
    auto msg_ptr = [&](uint32_t k, uint32_t b, uint32_t p, uint32_t c) -> uint8_t * {
      const uint32_t half = n >> k;
      return msg[k & 1] + moff[k][((size_t)b * n + p) * half + (c - keep_lo(p, k))];
    };
    for (uint32_t k = 1; k <= Lg; ++k) {
      const uint32_t half = n >> k;
      Step st;
      Launch send, keep;
      send.kind = k == 1 ? dq::kCompress : dq::kDar;
      keep.kind = dq::kDecompress;
      send.dtype = keep.dtype = (k <= 2) ? d->dtype : DQ_F32;  // later steps add into fp32 buffers
      for (uint32_t b = 0; b < d->n_buckets; ++b)
        for (uint32_t w = 0; w < n; ++w) {
          const uint32_t klo = keep_lo(w, k), partner = w ^ half;
          const uint32_t slo = klo ^ half;  // the other half of the range owned after step k-1
          for (uint32_t c = slo; c < slo + half; ++c) {
            const ChunkInfo &x = ci[(size_t)b * n + c];
            const uint8_t *in = k == 1 ? nullptr : msg_ptr(k - 1, b, w, c);
            const void *local = k <= 2 ? grad_ptr(w, b, c) : (const void *)acc_ptr(w, b, c);
            add(send, mk(x, in, local, k <= 2, msg_ptr(k, b, partner, c), w));
          }
          if (k >= 2)
            for (uint32_t c = klo; c < klo + half; ++c) {
              const ChunkInfo &x = ci[(size_t)b * n + c];
              const void *local = k == 2 ? grad_ptr(w, b, c) : (const void *)acc_ptr(w, b, c);
              add(keep, mk(x, msg_ptr(k - 1, b, w, c), local, k == 2, acc_ptr(w, b, c), w));
            }
        }
      st.launches.push_back(std::move(send));
      if (k >= 2) st.launches.push_back(std::move(keep));
      plan->steps.push_back(std::move(st));
    }
    // after the last exchange: worker w adds what it received for chunk w
    Step st;
    Launch fin;
    fin.kind = dq::kDecompress;
    fin.dtype = Lg == 1 ? d->dtype : DQ_F32;
    for (uint32_t b = 0; b < d->n_buckets; ++b)
      for (uint32_t w = 0; w < n; ++w) {
        const ChunkInfo &x = ci[(size_t)b * n + w];
        const void *local = Lg == 1 ? grad_ptr(w, b, w) : (const void *)acc_ptr(w, b, w);
        HostJob j = mk(x, msg_ptr(Lg, b, w, w), local, Lg == 1, out_ptr(b, w), w);
        if (!d->all_gather) j = finish(j, x, b);
        add(fin, j);
      }
    st.launches.push_back(std::move(fin));
    plan->steps.push_back(std::move(st));
  }

  if (d->all_gather) {
    // All-gather phase: the sink of each chunk compresses its fp32 sum (with its own rank: it has
    // compressed nothing of this chunk before, so these random numbers are fresh), and every
    // worker, the sink included, ends with the decompressed message.
    std::vector<size_t> slot(ci.size());
    off = align_up(off, 256);
    size_t region = 0;
    for (size_t i = 0; i < ci.size(); ++i) {
      slot[i] = region;
      region += align_up(ci[i].bytes, 256);
    }
    uint8_t *ag = base + off;
    off += region;
    Step sc, sd;
    Launch comp, dec;
    comp.kind = dq::kCompress;
    comp.dtype = DQ_F32;
    dec.kind = dq::kDecompress;
    dec.dtype = DQ_F32;
    dec.has_local = false;
    for (uint32_t b = 0; b < d->n_buckets; ++b)
      for (uint32_t c = 0; c < n_chunks; ++c) {
        const size_t i = (size_t)b * n_chunks + c;
        const uint32_t sink = d->topology == DQ_CHAIN ? n - 1 : (d->topology == DQ_RING ? (c + n - 1) % n : c);
        add(comp, mk(ci[i], nullptr, out_ptr(b, c), false, ag + slot[i], sink));
        add(dec, finish(mk(ci[i], ag + slot[i], nullptr, false, out_ptr(b, c), sink), ci[i], b));
      }
    sc.launches.push_back(std::move(comp));
    sd.launches.push_back(std::move(dec));
    plan->steps.push_back(std::move(sc));
    plan->steps.push_back(std::move(sd));
  }

  if (mx) plan_mx_walk(ctx, d, n_chunks, m, out, plan, &off);
  else plan_walk(ctx, d, ci.data(), n_chunks, m, out, plan, &off);

  // job tables
  for (Step &st : plan->steps)
    for (Launch &L : st.launches) {
      off = align_up(off, 256);
      L.table_off = off;
      off += (size_t)L.n_jobs * (mx ? sizeof(dq::MxJob) : sizeof(dq::Job));
      for (const HostJob &j : L.jobs) {
        if (j.src) L.gather = true;
        const uint32_t tiles = (j.n_sg[0] + 3) / 4 + (j.n_sg[1] + 3) / 4 + (j.n_sg[2] + 3) / 4 + (j.n_sg[3] + 3) / 4;
        const uint64_t e = ((uint64_t)j.n_sg[0] + j.n_sg[1] + j.n_sg[2] + j.n_sg[3]) * 256;
        if (tiles > L.max_tiles) L.max_tiles = tiles;
        if (e > L.max_entries) L.max_entries = e;
        L.entries += e;
      }
    }
  plan->scratch_bytes = align_up(off, 256);
  return DQ_OK;
}

// A plan's tables on their way to its scratch, in the order of their offsets; what lies between two pieces is padding.
//
// Scratch is recycled memory: the launch of an earlier replay, still running, may be reading its tables at the very place.  The binding
// therefore names the stream that the scratch belongs to, and the tables go there as that stream's work: a few blocks copy them
// from pinned memory (25 KB for 8 workers' ring of 8,192 super-groups) and then say so in flags that the host reads without a call
// into the runtime, for launches on other streams and under capture wait for them.  Without a stream, and for tables
// beyond kPinned, the host waits until nothing can be reading the scratch and copies.  (What bounds the blocks are their trips over
// PCIe, of which a CU has only so many under way: 25 KB take one block 8.0 us, sixteen 4.7.  A copy that the host waits for, besides needing
// an idle scratch: an all-reduce of 8 workers' 8,192 super-groups that made such a plan took 103 us instead of 88 to 94.)
constexpr size_t kPinned = 256u << 10;
constexpr size_t kStagings = 8;
constexpr uint32_t kUploadBlocks = 16, kUploadThreads = 128;
struct Staging {
  uint8_t *host = nullptr;            // pinned: kPinned bytes, then the flags
  volatile uint32_t *flag = nullptr;  // per block: number of the last upload of which its part has arrived
  uint32_t number = 0;
  bool arrived(uint32_t upload) const {  // or a later one
    bool all = true;
    for (uint32_t b = 0; b < kUploadBlocks; ++b) all = all && (int32_t)(__atomic_load_n(flag + b, __ATOMIC_ACQUIRE) - upload) >= 0;
    return all;
  }
  void set(uint32_t upload) {
    for (uint32_t b = 0; b < kUploadBlocks; ++b) __atomic_store_n(flag + b, upload, __ATOMIC_RELEASE);
  }
};
std::mutex g_staging_mutex;
std::vector<Staging *> g_stagings;  // at most kStagings, kept until the process ends; one is taken again when its last upload has arrived

__global__ void __launch_bounds__(kUploadThreads) k_upload(const uint4 *src, uint4 *dst, uint32_t words, uint32_t *flag, uint32_t number) {
  constexpr uint32_t kAll = kUploadBlocks * kUploadThreads;
  for (uint32_t i = blockIdx.x * kUploadThreads + threadIdx.x; i < words; i += 4 * kAll) {  // latency of the host's memory: four loads at a time
    const uint32_t j = i + kAll, k = i + 2 * kAll, l = i + 3 * kAll;
    const uint4 a = src[i], b = src[j < words ? j : i], c = src[k < words ? k : i], d = src[l < words ? l : i];
    dst[i] = a;
    if (j < words) dst[j] = b;
    if (k < words) dst[k] = c;
    if (l < words) dst[l] = d;
  }
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(flag + blockIdx.x, number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // fenced above
}

class Upload {
 public:
  // Stream: null pointer to one if the caller named none.
  Upload(uint8_t *scratch, const hipStream_t *stream) : scratch_(scratch), stream_(stream) {}
  void put(size_t off, const void *src, size_t bytes) {
    if (bytes == 0) return;
    if (!buf_.empty() && (off < first_ + buf_.size() || off - first_ + bytes > kMost)) send();
    if (buf_.empty()) first_ = off;
    buf_.resize(off - first_ + bytes);
    memcpy(buf_.data() + (off - first_), src, bytes);
  }
  // *staging: what the tables wait in, or null if they have arrived; *number: of the upload.
  dq_status finish(Staging **staging, uint32_t *number) {
    *staging = nullptr;
    if (buf_.empty() || status_ != DQ_OK) return status_;
    if (stream_ && !waited_ && buf_.size() <= kPinned) {
      hipError_t e = hipSuccess;
      if (enqueue(staging, number, &e)) return dq::hip_status(e);
    }
    send();
    if (status_ == DQ_OK) status_ = dq::hip_status(hipStreamSynchronize(nullptr));  // pageable memory: the copy may return before it is done
    return status_;
  }

 private:
  static constexpr size_t kMost = 16u << 20;
  static Staging *take() {  // its next upload is numbered `number`
    std::lock_guard<std::mutex> lock(g_staging_mutex);
    Staging *s = nullptr;
    for (Staging *x : g_stagings)
      if (x->arrived(x->number)) s = x;
    if (!s) {
      if (g_stagings.size() >= kStagings || !(s = new (std::nothrow) Staging)) return nullptr;
      if (hipHostMalloc((void **)&s->host, kPinned + 4 * kUploadBlocks, hipHostMallocPortable) != hipSuccess) {
        delete s;
        return nullptr;
      }
      s->flag = reinterpret_cast<volatile uint32_t *>(s->host + kPinned);
      s->set(0);
      g_stagings.push_back(s);
    }
    ++s->number;
    return s;
  }
  bool enqueue(Staging **staging, uint32_t *number, hipError_t *err) {
    Staging *s = take();
    if (!s) return false;
    const size_t bytes = align_up(buf_.size(), 16);  // scratch ends on a multiple of 256
    memcpy(s->host, buf_.data(), buf_.size());
    memset(s->host + buf_.size(), 0, bytes - buf_.size());
    const uint32_t mine = s->number;
    hipLaunchKernelGGL(k_upload, dim3(kUploadBlocks), dim3(kUploadThreads), 0, *stream_, reinterpret_cast<const uint4 *>(s->host),
                       reinterpret_cast<uint4 *>(scratch_ + first_), (uint32_t)(bytes / 16), const_cast<uint32_t *>(s->flag), mine);
    if ((*err = hipGetLastError()) == hipSuccess) {
      *number = mine;
      *staging = s;
    } else {
      s->set(mine);  // nothing reads it
    }
    return true;
  }
  void send() {
    if (status_ == DQ_OK && !waited_) {
      status_ = dq::hip_status(stream_ ? hipStreamSynchronize(*stream_) : hipDeviceSynchronize());
      waited_ = true;
    }
    if (!buf_.empty() && status_ == DQ_OK) status_ = dq::hip_status(hipMemcpy(scratch_ + first_, buf_.data(), buf_.size(), hipMemcpyHostToDevice));
    buf_.clear();
  }
  uint8_t *scratch_;
  const hipStream_t *stream_;
  size_t first_ = 0;
  std::vector<uint8_t> buf_;
  bool waited_ = false;  // for what may read the scratch
  dq_status status_ = DQ_OK;
};

}  // namespace

struct dq_replay {
  dq_ctx *ctx;
  dq_codec codec;
  Plan plan;
  uint8_t *scratch;
  std::vector<hipEvent_t> events;
  dq_dtype dtype;
  bool means, all_gather;
  // A whole replay in one launch leaves the steps' buffers behind: what they hold since then.
  bool complete = true;   // all that steps can read (of a ring or chain without all-gather a whole replay writes it)
  uint32_t filled = 0;    // else: the messages and keep-buffers of steps 0 .. filled-1
  bool gathered = false;  // else: the all-gather's messages
  // the upload of the tables: the stream it is ordered on, and what says that it has arrived (null: it has)
  hipStream_t stream = nullptr;
  std::atomic<Staging *> staging{nullptr};
  uint32_t upload = 0;
};

// Before anything is enqueued on s: the tables are there, or will be by the order of s.  A captured launch runs at another time
// and maybe on another stream, so for a capture they have to be there.
static dq_status await_tables(dq_replay *r, hipStream_t s) {
  Staging *staging = r->staging.load(std::memory_order_acquire);
  if (!staging) return DQ_OK;
  auto arrived = [&] { return staging->arrived(r->upload); };
  if (!arrived()) {
    bool captured;
    const hipError_t e = dq::is_captured(s, &captured);
    if (e != hipSuccess) return dq::hip_status(e);
    if (s == r->stream && !captured) return DQ_OK;
    for (uint32_t spin = 0; spin < 200000 && !arrived(); ++spin) __builtin_ia32_pause();
    if (!arrived() && !captured) {  // long work ahead of it
      const hipError_t d = hipDeviceSynchronize();
      if (d != hipSuccess) return dq::hip_status(d);
    }
    for (uint32_t ms = 0; ms < 60000 && !arrived(); ++ms) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    if (!arrived()) return dq::hip_status(hipErrorNotReady);
  }
  r->staging.store(nullptr, std::memory_order_release);
  return DQ_OK;
}

extern "C" {

size_t dq_replay_scratch_bytes(const dq_ctx *ctx, const dq_replay_desc *desc) {
  Plan p;
  if (build_plan(ctx, desc, nullptr, nullptr, nullptr, &p) != DQ_OK) return 0;
  return p.scratch_bytes;
}

static dq_status create(dq_ctx *ctx, const dq_replay_desc *desc, const void *const *worker_grads, void *scratch, size_t scratch_bytes,
                        float *out, dq_replay **plan_out, const hipStream_t *stream) {
  if (!ctx || !desc || !worker_grads || !scratch || !out || !plan_out) return DQ_EINVAL;
  *plan_out = nullptr;
  if (desc->n_grads != 0 && desc->n_grads != ctx->cfg.n_workers) return DQ_EINVAL;
  if ((reinterpret_cast<uintptr_t>(scratch) & 255u) || (reinterpret_cast<uintptr_t>(out) & 15u)) return DQ_EALIGN;
  for (uint32_t w = 0; w < ctx->cfg.n_workers; ++w) {
    if (!worker_grads[w]) return DQ_EINVAL;
    if (reinterpret_cast<uintptr_t>(worker_grads[w]) & 15u) return DQ_EALIGN;
  }
  dq_replay *r = new (std::nothrow) dq_replay;
  if (!r) return DQ_EINVAL;
  r->ctx = ctx;
  r->codec = desc->codec;
  r->dtype = desc->dtype;
  r->means = desc->mu != nullptr;
  r->all_gather = desc->all_gather != 0;
  r->scratch = static_cast<uint8_t *>(scratch);
  dq_status st = build_plan(ctx, desc, worker_grads, r->scratch, out, &r->plan);
  if (st == DQ_OK && r->plan.scratch_bytes > scratch_bytes) st = DQ_EINVAL;
  if (st != DQ_OK) {
    delete r;
    return st;
  }
  const bool mx = desc->codec != DQ_DYNAMIQ;
  Upload up(r->scratch, stream);
  Plan &p = r->plan;
  if (p.walk) {  // in the order of their offsets
    if (!mx) {
      dq::split_walk(p.paths.data(), desc->dtype, p.tree, p.w, &p.shares);
      up.put(p.paths_off, p.paths.data(), p.paths.size() * sizeof(dq::WalkPath));
      up.put(p.shares_off, p.shares.data(), p.shares.size() * sizeof(dq::WalkShare));
    }
    std::vector<const void *> twice;  // every tensor twice: a ring's order from any worker on is a run of entries
    for (int k = 0; k < 2; ++k) twice.insert(twice.end(), worker_grads, worker_grads + ctx->cfg.n_workers);
    up.put(p.grads_off, twice.data(), twice.size() * sizeof(void *));
    p.w.grads = p.mx.grads = reinterpret_cast<const void *const *>(r->scratch + p.grads_off);
    std::vector<dq::WalkPath>().swap(p.paths);
    std::vector<dq::WalkShare>().swap(p.shares);
  }
  for (Step &s : p.steps)
    for (Launch &L : s.launches) {
      if (L.jobs.empty()) continue;
      if (mx) {
        std::vector<dq::MxJob> t(L.jobs.size());
        for (size_t i = 0; i < t.size(); ++i) {
          const HostJob &j = L.jobs[i];
          t[i] = dq::MxJob{j.in, j.local, j.out, ((uint64_t)j.n_sg[0] + j.n_sg[1] + j.n_sg[2] + j.n_sg[3]) * 256};
        }
        up.put(L.table_off, t.data(), t.size() * sizeof(dq::MxJob));
      } else {
        std::vector<dq::Job> t(L.jobs.size());
        for (size_t i = 0; i < t.size(); ++i) {
          const HostJob &j = L.jobs[i];
          t[i] = dq::make_job(j.in, j.local, j.mu, j.out, j.first_sg, j.n_sg, j.rank);
          t[i].src = j.src;
          t[i].dest = j.dest;
          t[i].back = j.back;
        }
        up.put(L.table_off, t.data(), t.size() * sizeof(dq::Job));
      }
      std::vector<HostJob>().swap(L.jobs);
    }
  Staging *staging = nullptr;
  if ((st = up.finish(&staging, &r->upload)) != DQ_OK) {
    delete r;
    return st;
  }
  if (stream) r->stream = *stream;
  r->staging = staging;
  *plan_out = r;
  return DQ_OK;
}

dq_status dq_replay_create(dq_ctx *ctx, const dq_replay_desc *desc, const void *const *worker_grads, void *scratch,
                           size_t scratch_bytes, float *out, dq_replay **plan) {
  return create(ctx, desc, worker_grads, scratch, scratch_bytes, out, plan, nullptr);
}

dq_status dqx_replay_create(dq_ctx *ctx, const dq_replay_desc *desc, const void *const *worker_grads, void *scratch, size_t scratch_bytes,
                            float *out, dq_replay **plan, void *hip_stream) {
  const hipStream_t s = (hipStream_t)hip_stream;
  bool captured;
  const hipError_t e = dq::is_captured(s, &captured);
  if (e != hipSuccess) return dq::hip_status(e);
  if (captured) return dq::hip_status(hipErrorStreamCaptureUnsupported);  // the tables are sent once, now
  return create(ctx, desc, worker_grads, scratch, scratch_bytes, out, plan, &s);
}

uint32_t dq_replay_n_steps(const dq_replay *plan) { return plan ? (uint32_t)plan->plan.steps.size() : 0; }

dq_status dq_replay_step_info(const dq_replay *plan, uint32_t step, uint32_t *kind, uint64_t *entries_dar,
                              uint64_t *entries_other) {
  if (!plan || step >= plan->plan.steps.size()) return DQ_EINVAL;
  uint64_t dar = 0, other = 0;
  uint32_t k = 0;
  bool has_dar = false, has_da = false, has_c = false;
  for (const Launch &L : plan->plan.steps[step].launches) {
    if (L.kind == dq::kDar) { dar += L.entries; has_dar = true; }
    else { other += L.entries; (L.kind == dq::kCompress ? has_c : has_da) = true; }
  }
  k = has_dar ? (has_da ? 3 : 1) : (has_c ? 0 : 2);
  if (kind) *kind = k;
  if (entries_dar) *entries_dar = dar;
  if (entries_other) *entries_other = other;
  return DQ_OK;
}

// only: -1 = every launch of the step, else the index of the one launch to enqueue
static dq_status run_step(dq_replay *plan, size_t i, hipStream_t s, int only = -1) {
  const bool mx = plan->codec != DQ_DYNAMIQ;
  int index = -1;
  for (const Launch &L : plan->plan.steps[i].launches) {
    ++index;
    if (only >= 0 && index != only) continue;
    if (L.n_jobs == 0) continue;
    hipError_t e;
    if (mx)
      e = dq::mx_launch_batch(L.kind, plan->codec, L.dtype, L.has_local,
                              reinterpret_cast<const dq::MxJob *>(plan->scratch + L.table_off),
                              L.n_jobs, L.max_entries, plan->ctx->n_cu, s);
    else
      e = dq::launch_batch(L.kind, L.dtype, L.has_local, L.gather, reinterpret_cast<const dq::Job *>(plan->scratch + L.table_off),
                           L.n_jobs, L.max_tiles, plan->ctx->params, plan->ctx->grid_blocks, s);
    if (e != hipSuccess) return dq::hip_status(e);
  }
  return DQ_OK;
}

// Before step `first` is enqueued on its own: what it reads is there.  After a whole replay in one launch the buffers of
// a butterfly and of an all-gather hold an older replay's content, so the schedule is run step by step once, which leaves them as a
// replay in steps would have, and then the steps that have been run since.
static dq_status fill_buffers(dq_replay *r, uint32_t first, hipStream_t s) {
  const size_t ns = r->plan.steps.size();
  if (r->complete || first <= r->filled || (r->all_gather && (first + 2 == ns || (first + 1 == ns && r->gathered)))) return DQ_OK;
  const size_t again = r->filled;
  for (size_t i = 0; i < ns + again; ++i) {
    const dq_status st = run_step(r, i < ns ? i : i - ns, s);
    if (st != DQ_OK) return st;
  }
  bool captured;
  const hipError_t e = dq::is_captured(s, &captured);
  if (e == hipSuccess && !captured) r->complete = true;
  return dq::hip_status(e);
}
// After steps first .. end-1 have been enqueued.
static dq_status note_steps(dq_replay *r, uint32_t first, uint32_t end, hipStream_t s) {
  if (r->complete) return DQ_OK;
  bool captured;
  const hipError_t e = dq::is_captured(s, &captured);
  if (e != hipSuccess || captured) return dq::hip_status(e);  // captured: they have not run
  const uint32_t ns = (uint32_t)r->plan.steps.size();
  if (first + 2 <= ns && end + 1 >= ns) r->gathered = true;
  if (first <= r->filled && end > r->filled) r->filled = end;
  if (r->filled == ns) r->complete = true;
  return DQ_OK;
}

// The whole schedule in one launch.
static dq_status run_walk(dq_replay *r, hipStream_t s) {
  const Plan &p = r->plan;
  const bool complete = p.ring_chunks != 0 && !r->all_gather;
  if (r->complete != complete || r->filled || r->gathered) {
    bool captured;
    const hipError_t e = dq::is_captured(s, &captured);
    if (e != hipSuccess) return dq::hip_status(e);
    if (!captured) {
      r->complete = complete;
      r->filled = 0;
      r->gathered = false;
    }
  }
  if (r->codec != DQ_DYNAMIQ) return dq::hip_status(dq::launch_mx_walk(r->codec, r->dtype, p.tree, p.mx, r->ctx->n_cu, s));
  return dq::hip_status(dq::launch_walk(r->dtype, p.tree, r->means, reinterpret_cast<const dq::WalkPath *>(r->scratch + p.paths_off),
                                        reinterpret_cast<const dq::WalkShare *>(r->scratch + p.shares_off), p.w, r->ctx->params, s));
}

dq_status dq_replay_run_steps(dq_replay *plan, uint32_t first, uint32_t count, void *hip_stream) {
  if (!plan || (size_t)first + count > plan->plan.steps.size()) return DQ_EINVAL;
  const dq_status ready = await_tables(plan, (hipStream_t)hip_stream);
  if (ready != DQ_OK) return ready;
  if (plan->plan.walk && count == plan->plan.steps.size()) return run_walk(plan, (hipStream_t)hip_stream);
  if (count == 0) return DQ_OK;
  dq_status st = fill_buffers(plan, first, (hipStream_t)hip_stream);
  for (uint32_t i = first; i < first + count && st == DQ_OK; ++i) st = run_step(plan, i, (hipStream_t)hip_stream);
  return st == DQ_OK ? note_steps(plan, first, first + count, (hipStream_t)hip_stream) : st;
}

dq_status dq_replay_run_launch(dq_replay *plan, uint32_t step, uint32_t launch, void *hip_stream) {
  if (!plan || step >= plan->plan.steps.size() || launch >= plan->plan.steps[step].launches.size()) return DQ_EINVAL;
  const dq_status ready = await_tables(plan, (hipStream_t)hip_stream);
  if (ready != DQ_OK) return ready;
  dq_status st = fill_buffers(plan, step, (hipStream_t)hip_stream);
  if (st == DQ_OK) st = run_step(plan, step, (hipStream_t)hip_stream, (int)launch);
  const bool done = launch + 1 == plan->plan.steps[step].launches.size();
  return st == DQ_OK && done ? note_steps(plan, step, step + 1, (hipStream_t)hip_stream) : st;
}

dq_status dq_replay_run(dq_replay *plan, float *step_ms, void *hip_stream) {
  if (!plan) return DQ_EINVAL;
  hipStream_t s = (hipStream_t)hip_stream;
  const size_t ns = plan->plan.steps.size();
  const dq_status ready = await_tables(plan, s);
  if (ready != DQ_OK) return ready;
  if (plan->plan.walk && !step_ms) return run_walk(plan, s);
  hipError_t he = hipSuccess;
  while (step_ms && he == hipSuccess && plan->events.size() < ns + 1) {
    hipEvent_t e;
    he = hipEventCreate(&e);
    if (he == hipSuccess) plan->events.push_back(e);
  }
  if (step_ms && he == hipSuccess) he = hipEventRecord(plan->events[0], s);
  for (size_t i = 0; i < ns && he == hipSuccess; ++i) {
    const dq_status st = run_step(plan, i, s);
    if (st != DQ_OK) return st;
    if (step_ms) he = hipEventRecord(plan->events[i + 1], s);
  }
  if (he == hipSuccess) {
    const dq_status st = note_steps(plan, 0, (uint32_t)ns, s);
    if (st != DQ_OK) return st;
  }
  if (step_ms && he == hipSuccess) he = hipEventSynchronize(plan->events[ns]);
  for (size_t i = 0; step_ms && i < ns && he == hipSuccess; ++i)
    he = hipEventElapsedTime(&step_ms[i], plan->events[i], plan->events[i + 1]);
  return dq::hip_status(he);
}

dq_status dq_replay_message(const dq_replay *plan, uint32_t step, uint32_t bucket, uint32_t chunk, const void **ptr,
                            size_t *bytes) {
  if (!plan || !ptr || !bytes) return DQ_EINVAL;
  const Plan &p = plan->plan;
  if (p.ring_chunks == 0) return DQ_EUNSUPPORTED;
  const size_t i = (size_t)bucket * p.ring_chunks + chunk;
  if (step >= p.ring_message_steps || chunk >= p.ring_chunks || i >= p.ring_slot.size()) return DQ_EINVAL;
  *ptr = p.ring_msg[step & 1] + p.ring_slot[i];
  *bytes = p.ring_bytes[i];
  return DQ_OK;
}

void dq_replay_destroy(dq_replay *plan) {
  if (!plan) return;
  for (hipEvent_t e : plan->events) (void)hipEventDestroy(e);
  delete plan;
}

}  // extern "C"

// ---- a whole simulated all-reduce on the original tensors, enqueued without waiting: statistics, search, then (arrange) means, origins and the
// tables of the replay, then the replay.  The host never needs the class counts to go on: how many waves there are follows from the
// schedule's super-groups, and which tiles each takes is worked out on the device.  With the counts sent to the host and the plan made there the GPU
// waited 15 us for it, and 5.4 for the tables' upload: 8 workers' ring of 8,192 super-groups in bf16 58.1 -> 36.3 us, 16 workers' of 1,936 60.9 -> 32.2,
// recursive halving over 2 of 30,416 61.4 -> 42.2.
namespace {
struct WholePlan {
  dq::WalkGrid w = {};
  dq::Tables t = {};
  size_t paths = 0, shares = 0, grads = 0, mu = 0, F = 0, places = 0, counts = 0, mu_main = 0, origin = 0, bytes = 0;
};
// False: not for these kernels.
bool plan_whole(const dq_ctx *ctx, const dqx_whole *d, WholePlan *p) {
  const uint32_t n = ctx->cfg.n_workers, J = d->n_sg_bucket, nb = d->n_buckets;
  const bool tree = d->topology == DQ_BUTTERFLY;
  if ((d->topology != DQ_RING && !tree) || (d->dtype != DQ_F32 && d->dtype != DQ_BF16) || n < 2 || n > dq::kMostTensors || d->n_tensors != n || J == 0 || nb == 0 || nb > dq::kAnnounced || J % n ||
      (tree && (n & (n - 1))) || J > dq::kMostSearched || (uint64_t)n * nb > dq::kMostTablePaths || (d->max_width != 8 && d->max_width != 16) ||
      d->max_code_bits < 2ull * J)
    return false;
  const uint32_t m = J / n;
  dq::WalkGrid &w = p->w;
  describe(n, d->topology, d->all_gather != 0, &w);
  w.first_kept = n - 1;  // nobody asks for messages
  w.raw = d->max_width == 16;
  w.n_paths = n * nb;
  // at most: a bucket's three edges between widths each begin a tile anew
  const uint64_t tiles[3] = {(uint64_t)J * nb, (uint64_t)nb * (n * ((m + 1) / 2) + 3), (uint64_t)nb * (n * ((m + 3) / 4) + 3)};
  if (!dq::grid_walk(ctx->params, d->dtype, tree, ctx->n_cu, tiles, &w)) return false;
  dq::Tables &t = p->t;
  t.n_chunks = n;
  t.n_buckets = nb;
  t.chunk_sgs = m;
  t.bucket_sgs = J;
  t.by_chunk = by_chunk_number(w, nb, J);
  t.entry_bytes = (uint32_t)elt_size(d->dtype);
  // A tile per wave at most, found by counting, which takes the arrange launch or the search before it 1 to 3 us less than weighing the tiles.  Not where the waves that a
  // path's one to three tiles fewer leave without one are more than a 16th; nor, over more than eight workers and unless they are less than a 96th, where they give some CU a
  // block more than the fullest has without them, or fill the last round of CUs: the fullest CU is what a replay waits for, hop by hop.  All-reduces, us, weighed and counted:
  // tiles of one super-group 6 % faster counted on average of 3,618; of two and four, without a block more 7 % (931, three of them 2 to 5 % slower), with one 6 % inside this line
  // (828, 20 of them 2 to 5 % slower) and outside, of 2,633, 10 % faster to 18 % slower (fp32 ring of 57, 2 x 5,529: 714 blocks, counted 798, 227 and 269; of 37, 12,062 up
  // to 16 bits 760, 787, 165 and 199; bf16 of 16 by halves, 5 x 1,664 up to 16 bits: 262 and 290 blocks, 55.2 and 58.2; but of 8, 8,160 511 and 516, 35.1 and 31.8).
  const uint64_t each = (m + w.tile_sgs - 1) / w.tile_sgs, slots = w.tile_sgs == 1 ? each : each + 3, slot_blocks = (slots * w.n_paths + w.waves - 1) / w.waves;
  const bool fuller = (slot_blocks - 1) / ctx->n_cu != (w.blocks - 1) / ctx->n_cu || slot_blocks / ctx->n_cu != w.blocks / ctx->n_cu;
  if (slot_blocks <= w.most_blocks && slots <= each + each / (fuller && n > 8 ? 96 : 16)) {
    t.slots = (uint32_t)slots;
    w.blocks = (uint32_t)slot_blocks;
  }
  t.waves = w.blocks * w.waves;
  t.tile_log = w.tile_sgs / 2;
  t.cost = dq::costs_of(d->dtype, tree, n, w.tile_sgs);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off = align_up(off + bytes, 256);
    return at;
  };
  const size_t sgs = (size_t)J * nb;
  p->paths = take(w.n_paths * sizeof(dq::WalkPath));
  p->shares = take(((size_t)t.waves + 1) * sizeof(dq::WalkShare));
  p->grads = take(2 * (size_t)n * sizeof(void *));
  p->mu = take(4 * sgs);
  p->F = take(4 * sgs);
  p->places = take(4 * sgs);
  p->counts = take(20 * (size_t)nb);
  p->mu_main = take(4 * sgs);
  p->origin = take(4 * sgs);
  p->bytes = off;
  return true;
}
}  // namespace

extern "C" {

size_t dqx_whole_scratch_bytes(const dq_ctx *ctx, const dqx_whole *desc) {
  WholePlan p;
  return ctx && desc && plan_whole(ctx, desc, &p) ? p.bytes : 0;
}

dq_status dqx_whole_tables(const dq_ctx *ctx, const dqx_whole *desc, dqx_tables *tables) {
  WholePlan p;
  if (!ctx || !desc || !tables || !plan_whole(ctx, desc, &p)) return DQ_EINVAL;
  *tables = dqx_tables{p.shares, p.w.blocks, p.w.waves, p.w.tile_sgs, p.t.by_chunk};
  return DQ_OK;
}

dq_status dqx_whole_run(const dq_ctx *ctx, const dqx_whole *desc, const void *const *tensors, void *scratch, float *out, void *hip_stream, void **ticket) {
  WholePlan p;
  *ticket = nullptr;
  if (!ctx || !desc || !tensors || !scratch || !out || !plan_whole(ctx, desc, &p)) return DQ_EINVAL;
  if ((reinterpret_cast<uintptr_t>(scratch) & 255u) || (reinterpret_cast<uintptr_t>(out) & 15u)) return DQ_EALIGN;
  uint8_t *const base = static_cast<uint8_t *>(scratch);
  auto floats = [&](size_t at) { return reinterpret_cast<float *>(base + at); };
  auto words = [&](size_t at) { return reinterpret_cast<uint32_t *>(base + at); };
  const hipStream_t s = (hipStream_t)hip_stream;
  const uint32_t J = desc->n_sg_bucket, nb = desc->n_buckets;
  const bool means = desc->means != 0;
  dq::Announce announce = {nullptr, 0};
  const hipError_t e = dq::announce_begin(nb, s, &announce, ticket);
  if (e != hipSuccess) return dq::hip_status(e);
  p.t.paths = reinterpret_cast<dq::WalkPath *>(base + p.paths);
  p.t.shares = reinterpret_cast<dq::WalkShare *>(base + p.shares);
  p.t.out = out;
  p.t.origin = words(p.origin);
  p.t.mu = means ? floats(p.mu_main) : nullptr;
  const void **grads = reinterpret_cast<const void **>(base + p.grads);
  p.w.grads = grads;
  bool searched = false;
  dq_status st = *ticket ? dq::stats_all(tensors, ctx->cfg.n_workers, desc->dtype, (uint64_t)J * nb, floats(p.mu), floats(p.F), grads, s) : DQ_EINVAL;
  const bool both = dq::takes_search_arrange(J, nb, p.t);
  if (st == DQ_OK && both) {
    searched = true;
    st = dq::search_arrange(floats(p.F), means ? floats(p.mu) : nullptr, J, desc->max_code_bits, desc->max_width, words(p.places),
                            means ? floats(p.mu_main) : nullptr, words(p.origin), announce, p.t, s);
  } else if (st == DQ_OK) {
    searched = true;
    st = dq::search(floats(p.F), J, nb, desc->max_code_bits, desc->max_width, words(p.places), words(p.counts), announce, s);
  }
  if (st == DQ_OK && !both)
    st = dq::arrange(floats(p.F), means ? floats(p.mu) : nullptr, J, nb, desc->max_width, words(p.counts), words(p.places),
                     means ? floats(p.mu_main) : nullptr, words(p.origin), p.t, s);
  if (st == DQ_OK)
    st = dq::hip_status(dq::launch_walk(desc->dtype, desc->topology == DQ_BUTTERFLY, means, p.t.paths, p.t.shares, p.w, ctx->params, s));
  if (st != DQ_OK && *ticket) {  // a search that runs still writes to the ticket's workspace: its counts are waited for
    std::vector<uint32_t> rows(4 * (size_t)nb);
    if (searched) (void)dqx_allocate_end(*ticket, J, nb, rows.data(), hip_stream);
    else dq::announce_drop(*ticket);
    *ticket = nullptr;
  }
  return st;
}

}  // extern "C"
