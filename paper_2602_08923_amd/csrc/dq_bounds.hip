// What the Python binding needs beside the C ABI: a bounds check of super-group indices, and a few words brought to the host.
//
// The bounds check: the binding, unlike the C ABI, knows how large the tensor is that
// the indices point into.  The host enqueues check and call without waiting and only then looks at the verdict, which arrives in pinned
// host memory while the call runs.  A call on few super-groups checks all its indices itself, in every block, beside the trips that
// the block waits for anyway (dq_few.hip).  For others the check is one small launch in front of the call on the same stream; the call's
// kernel starts by reading the verdict and does nothing if an index is out of bounds.
// (Reductions on the stream, each waited for on the host before the call was enqueued, took 38 us
// per index and left the GPU idle between calls.)
#include <string.h>

#include <mutex>
#include <new>
#include <vector>

#include "dq_bounds.h"
#include "dq_device.h"

namespace dq {
namespace {

// A workspace belongs to one call at a time, from its enqueueing until its verdict has come, and goes to the next call, maybe on
// another stream, as it is: nothing in it is reset, and the kernels of earlier calls may still look at `refused`.
struct Tally {
  unsigned long long done;  // blocks of all calls that have finished (kDoneBits), and above them those of this call that found something
  uint32_t refused;         // the last call that had an index out of bounds; a call's kernels do nothing if it is theirs
};
struct Workspace {
  Tally *tally = nullptr;    // device
  uint32_t *host = nullptr;  // pinned: the last verdict, 4 * call number + [first array out of bounds] + 2 * [second]
  uint32_t calls = 0;
  uint64_t done = 0;         // blocks of all calls so far
  int device = -1;
};
constexpr uint32_t kDoneBits = 40, kLastCall = (1u << 30) - 1;  // a workspace is retired before either count runs over

// Workspaces at rest (4 KB each), one for every call that was ever waiting at the same time as others, kIdle of them at most.
constexpr size_t kIdle = 8;
std::mutex g_mutex;
std::vector<Workspace *> g_idle;

struct Armed {
  Workspace *w = nullptr;
  Bound a, b;
  bool started = false;  // enqueued, or left to the call's kernel
};
thread_local Armed t_armed;

// A restore of what was gathered by the same array names it twice; it is read once (488,282 indices:
// the restore behind the check 186.35 -> 186.0 us).
// What bounds it is latency: eight indices per thread, all loaded before the first is looked at, and one atomic
// per block, which also says whether it found something.  (Findings in a word of their
// own needed a fence per block, a write-back of the L2, and took 10 us for 488,282 indices, 6.4.)
constexpr uint32_t kPerThread = 8, kMaxBlocks = 512;
constexpr uint32_t kBadA = kDoneBits, kBadB = kDoneBits + 12;  // fields of 12 bits for at most kMaxBlocks each
__global__ void k_clear(Tally *tally) { *tally = Tally{0, 0}; }
__global__ void __launch_bounds__(256) k_bounds(Bound a, Bound b, Tally *tally, uint32_t *host, uint32_t call, uint64_t last) {
  auto largest = [](const Bound &x) {
    const uint32_t stride = gridDim.x * 256;
    uint32_t most = 0;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < x.n; i += kPerThread * stride) {
      uint32_t v[kPerThread];
#pragma unroll
      for (uint32_t k = 0; k < kPerThread; ++k) {
        const uint64_t at = i + (uint64_t)k * stride;
        v[k] = x.index[at < x.n ? (uint32_t)at : i];
      }
#pragma unroll
      for (uint32_t k = 0; k < kPerThread; ++k) most = v[k] > most ? v[k] : most;
    }
    return most;
  };
  const uint32_t most_a = largest(a), most_b = same_array(a, b) ? most_a : largest(b);
  const bool out_a = a.n != 0 && most_a >= a.limit, out_b = b.n != 0 && most_b >= b.limit;
  const int bad_a = __syncthreads_or(out_a), bad_b = __syncthreads_or(out_b);
  if (threadIdx.x != 0) return;
  const unsigned long long mine = 1ull + (bad_a ? 1ull << kBadA : 0ull) + (bad_b ? 1ull << kBadB : 0ull);
  const unsigned long long all = atomicAdd(&tally->done, mine) + mine;
  if ((all & ((1ull << kDoneBits) - 1)) != last) return;
  const unsigned long long bad = all >> kDoneBits << kDoneBits;
  uint32_t verdict = 0;
  if (bad) {
    verdict = (all >> kBadA & 0xFFFu ? 1u : 0u) + (all >> kBadB ? 2u : 0u);
    atomicAdd(&tally->done, 0ull - bad);
    tally->refused = call;  // the next kernel on the stream sees it as it sees any store; the host waits for the stream
  }
  __hip_atomic_store(host, 4 * call + verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // nothing else to order
}

// A few words to pinned host memory, then the call number in front of them.
__global__ void __launch_bounds__(256) k_fetch(const uint32_t *src, uint32_t n, uint32_t *host, uint32_t call) {
  for (uint32_t i = threadIdx.x; i < n; i += 256) __hip_atomic_store(host + 1 + i, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(host, 4 * call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // fenced above
}

// One for a call on stream s, which must not be under capture: a captured check would run again, with this call's number.
Workspace *take(hipStream_t s, hipError_t *err) {
  bool captured;
  if ((*err = is_captured(s, &captured)) != hipSuccess) return nullptr;
  if (captured) {
    *err = hipErrorStreamCaptureUnsupported;
    return nullptr;
  }
  int device = -1;
  if ((*err = hipGetDevice(&device)) != hipSuccess) return nullptr;
  {
    std::lock_guard<std::mutex> lock(g_mutex);
    for (size_t i = 0; i < g_idle.size(); ++i)
      if (g_idle[i]->device == device) {
        Workspace *w = g_idle[i];
        g_idle.erase(g_idle.begin() + i);
        return w;
      }
  }
  Workspace *w = new (std::nothrow) Workspace;
  if (!w) {
    *err = hipErrorOutOfMemory;
    return nullptr;
  }
  w->device = device;
  if ((*err = hipMalloc((void **)&w->tally, sizeof(Tally))) != hipSuccess ||
      (*err = hipHostMalloc((void **)&w->host, 4 * (1 + kFetchWords), hipHostMallocDefault)) != hipSuccess) {
    if (w->tally) (void)hipFree(w->tally);
    delete w;
    return nullptr;
  }
  *w->host = 0;
  // ahead of the first call on its own stream; other streams meet the workspace only after that call's verdict
  hipLaunchKernelGGL(k_clear, dim3(1), dim3(1), 0, s, w->tally);
  *err = hipGetLastError();
  return *err == hipSuccess ? w : nullptr;
}

// After a call whose verdict has come.  (After an error something may still write to the workspace: it is left alone for good.)
void give_back(Workspace *w) {
  if (w->calls < kLastCall && w->done < 1ull << (kDoneBits - 1)) {
    std::lock_guard<std::mutex> lock(g_mutex);
    if (g_idle.size() < kIdle) {
      g_idle.push_back(w);
      return;
    }
  }
  (void)hipFree(w->tally);  // waits for the kernels that look at it
  (void)hipHostFree(w->host);
  delete w;
}

// The verdict of w's last call.
hipError_t await_call(Workspace *w, hipStream_t s, uint32_t *word) {
  for (uint32_t spin = 0; spin < 200000; ++spin) {
    *word = __atomic_load_n(w->host, __ATOMIC_ACQUIRE);
    if (*word >> 2 == w->calls) return hipSuccess;
    __builtin_ia32_pause();
  }
  const hipError_t e = hipStreamSynchronize(s);  // long work ahead on the stream, or an error there
  if (e != hipSuccess) return e;
  *word = __atomic_load_n(w->host, __ATOMIC_ACQUIRE);
  return *word >> 2 == w->calls ? hipSuccess : hipErrorLaunchFailure;
}

// The armed check as a launch of its own.
hipError_t enqueue_check(hipStream_t s) {
  Workspace *w = t_armed.w;
  const uint32_t most = t_armed.a.n > t_armed.b.n ? t_armed.a.n : t_armed.b.n;
  uint32_t blocks = (most + 256 * kPerThread - 1) / (256 * kPerThread);
  blocks = blocks > kMaxBlocks ? kMaxBlocks : blocks ? blocks : 1;
  w->done += blocks;
  t_armed.started = true;
  hipLaunchKernelGGL(k_bounds, dim3(blocks), dim3(256), 0, s, t_armed.a, t_armed.b, w->tally, w->host, w->calls, w->done);
  return hipGetLastError();
}

}  // namespace

uint64_t own_check_due() {
  const Armed &x = t_armed;
  if (!x.w) return 0;
  return x.started || x.a.limit == 0 || (x.b.n && x.b.limit == 0) ? ~0ull : x.a.n + (same_array(x.a, x.b) ? 0ull : x.b.n);
}

bool take_own_check(const uint32_t *src, OwnCheck *check) {
  Armed &x = t_armed;
  const uint64_t due = own_check_due();
  if (due == 0 || due == ~0ull) return false;
  *check = OwnCheck{x.a, x.b, x.w->host, x.w->calls, src == x.a.index ? x.a.limit : src && src == x.b.index ? x.b.limit : 0xFFFFFFFFu};
  x.started = true;
  return true;
}

hipError_t armed_guard(hipStream_t s, Guard *guard) {
  *guard = Guard{nullptr, 0};
  if (!t_armed.w) return hipSuccess;
  *guard = Guard{&t_armed.w->tally->refused, t_armed.w->calls};
  return t_armed.started ? hipSuccess : enqueue_check(s);
}

// Counts ahead of an allocation.  The host needs nothing of it but how many super-groups have each width; with them it plans the replay,
// meanwhile the GPU writes positions, origins and means.  Fetched by a launch behind the allocation they came 10 us later, and
// what followed was enqueued after the wait.  (An all-reduce that is enqueued whole, dqx_whole_run, only reports them.)
// Their words lie behind the workspace's first two.
static_assert(kAnnounced == (kFetchWords - 1) / 2, "two words each");
static uint64_t *announced(Workspace *w) { return reinterpret_cast<uint64_t *>(w->host + 2); }
static uint32_t tag_of(const Workspace *w) { return w->calls % 8191 + 1; }
hipError_t announce_begin(uint32_t n_buckets, hipStream_t s, Announce *announce, void **ticket) {
  if (n_buckets > kAnnounced) return hipSuccess;
  hipError_t e = hipSuccess;
  Workspace *w = take(s, &e);
  if (!w) return e;
  ++w->calls;
  for (uint32_t b = 0; b < n_buckets; ++b) __atomic_store_n(announced(w) + b, 0, __ATOMIC_RELAXED);
  *announce = Announce{announced(w), tag_of(w)};
  *ticket = w;
  return hipSuccess;
}
void announce_drop(void *ticket) { give_back(static_cast<Workspace *>(ticket)); }

}  // namespace dq

extern "C" {

dq_status dqx_allocate_end(void *ticket, uint32_t J, uint32_t n_buckets, uint32_t *rows, void *hip_stream) {
  dq::Workspace *w = static_cast<dq::Workspace *>(ticket);
  if (!w) return DQ_EINVAL;
  for (uint32_t b = 0, spin = 0; b < n_buckets;) {
    const uint64_t word = __atomic_load_n(dq::announced(w) + b, __ATOMIC_ACQUIRE);
    if (word >> 51 == dq::tag_of(w)) {
      uint32_t *row = rows + 4 * (size_t)b++;
      for (int k = 0; k < 3; ++k) row[k] = (uint32_t)(word >> (17 * k)) & 0x1FFFFu;
      row[3] = J - row[0] - row[1] - row[2];
    } else if (++spin > 200000) {  // long work ahead on the stream, or an error there
      if (spin != 200001) return dq::hip_status(hipErrorLaunchFailure);
      const hipError_t e = hipStreamSynchronize((hipStream_t)hip_stream);
      if (e != hipSuccess) return dq::hip_status(e);
    } else {
      __builtin_ia32_pause();
    }
  }
  dq::give_back(w);
  return DQ_OK;
}

dq_status dqx_bounds_begin(const dq::Bound *bounds, int n_bounds, void *hip_stream) {
  hipError_t e = hipSuccess;
  dq::Workspace *w = dq::take((hipStream_t)hip_stream, &e);
  if (!w) return dq::hip_status(e);
  ++w->calls;
  dq::t_armed = dq::Armed{w, bounds[0], n_bounds > 1 ? bounds[1] : dq::Bound{nullptr, 0, 0}};
  return DQ_OK;
}

dq_status dqx_bounds_end(void *hip_stream, int *out_of_bounds) {
  dq::Workspace *w = dq::t_armed.w;
  if (!w) return DQ_EINVAL;
  hipError_t e = dq::t_armed.started ? hipSuccess : dq::enqueue_check((hipStream_t)hip_stream);  // no call came to it
  dq::t_armed = dq::Armed{};
  uint32_t word = 0;
  if (e == hipSuccess) e = dq::await_call(w, (hipStream_t)hip_stream, &word);
  if (e != hipSuccess) return dq::hip_status(e);
  *out_of_bounds = (int)(word & 3u);
  // the refused call's kernel has read its refusal before another call can be refused
  if (*out_of_bounds && (e = hipStreamSynchronize((hipStream_t)hip_stream)) != hipSuccess) return dq::hip_status(e);
  dq::give_back(w);
  return DQ_OK;
}

dq_status dqx_fetch(const uint32_t *src, uint32_t n, uint32_t *dst, void *hip_stream) {
  if (n > dq::kFetchWords) return DQ_EUNSUPPORTED;
  hipError_t e = hipSuccess;
  dq::Workspace *w = dq::take((hipStream_t)hip_stream, &e);
  if (!w) return dq::hip_status(e);
  ++w->calls;
  hipLaunchKernelGGL(dq::k_fetch, dim3(1), dim3(256), 0, (hipStream_t)hip_stream, src, n, w->host, w->calls);
  uint32_t word = 0;
  if ((e = hipGetLastError()) != hipSuccess || (e = dq::await_call(w, (hipStream_t)hip_stream, &word)) != hipSuccess) return dq::hip_status(e);
  memcpy(dst, w->host + 1, 4 * (size_t)n);
  dq::give_back(w);
  return DQ_OK;
}

}  // extern "C"
