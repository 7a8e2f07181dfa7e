// What the Python binding needs beside the C ABI: a bounds check of super-group indices, and a few words brought to the host.
//
// The bounds check: the binding, unlike the C ABI, knows how large the tensor is that
// the indices point into.  The check is one small launch in front of the call on the same
// stream; the call's kernel starts by reading the verdict and does nothing if an index is out of bounds,
// so the host can enqueue it without waiting and only then look at the verdict, which arrives in pinned host memory
// while the call runs.  (Reductions on the stream, each waited for on the host before the call was enqueued, took 38 us
// per index and left the GPU idle between calls.)
#include <string.h>

#include <mutex>
#include <vector>

#include "dq_bounds.h"
#include "dq_device.h"

namespace dq {
namespace {

constexpr uint32_t kSlots = 256;  // calls a workspace serves before its slots are used again
struct Slot {
  uint32_t found, guard;
};
struct Workspace {
  Slot *slots = nullptr;      // device, zero at rest
  uint32_t *host = nullptr;   // pinned: the last verdict, 4 * call number + [first array out of bounds] + 2 * [second]
  uint32_t calls = 0;
  int device = -1;
};

// Workspaces at rest (2 KB each), one for every call that was ever waiting at the same time as others, kIdle of them at most.
constexpr size_t kIdle = 8;
std::mutex g_mutex;
std::vector<Workspace *> g_idle;

thread_local Workspace *t_armed = nullptr;
thread_local const uint32_t *t_guard = nullptr;

// What bounds it is latency: eight indices per thread, all loaded before the first is looked at, and one atomic
// per block, blocks done in its low ten bits, those that found something in the two fields above.  (Findings in a word of their
// own needed a fence per block, a write-back of the L2, and took 10 us for 488,282 indices, 6.4.)
constexpr uint32_t kPerThread = 8, kMaxBlocks = 512;
__global__ void __launch_bounds__(256) k_bounds(Bound a, Bound b, Slot *slot, uint32_t *host, uint32_t call) {
  auto outside = [](const Bound &x) {
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
    return x.n != 0 && most >= x.limit;
  };
  const bool out_a = outside(a), out_b = outside(b);
  const int bad_a = __syncthreads_or(out_a), bad_b = __syncthreads_or(out_b);
  if (threadIdx.x != 0) return;
  const uint32_t mine = 1u + (bad_a ? 1u << 10 : 0u) + (bad_b ? 1u << 20 : 0u), all = atomicAdd(&slot->found, mine) + mine;
  if ((all & 0x3FFu) != gridDim.x) return;
  const uint32_t verdict = ((all >> 10 & 0x3FFu) ? 1u : 0u) + (all >> 20 ? 2u : 0u);
  slot->found = 0;  // the next kernels on the stream see these two as they see any store
  slot->guard = verdict;
  __hip_atomic_store(host, 4 * call + verdict, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // nothing else to order
}

// A few words to pinned host memory, then the call number in front of them.
__global__ void __launch_bounds__(256) k_fetch(const uint32_t *src, uint32_t n, uint32_t *host, uint32_t call) {
  for (uint32_t i = threadIdx.x; i < n; i += 256) __hip_atomic_store(host + 1 + i, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __threadfence_system();
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(host, 4 * call, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);  // fenced above
}

Workspace *take(hipError_t *err) {
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
  Workspace *w = new Workspace;
  w->device = device;
  if ((*err = hipMalloc((void **)&w->slots, kSlots * sizeof(Slot))) != hipSuccess ||
      (*err = hipMemset(w->slots, 0, kSlots * sizeof(Slot))) != hipSuccess ||
      (*err = hipHostMalloc((void **)&w->host, 4 * (1 + kFetchWords), hipHostMallocDefault)) != hipSuccess) {
    if (w->slots) (void)hipFree(w->slots);
    delete w;
    return nullptr;
  }
  *w->host = 0;
  return w;
}

void drop(Workspace *w) {
  (void)hipFree(w->slots);
  (void)hipHostFree(w->host);
  delete w;
}

}  // namespace

const uint32_t *armed_guard() { return t_guard; }

}  // namespace dq

extern "C" {

static hipError_t await_call(dq::Workspace *w, void *hip_stream, uint32_t *word_out) {
  volatile uint32_t *word = w->host;
  hipError_t e = hipSuccess;
  for (uint32_t spin = 0;; ++spin) {
    *word_out = __atomic_load_n(word, __ATOMIC_ACQUIRE);
    if (*word_out >> 2 == (w->calls & 0x3FFFFFFFu)) break;
    if (spin > 200000) {  // long work ahead on the stream, or an error there: wait in the runtime
      e = hipStreamSynchronize((hipStream_t)hip_stream);
      *word_out = __atomic_load_n(word, __ATOMIC_ACQUIRE);
      break;
    }
    __builtin_ia32_pause();
  }
  return e;
}
static void give_back(dq::Workspace *w) {
  {
    std::lock_guard<std::mutex> lock(dq::g_mutex);
    if (dq::g_idle.size() < dq::kIdle) {
      dq::g_idle.push_back(w);
      return;
    }
  }
  dq::drop(w);
}

dq_status dqx_bounds_begin(const dq::Bound *bounds, int n_bounds, void *hip_stream) {
  hipError_t e = hipSuccess;
  dq::Workspace *w = dq::take(&e);
  if (!w) return dq::hip_status(e);
  ++w->calls;
  if (w->calls % dq::kSlots == 0) (void)hipDeviceSynchronize();  // a slot is read by its own call only: let all of them finish
  dq::Slot *slot = w->slots + w->calls % dq::kSlots;
  const dq::Bound a = bounds[0], b = n_bounds > 1 ? bounds[1] : dq::Bound{nullptr, 0, 0};
  const uint32_t most = a.n > b.n ? a.n : b.n;
  uint32_t blocks = (most + 256 * dq::kPerThread - 1) / (256 * dq::kPerThread);
  if (blocks > dq::kMaxBlocks) blocks = dq::kMaxBlocks;
  hipLaunchKernelGGL(dq::k_bounds, dim3(blocks ? blocks : 1), dim3(256), 0, (hipStream_t)hip_stream, a, b, slot, w->host, w->calls);
  e = hipGetLastError();
  if (e != hipSuccess) {
    give_back(w);
    return dq::hip_status(e);
  }
  dq::t_armed = w;
  dq::t_guard = &slot->guard;
  return DQ_OK;
}

dq_status dqx_bounds_end(void *hip_stream, int *out_of_bounds) {
  dq::Workspace *w = dq::t_armed;
  dq::t_armed = nullptr;
  dq::t_guard = nullptr;
  if (!w) return DQ_EINVAL;
  uint32_t word = 0;
  const hipError_t e = await_call(w, hip_stream, &word);
  *out_of_bounds = (int)(word & 3u);
  give_back(w);
  return dq::hip_status(e);
}

dq_status dqx_fetch(const uint32_t *src, uint32_t n, uint32_t *dst, void *hip_stream) {
  if (n > dq::kFetchWords) return DQ_EUNSUPPORTED;
  hipError_t e = hipSuccess;
  dq::Workspace *w = dq::take(&e);
  if (!w) return dq::hip_status(e);
  ++w->calls;
  hipLaunchKernelGGL(dq::k_fetch, dim3(1), dim3(256), 0, (hipStream_t)hip_stream, src, n, w->host, w->calls);
  e = hipGetLastError();
  uint32_t word = 0;
  if (e == hipSuccess) e = await_call(w, hip_stream, &word);
  if (e == hipSuccess) memcpy(dst, w->host + 1, 4 * (size_t)n);
  give_back(w);
  return dq::hip_status(e);
}

}  // extern "C"
