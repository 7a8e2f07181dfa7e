// Between libdq and its Python binding (not part of the C ABI): see dq_bounds.hip.
#pragma once
#include <stdint.h>

#include "dq.h"

namespace dq {
struct Bound {
  const uint32_t *index;  // device
  uint32_t n, limit;      // every index must be below limit
};
const uint32_t *armed_guard();     // this thread's armed verdict (device), or null
void bounds_context(int change);   // a context was made (1) or destroyed (-1)
}  // namespace dq

extern "C" {
// Enqueue the check of one or two index arrays and arm its verdict for the calls this thread makes until
// dqx_bounds_end, which waits for it (bit k: array k has an index out of bounds).  The calls in between do nothing
// if a bit is set.
dq_status dqx_bounds_begin(const dq::Bound *bounds, int n_bounds, void *hip_stream);
dq_status dqx_bounds_end(void *hip_stream, int *out_of_bounds);
}
