/* Stands in for the HIP runtime's launches where there is no GPU: loaded in front of it, it notes every launch's grid, block and first
 * arguments, and refuses what HIP refuses, 2^32 or more threads along a dimension. */
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct {
  uint32_t grid[3], block[3];
  uint64_t args[8]; /* the first args_taken, as 8 bytes each */
} launch_t;

static launch_t launches[4096];
static int n_launches, failed;
int args_taken = 0; /* of a launch, at most eight: the kernels have as many */
static struct { dim3_t grid, block; size_t shared; void *stream; } pushed;

int recorded(launch_t *out, int most) {
  const int n = n_launches < most ? n_launches : most;
  memcpy(out, launches, (size_t)n * sizeof(launch_t));
  n_launches = 0;
  return n;
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void *stream) {
  pushed.grid = grid; pushed.block = block; pushed.shared = shared; pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *shared, void **stream) {
  *grid = pushed.grid; *block = pushed.block; *shared = pushed.shared; *stream = pushed.stream;
  return 0;
}
int hipLaunchKernel(const void *kernel, dim3_t grid, dim3_t block, void **args, size_t shared, void *stream) {
  (void)kernel; (void)shared; (void)stream;
  const uint64_t limit = 1ull << 32;
  if ((uint64_t)grid.x * block.x >= limit || (uint64_t)grid.y * block.y >= limit || (uint64_t)grid.z * block.z >= limit) return failed = 9;
  if (n_launches < (int)(sizeof(launches) / sizeof(launches[0]))) {
    launch_t *l = &launches[n_launches++];
    l->grid[0] = grid.x; l->grid[1] = grid.y; l->grid[2] = grid.z;
    l->block[0] = block.x; l->block[1] = block.y; l->block[2] = block.z;
    for (int i = 0; i < args_taken; ++i) memcpy(&l->args[i], args[i], 8);
  }
  return 0;
}
int hipGetLastError(void) {
  const int e = failed;
  failed = 0;
  return e;
}
