/* What rehyat_phi_backward launches, without a GPU: the few runtime entry points that a launch passes through
 * are defined here and take the place of the runtime's, so that each launch is printed instead of made.
 *   record_launches LIB B H T HW d chunk overlap saved workspace_bytes
 * One line per launch (grid x y z, kernel), then "status S".  Pointers are fake and never dereferenced. */
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>

#include "../../include/rehyat.h"

typedef struct { unsigned x, y, z; } dim3;

static struct { const void* host; const char* name; } kernels[256];
static int n_kernels;
static dim3 cfg_grid, cfg_block;

void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid,
                           void* bid, void* block, void* grid, int* wsize) {
  (void)modules, (void)device, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)wsize;
  if (n_kernels < 256) kernels[n_kernels].host = host, kernels[n_kernels++].name = name;
}
void __hipRegisterVar(void** modules, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
  (void)modules, (void)var, (void)host, (void)device, (void)ext, (void)size, (void)constant, (void)global;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void* stream) {
  (void)shared, (void)stream;
  cfg_grid = grid, cfg_block = block;
  return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, void** stream) {
  *grid = cfg_grid, *block = cfg_block, *shared = 0, *stream = NULL;
  return 0;
}
int hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t shared, void* stream) {
  const char* name = "?";
  (void)block, (void)args, (void)shared, (void)stream;
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == host) name = kernels[i].name;
  printf("%u %u %u %s\n", grid.x, grid.y, grid.z, name);
  return 0;
}
int hipGetLastError(void) { return 0; }

int main(int argc, char** argv) {
  if (argc != 11) return 2;
  void* const lib = dlopen(argv[1], RTLD_NOW);
  if (!lib) {
    fprintf(stderr, "%s\n", dlerror());
    return 2;
  }
  int (*const backward)(const void*, const void*, const void*, const rehyat_phi_params*, const void*, void*,
                        const rehyat_forward_saved*, const rehyat_phi_grads*, int, int, int, int, int, int, int, void*,
                        size_t, void*) = dlsym(lib, "rehyat_phi_backward");
  if (!backward) return 2;
  const int d = atoi(argv[6]);
  void* const A = (void*)0x1000;
  const rehyat_phi_params phi = {A, A, A, A, A, A, A, A, 2 * d, 2 * d, 2, 0};
  const rehyat_phi_grads grads = {A, A, A, A, A, A, A, A};
  const rehyat_forward_saved saved = {A, A};
  const int rc = backward(A, A, A, &phi, A, A, atoi(argv[9]) ? &saved : NULL, &grads, atoi(argv[2]), atoi(argv[3]),
                          atoi(argv[4]), atoi(argv[5]), d, atoi(argv[7]), atoi(argv[8]), A,
                          strtoull(argv[10], NULL, 10), NULL);
  printf("status %d\n", rc);
  return 0;
}
