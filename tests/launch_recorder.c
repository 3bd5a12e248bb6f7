/*
 * A stand-in for the few HIP entry points that the library uses, for tests of the host code without a GPU: kernels are
 * registered by name and every launch is written down instead of run.  It is loaded before the library with RTLD_GLOBAL,
 * so that the library's references bind to it, in a process that loads neither torch nor anything else that uses HIP.
 */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { const void *host; const char *name; } kernel_t;
typedef struct { const char *name; dim3_t grid, block; } launch_t;

static kernel_t kernels[8192];
static int n_kernels;
static launch_t launches[256];
static int n_launches;
static struct { dim3_t grid, block; size_t lds; void *stream; } config;

void **__hipRegisterFatBinary(const void *data) { static void *handle; (void)data; return &handle; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *var, char *host, char *device, int ext, size_t size, int constant, int global) {
  (void)m; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
void __hipRegisterFunction(void **m, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid,
                           void *block, void *grid, int *wsize) {
  (void)m; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
  if (n_kernels == sizeof kernels / sizeof *kernels) abort();
  kernels[n_kernels].host = host;
  kernels[n_kernels++].name = strdup(name);
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
  config.grid = grid; config.block = block; config.lds = lds; config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
  *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void *host, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
  (void)args; (void)lds; (void)stream;
  if (n_launches == sizeof launches / sizeof *launches) abort();
  launch_t *l = &launches[n_launches++];
  l->name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].host == host) l->name = kernels[i].name;
  l->grid = grid;
  l->block = block;
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = NULL; return 1; }

void recorder_reset(void) { n_launches = 0; }
int recorder_count(void) { return n_launches; }
const char *recorder_name(int i) { return launches[i].name; }
uint64_t recorder_workgroups(int i) {
  const dim3_t g = launches[i].grid;
  return (uint64_t)g.x * g.y * g.z;
}
