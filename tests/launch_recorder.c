/* Stands in for the HIP calls that libsonicmoe.so makes on the host path of an
 * entry point, so that a test without a GPU can ask which kernels a call
 * launches: loaded with RTLD_GLOBAL before the library, it receives the kernel
 * registrations and the launches, and keeps the names and grids. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;

enum { kMax = 4096 };
static struct { const void *f; const char *name; } kernels[kMax];
static struct { const char *name; dim3_t grid, block; } launches[kMax];
static int n_kernels, n_launches, cus = 256;

void __hipRegisterFunction(void **modules, const void *f, char *device_function, const char *device_name,
                           unsigned limit, void *tid, void *bid, void *block, void *grid, int *wsize) {
  (void)modules, (void)device_function, (void)limit, (void)tid, (void)bid, (void)block, (void)grid, (void)wsize;
  if (n_kernels < kMax) {
    kernels[n_kernels].f = f;
    kernels[n_kernels++].name = strdup(device_name);
  }
}
static struct { dim3_t grid, block; size_t lds; void *stream; } config;
unsigned __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
  config.grid = grid, config.block = block, config.lds = lds, config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
  *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
  return 0;
}
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
  (void)args, (void)lds, (void)stream;
  if (n_launches == kMax) return 1;
  const char *name = "?";
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].f == f) name = kernels[i].name;
  launches[n_launches].name = name;
  launches[n_launches].grid = grid;
  launches[n_launches++].block = block;
  return 0;
}
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int attr, int value) { return (void)f, (void)attr, (void)value, 0; }
int hipGetDevice(int *dev) { return *dev = 0; }
int hipDeviceGetAttribute(int *value, int attr, int dev) { return (void)attr, (void)dev, *value = cus, 0; }

void rec_set_cus(int n) { cus = n; }
int rec_count(void) { return n_launches; }
void rec_clear(void) { n_launches = 0; }
const char *rec_name(int i) { return launches[i].name; }
int rec_grid(int i, int axis) { return axis == 0 ? launches[i].grid.x : axis == 1 ? launches[i].grid.y : launches[i].grid.z; }
