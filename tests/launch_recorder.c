/* Stand-ins for the HIP runtime calls that libsparoa.so makes on its launch
 * path.  Loaded with global scope before the library, they take the place of
 * the runtime's: no device is needed, nothing runs, and every launch is kept
 * as its kernel's name and grid.  A launch with an empty dimension fails as
 * the runtime has it fail (invalid configuration). */
#include <stddef.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
enum { kInvalidConfiguration = 9, kMaxKernels = 4096, kMaxLaunches = 256 };

static struct { const void *host; char name[256]; } kernels[kMaxKernels];
static struct { char name[256]; dim3_t grid, block; } launches[kMaxLaunches];
static int n_kernels, n_launches, last_error;
static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void *cfg_stream;

int recorded_launches(void) { return n_launches; }
const char *recorded_name(int i) { return launches[i].name; }
void recorded_grid(int i, unsigned *g) { memcpy(g, &launches[i].grid, sizeof(dim3_t)); }
void forget_launches(void) { n_launches = 0; last_error = 0; }

void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterVar(void **h, void *v, char *a, char *b, int e, size_t s, int c, int g) {
  (void)h; (void)v; (void)a; (void)b; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **h, const void *host, char *dev, const char *name, unsigned t,
                           void *a, void *b, void *c, void *d, int *w) {
  (void)h; (void)dev; (void)t; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_kernels == kMaxKernels) return;
  kernels[n_kernels].host = host;
  snprintf(kernels[n_kernels++].name, sizeof kernels[0].name, "%s", name);
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
  cfg_grid = grid; cfg_block = block; cfg_lds = lds; cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
  *grid = cfg_grid; *block = cfg_block; *lds = cfg_lds; *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void *fn, dim3_t grid, dim3_t block, void **args, size_t lds,
                    void *stream) {
  (void)args; (void)lds; (void)stream;
  if (n_launches < kMaxLaunches) {
    const char *name = "?";
    for (int i = 0; i < n_kernels; ++i)
      if (kernels[i].host == fn) name = kernels[i].name;
    snprintf(launches[n_launches].name, sizeof launches[0].name, "%s", name);
    launches[n_launches].grid = grid;
    launches[n_launches++].block = block;
  }
  if (!grid.x || !grid.y || !grid.z || !block.x || !block.y || !block.z)
    return last_error = kInvalidConfiguration;
  return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e ? "invalid configuration" : "no error"; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *fn, int t, size_t lds) {
  (void)fn; (void)t; (void)lds;
  *n = 2;
  return 0;
}
