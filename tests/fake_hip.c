/* A stand-in for the HIP runtime calls that libmmf.so makes, for tests without
 * a GPU: launches are recorded instead of run, device memory is made-up
 * addresses, and a launch past the runtime's limits is refused as there
 * (fewer than 2^32 threads per dimension, at most 1024 per block).
 * Built with gcc by tests/record.py and loaded in front of the library. */
#include <dlfcn.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct {
  unsigned x, y, z;
} dim3;

enum { kMaxKernels = 8192, kMaxLaunches = 4096, kArgs = 6 };
static struct {
  const void *fn;
  const char *name;
} kernels[kMaxKernels];
static int n_kernels;

typedef struct {
  const char *name;
  unsigned grid[3], block[3];
  uint64_t args[kArgs]; /* the first pointer arguments of act-quant kernels */
} Launch;
static Launch launches[kMaxLaunches];
static int n_launches, n_allocs, n_frees, last_error;

/* what the next call meets: capture status, failing allocations, and a
 * mmf_set_path(switch_path) from "another thread" at the switch_at-th query */
static int capturing, fail_alloc, switch_at, switch_path, queries;
static int (*set_path)(int);

static void query(void) {
  if (set_path && ++queries == switch_at) set_path(switch_path);
}

void fake_reset(int capture, int fail, int at, int path, void *set) {
  n_launches = n_allocs = n_frees = last_error = queries = 0;
  capturing = capture;
  fail_alloc = fail;
  switch_at = at;
  switch_path = path;
  set_path = (int (*)(int))set;
}
int fake_launches(void) { return n_launches; }
const Launch *fake_launch(int i) { return &launches[i]; }
int fake_allocs(void) { return n_allocs; }
int fake_frees(void) { return n_frees; }

void **__hipRegisterFatBinary(const void *data) {
  static void *handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterVar(void *a, void *b, char *c, char *d, int e, size_t f, int g, int h) {
  (void)a, (void)b, (void)c, (void)d, (void)e, (void)f, (void)g, (void)h;
}
void __hipRegisterFunction(void *modules, const void *host, char *device, const char *name, unsigned limit, void *tid,
                           void *bid, void *bdim, void *gdim, int *wsize) {
  (void)modules, (void)device, (void)limit, (void)tid, (void)bid, (void)bdim, (void)gdim, (void)wsize;
  if (n_kernels < kMaxKernels) {
    kernels[n_kernels].fn = host;
    kernels[n_kernels++].name = name;
  }
}

static struct {
  dim3 grid, block;
  size_t shared;
  void *stream;
} config;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, void *stream) {
  config.grid = grid, config.block = block, config.shared = shared, config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, void **stream) {
  *grid = config.grid, *block = config.block, *shared = config.shared, *stream = config.stream;
  return 0;
}

int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t shared, void *stream) {
  (void)shared, (void)stream;
  const unsigned g[3] = {grid.x, grid.y, grid.z}, b[3] = {block.x, block.y, block.z};
  for (int i = 0; i < 3; ++i)
    if (g[i] == 0 || b[i] == 0 || (uint64_t)g[i] * b[i] > 0xFFFFFFFFull || (i > 0 && g[i] > 65535)) return last_error = 9;
  if ((uint64_t)b[0] * b[1] * b[2] > 1024) return last_error = 9;
  if (n_launches == kMaxLaunches) return last_error = 1;
  Launch *l = &launches[n_launches++];
  memset(l, 0, sizeof *l);
  for (int i = 0; i < n_kernels; ++i)
    if (kernels[i].fn == fn) l->name = kernels[i].name;
  memcpy(l->grid, g, sizeof g);
  memcpy(l->block, b, sizeof b);
  if (l->name && strstr(l->name, "act_quant_kernel"))
    for (int i = 0; i < kArgs; ++i) memcpy(&l->args[i], args[i], 8);
  return 0;
}

int hipGetLastError(void) {
  const int e = last_error;
  last_error = 0;
  return e;
}
int hipGetDevice(int *device) {
  query();
  *device = 0;
  return 0;
}
int hipDeviceGetAttribute(int *value, int attribute, int device) {
  (void)attribute, (void)device;
  *value = 256; /* compute units: the one attribute the library asks for */
  return 0;
}
int hipStreamIsCapturing(void *stream, int *status) {
  (void)stream;
  query();
  *status = capturing ? 1 : 0;
  return 0;
}
int hipMallocAsync(void **p, size_t bytes, void *stream) {
  (void)bytes, (void)stream;
  query();
  if (fail_alloc) return last_error = 2;
  *p = (void *)(uintptr_t)(0x7000000000ull + ((uint64_t)++n_allocs << 32));
  return 0;
}
int hipFreeAsync(void *p, void *stream) {
  (void)p, (void)stream;
  ++n_frees;
  return 0;
}
int hipGetSymbolAddress(void **p, const void *symbol) {
  (void)symbol;
  *p = (void *)(uintptr_t)0x6000000000ull;
  return 0;
}
