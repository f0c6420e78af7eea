/* A HIP runtime without a device: every call the library makes succeeds at
 * once, and each kernel launch is recorded (kernel name, grid) instead of run,
 * so that host decisions (which kernel, how many workgroups, which errors) can
 * be tested on a CPU.  Loaded before the library, whose HIP symbols then bind
 * here.  Device pointers are never dereferenced by host code. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int err_t;

enum { kMaxKernels = 4096, kMaxLaunches = 1 << 18 };
static const void* g_host[kMaxKernels];
static const char* g_name[kMaxKernels];
static int g_kernels;
static int g_launch[kMaxLaunches];
static dim3_t g_grid[kMaxLaunches];
static int g_launches;

/* test side */
int rec_device = 0;        /* the current device */
int rec_fail_capture = 0;  /* hipStreamEndCapture fails */
void rec_reset(void) { g_launches = 0; }
int rec_count(void) { return g_launches; }
const char* rec_name(int i) { return g_launch[i] < 0 ? "?" : g_name[g_launch[i]]; }
uint32_t rec_grid_x(int i) { return g_grid[i].x; }

static void record(const void* f, dim3_t grid) {
  int k = -1;
  for (int i = 0; i < g_kernels; ++i)
    if (g_host[i] == f) k = i;
  if (g_launches < kMaxLaunches) {
    g_launch[g_launches] = k;
    g_grid[g_launches++] = grid;
  }
}

void** __hipRegisterFatBinary(const void* data) {
  static void* handle;
  (void)data;
  return &handle;
}
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned lim, void* tid, void* bid,
                           dim3_t* bd, dim3_t* gd, int* ws) {
  (void)m; (void)dev; (void)lim; (void)tid; (void)bid; (void)bd; (void)gd; (void)ws;
  if (g_kernels < kMaxKernels) {
    g_host[g_kernels] = host;
    g_name[g_kernels++] = name;
  }
}
void __hipRegisterVar(void** m, void* var, char* h, char* d, int ext, size_t size, int c, int g) {
  (void)m; (void)var; (void)h; (void)d; (void)ext; (void)size; (void)c; (void)g;
}
static dim3_t g_cfg_grid, g_cfg_block;
static size_t g_cfg_shmem;
static void* g_cfg_stream;
err_t __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void* stream) {
  g_cfg_grid = grid;
  g_cfg_block = block;
  g_cfg_shmem = shmem;
  g_cfg_stream = stream;
  return 0;
}
err_t __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shmem, void** stream) {
  *grid = g_cfg_grid;
  *block = g_cfg_block;
  *shmem = g_cfg_shmem;
  *stream = g_cfg_stream;
  return 0;
}
err_t hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t shmem, void* s) {
  (void)block; (void)args; (void)shmem; (void)s;
  record(f, grid);
  return 0;
}
err_t hipLaunchCooperativeKernel(const void* f, dim3_t grid, dim3_t block, void** args, unsigned shmem, void* s) {
  (void)block; (void)args; (void)shmem; (void)s;
  record(f, grid);
  return 0;
}
err_t hipGetDeviceCount(int* n) { *n = 0; return 0; }
err_t hipGetDevice(int* d) { *d = rec_device; return 0; }
err_t hipGetDevicePropertiesR0600(void* p, int d) { (void)p; (void)d; return 0; }
err_t hipDeviceGetAttribute(int* v, int a, int d) { (void)a; (void)d; *v = 256; return 0; }
err_t hipDeviceSynchronize(void) { return 0; }
err_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t sh) {
  (void)f; (void)b; (void)sh;
  *n = 1;
  return 0;
}
const char* hipGetErrorString(err_t e) { return e ? "error" : "no error"; }
err_t hipGetLastError(void) { return 0; }
err_t hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = (void*)256; return 0; }
err_t hipMalloc(void** p, size_t n) { (void)n; *p = (void*)256; return 0; }
err_t hipFree(void* p) { (void)p; return 0; }
err_t hipEventCreate(void** e) { *e = (void*)256; return 0; }
err_t hipEventDestroy(void* e) { (void)e; return 0; }
err_t hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
err_t hipEventSynchronize(void* e) { (void)e; return 0; }
err_t hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.f; return 0; }
err_t hipStreamCreateWithFlags(void** s, unsigned f) { (void)f; *s = (void*)256; return 0; }
err_t hipStreamDestroy(void* s) { (void)s; return 0; }
err_t hipStreamSynchronize(void* s) { (void)s; return 0; }
err_t hipStreamIsCapturing(void* s, int* st) { (void)s; *st = 0; return 0; }
err_t hipStreamBeginCapture(void* s, int mode) { (void)s; (void)mode; return 0; }
err_t hipStreamEndCapture(void* s, void** g) {
  (void)s;
  *g = rec_fail_capture ? NULL : (void*)256;
  return rec_fail_capture ? 1 : 0;
}
err_t hipGraphInstantiate(void** x, void* g, void* n, char* b, size_t sz) {
  (void)g; (void)n; (void)b; (void)sz;
  *x = (void*)256;
  return 0;
}
err_t hipGraphDestroy(void* g) { (void)g; return 0; }
err_t hipGraphExecDestroy(void* g) { (void)g; return 0; }
err_t hipGraphLaunch(void* g, void* s) { (void)g; (void)s; return 0; }
