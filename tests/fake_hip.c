/* A HIP runtime without a device: it launches nothing and keeps the name and grid of every launch.  The host side of the
 * library (argument checks, plans, workspace carving) can so be driven on a machine without a GPU, on addresses that
 * nothing reads. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
static struct { const void* fn; const char* name; } kernels[512];
static int n_kernels;
static struct { const char* name; uint32_t grid[3]; uint64_t word; } launches[4096];
static int n_launches;
static dim3_t cfg_grid, cfg_block;
static char device_array[1];

void fake_clear(void) { n_launches = 0; }
int fake_count(void) { return n_launches; }
const char* fake_name(int i) { return launches[i].name; }
uint32_t fake_grid(int i, int d) { return launches[i].grid[d]; }
/* Of launches of the kernels whose name holds this, the eight bytes at `offset` of parameter `arg` are kept as well. */
static const char* watched;
static int watched_arg, watched_offset;
void fake_watch(const char* name, int arg, int offset) { watched = strdup(name); watched_arg = arg; watched_offset = offset; }
uint64_t fake_word(int i) { return launches[i].word; }

void** __hipRegisterFatBinary(const void* data) { (void)data; static void* handle; return &handle; }
void __hipUnregisterFatBinary(void** m) { (void)m; }
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned limit, void* a, void* b, void* c, void* d, int* e) {
  (void)m; (void)dev; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)e;
  if (n_kernels < 512) { kernels[n_kernels].fn = host; kernels[n_kernels++].name = strdup(name); }
}
void __hipRegisterVar(void** m, void* var, char* a, char* b, int c, size_t d, int e, int f) {
  (void)m; (void)var; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f;
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void* stream) {
  (void)shared; (void)stream;
  cfg_grid = grid; cfg_block = block;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shared, void** stream) {
  *grid = cfg_grid; *block = cfg_block; *shared = 0; *stream = 0;
  return 0;
}
int hipLaunchKernel(const void* fn, dim3_t grid, dim3_t block, void** args, size_t shared, void* stream) {
  (void)block; (void)shared; (void)stream;
  const char* name = "?";
  for (int i = 0; i < n_kernels; ++i) if (kernels[i].fn == fn) name = kernels[i].name;
  if (n_launches < 4096) {
    launches[n_launches].name = name;
    launches[n_launches].word = 0;
    if (watched && strstr(name, watched)) memcpy(&launches[n_launches].word, (const char*)args[watched_arg] + watched_offset, 8);
    launches[n_launches].grid[0] = grid.x; launches[n_launches].grid[1] = grid.y; launches[n_launches++].grid[2] = grid.z;
  }
  return 0;
}
int hipGetDeviceCount(int* n) { *n = 1; return 0; }
int hipSetDevice(int d) { (void)d; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "fake"; }
int hipHostMalloc(void** p, size_t n, unsigned flags) { (void)flags; *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = device_array; return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) { (void)d; (void)s; (void)n; (void)kind; (void)stream; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipEventCreate(void** e) { *e = device_array; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { (void)e; (void)s; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }
