/* A HIP runtime without a device: it launches nothing and keeps the name and grid of every launch.  The host side of the
 * library (argument checks, plans, workspace carving) can so be driven on a machine without a GPU, on addresses that
 * nothing reads. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
static struct { const void* fn; const char* name; } kernels[512];
static int n_kernels;
/* Launches and events keep, for every stream, how many of its launches are sure to be over before them. */
typedef struct { int over[8]; } order_t;
static struct { const char* name; uint32_t grid[3]; uint64_t word; int stream; order_t order; } launches[4096];
static struct { void* handle; order_t order; } streams[8];
static int n_streams, streams_on;
static int stream_of(void* s) {
  for (int i = 0; i < n_streams; ++i) if (streams[i].handle == s) return i;
  if (n_streams == 8) abort();
  memset(&streams[n_streams], 0, sizeof(streams[0]));
  streams[n_streams].handle = s;
  return n_streams++;
}
/* Without fake_streams(1) no stream can be created. */
void fake_streams(int on) { streams_on = on; }
static int n_launches;
static dim3_t cfg_grid, cfg_block;
static void* cfg_stream;
static char device_array[1];

void fake_clear(void) { n_launches = 0; }
int fake_count(void) { return n_launches; }
const char* fake_name(int i) { return launches[i].name; }
uint32_t fake_grid(int i, int d) { return launches[i].grid[d]; }
int fake_stream(int i) { return launches[i].stream; }
/* whether launch i is over before launch j begins */
int fake_before(int i, int j) { return launches[j].order.over[launches[i].stream] > launches[i].order.over[launches[i].stream]; }
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
  (void)shared;
  cfg_grid = grid; cfg_block = block; cfg_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* shared, void** stream) {
  *grid = cfg_grid; *block = cfg_block; *shared = 0; *stream = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* fn, dim3_t grid, dim3_t block, void** args, size_t shared, void* stream) {
  (void)block; (void)shared;
  const char* name = "?";
  const int at = stream_of(stream);
  for (int i = 0; i < n_kernels; ++i) if (kernels[i].fn == fn) name = kernels[i].name;
  if (n_launches < 4096) {
    launches[n_launches].name = name;
    launches[n_launches].word = 0;
    launches[n_launches].stream = at;
    launches[n_launches].order = streams[at].order;
    ++streams[at].order.over[at];
    if (watched && strstr(name, watched)) memcpy(&launches[n_launches].word, (const char*)args[watched_arg] + watched_offset, 8);
    launches[n_launches].grid[0] = grid.x; launches[n_launches].grid[1] = grid.y; launches[n_launches++].grid[2] = grid.z;
  }
  return 0;
}
/* Two devices, one of them current; streams and events belong to the one that is current as they are made. */
static int device, made[2];
int fake_made(int d) { return made[d]; }
int hipGetDeviceCount(int* n) { *n = 2; return 0; }
int hipSetDevice(int d) { device = d; return 0; }
int hipGetDevice(int* d) { *d = device; return 0; }
int hipGetLastError(void) { return 0; }
const char* hipGetErrorString(int e) { (void)e; return "fake"; }
int hipHostMalloc(void** p, size_t n, unsigned flags) { (void)flags; *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipGetSymbolAddress(void** p, const void* s) { (void)s; *p = device_array; return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* stream) { (void)d; (void)s; (void)n; (void)kind; (void)stream; return 0; }
int hipStreamSynchronize(void* s) { (void)s; return 0; }
int hipEventCreate(void** e) { *e = device_array; return 0; }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; *e = calloc(1, sizeof(order_t)); ++made[device]; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* s) { if (e != device_array) *(order_t*)e = streams[stream_of(s)].order; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned flags) {
  (void)flags;
  order_t* o = &streams[stream_of(s)].order;
  for (int i = 0; i < 8; ++i) if (o->over[i] < ((order_t*)e)->over[i]) o->over[i] = ((order_t*)e)->over[i];
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned flags) { (void)flags; *s = malloc(1); made[device] += streams_on; return !streams_on; }
int hipStreamDestroy(void* s) { (void)s; return 0; }
int hipStreamIsCapturing(void* s, int* status) { (void)s; *status = 0; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0; return 0; }
