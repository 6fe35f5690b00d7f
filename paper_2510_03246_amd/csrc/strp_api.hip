// C ABI of libstrp.so: argument validation, workspace carving and the per-module ADMM drivers.
#include <stdarg.h>

#include <atomic>
#include <cmath>
#include <new>
#include <string>
#include <vector>

#include "cojob.h"
#include "strp_internal.h"

struct Profiler {
  struct Rec { const char* name; double flops, bytes; hipEvent_t e0, e1; };
  bool on = false;
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;
  hipEvent_t get() {
    if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  void clear() {
    for (auto& r : recs) { pool.push_back(r.e0); pool.push_back(r.e1); }
    recs.clear();
  }
  ~Profiler() {
    clear();
    for (auto e : pool) if (e) (void)hipEventDestroy(e);
  }
};

// Scratch of strp_mask_topk_static (the entry point for callers that cannot allocate): histograms and counters of the
// multi-block select.  Every GPU the library runs on
// holds its own copy of the array until the process ends; in host code the array's name is only a handle for
// hipGetSymbolAddress, the device address is resolved once per device in strp_create and kept in g_topk_scratch.
constexpr size_t TOPK_STATIC_BYTES = 1u << 20;
static __device__ __align__(256) unsigned char topk_static_scratch[TOPK_STATIC_BYTES];
constexpr int MAX_DEVICES = 64;
static void* g_topk_scratch[MAX_DEVICES];
// Counters of the weight statistics (strp_ctx::ticket): a context takes the next one, and another for the first weight statistics on
// another workspace.  Calls that may overlap in time -- captured ones, replayed on several streams -- have their scratch in
// workspaces of their own, and so never meet on a counter.  None is used again, so work that is still in flight when its context
// is destroyed or its workspace replaced meets nobody on it.
constexpr unsigned int MAX_TICKETS = 16384;
static __device__ unsigned int context_tickets[MAX_TICKETS];
static std::atomic<unsigned int> g_tickets_taken{0};
static unsigned int* next_ticket(unsigned int* tickets) {
  if (!tickets || g_tickets_taken.load() >= MAX_TICKETS) return nullptr;
  const unsigned int slot = g_tickets_taken.fetch_add(1);
  return slot < MAX_TICKETS ? tickets + slot : nullptr;
}

namespace strp {

int prof_begin(strp_ctx* ctx, const char* name, double flops, double bytes) {
  Profiler* pr = ctx->prof;
  if (!pr || !pr->on) return -1;
  Profiler::Rec r{name, flops, bytes, pr->get(), pr->get()};
  if (!r.e0 || !r.e1) return -1;
  (void)hipEventRecord(r.e0, ctx->stream);
  pr->recs.push_back(r);
  return (int)pr->recs.size() - 1;
}
void prof_end(strp_ctx* ctx, int rec) {
  if (rec < 0) return;
  (void)hipEventRecord(ctx->prof->recs[rec].e1, ctx->stream);
}

strp_status fail(strp_ctx* ctx, strp_status st, const char* fmt, ...) {
  if (ctx) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(ctx->err, sizeof(ctx->err), fmt, ap);
    va_end(ap);
  }
  return st;
}

static inline long long round_up(long long x, long long a) { return (x + a - 1) / a * a; }
static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// ---- small kernels ------------------------------------------------------------------------------
// raw = sum of v[0], v[stride], .. (n of them; single block, fixed order), *out = scale * raw, added to the diagonal of
// A [nd x nd, ld] when A is given
__global__ __launch_bounds__(1024) void scaled_sum_kernel(const double* v, int stride, int n, double scale, double* raw, double* out, double* A,
                                                          long long ld, int nd) {
  __shared__ double s[1024];
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 1024) a += v[(long long)i * stride];
  s[threadIdx.x] = a;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
    __syncthreads();
  }
  const double t = s[0];
  if (threadIdx.x == 0) {
    *raw = t;
    *out = t * scale;
  }
  if (A)
    for (int i = threadIdx.x; i < nd; i += 1024) A[(long long)i * ld + i] += t * scale;
}

// The pruned rows where the a- and z-stages come in separate calls, one block per row (rules: pruned_elem, cojob.h): phase 0 the
// a-update, phase 1 the z-update (write) and the row's share of the objective, red[2 j].
__global__ __launch_bounds__(256) void pruned_rows_kernel(const uint8_t* mask, float* Z, float* A, long long lda, long long T, int phase,
                                                          float alpha, float beta, int write, double* red) {
  const int j = blockIdx.x;
  double r0 = 0.0, r1 = 0.0;
  if (!mask[j]) {
    float* z = Z + (long long)j * lda;
    float* a = A + (long long)j * lda;
    const long long T4 = T >> 2;
    // two independent 16-byte groups per thread and trip: all loads of a trip are issued before its first store
    auto body = [&](long long c, float4 zv, float4 av) {
      pruned_elem(zv.x, av.x, phase, alpha, beta, write, r0, r1);
      pruned_elem(zv.y, av.y, phase, alpha, beta, write, r0, r1);
      pruned_elem(zv.z, av.z, phase, alpha, beta, write, r0, r1);
      pruned_elem(zv.w, av.w, phase, alpha, beta, write, r0, r1);
      if (phase != 1) ((float4*)a)[c] = av;
      if (phase != 0 && write) ((float4*)z)[c] = zv;
    };
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    long long c = threadIdx.x;
    for (; c + 256 < T4; c += 512) {
      const float4 zv0 = ((const float4*)z)[c], zv1 = ((const float4*)z)[c + 256];
      const float4 av0 = phase == 1 ? ((const float4*)a)[c] : zero4, av1 = phase == 1 ? ((const float4*)a)[c + 256] : zero4;
      body(c, zv0, av0);
      body(c + 256, zv1, av1);
    }
    if (c < T4) body(c, ((const float4*)z)[c], phase == 1 ? ((const float4*)a)[c] : zero4);
    for (long long t = T4 * 4 + threadIdx.x; t < T; t += 256) {
      float zv = z[t], av = phase == 1 ? a[t] : 0.0f;
      pruned_elem(zv, av, phase, alpha, beta, write, r0, r1);
      if (phase != 1) a[t] = av;
      if (phase != 0 && write) z[t] = zv;
    }
  }
  if (red) {
    __shared__ double sh[4][2];
    for (int o = 32; o > 0; o >>= 1) {
      r0 += __shfl_down(r0, o, 64);
      r1 += __shfl_down(r1, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
      sh[threadIdx.x >> 6][0] = r0;
      sh[threadIdx.x >> 6][1] = r1;
    }
    __syncthreads();
    if (threadIdx.x < 2) red[2 * (long long)j + threadIdx.x] = sh[0][threadIdx.x] + sh[1][threadIdx.x] + sh[2][threadIdx.x] + sh[3][threadIdx.x];
  }
}

// ---- the fused a/z pass of the pruned rows as a ride-along job (cojob.h) ---------------------------------------------
// rows[0 .. f - s) = the rows with mask == 0, ascending (one block; f is a few ten thousand at most)
__global__ __launch_bounds__(1024) void pruned_list_kernel(const uint8_t* mask, int f, int32_t* rows) {
  __shared__ int scan[1024];
  const int tid = threadIdx.x;
  const int per = (f + 1023) / 1024;
  const int j0 = tid * per, j1 = (j0 + per < f) ? j0 + per : f;
  int cnt = 0;
  for (int j = j0; j < j1; ++j) cnt += mask[j] ? 0 : 1;
  scan[tid] = cnt;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int v = tid >= o ? scan[tid - o] : 0;
    __syncthreads();
    scan[tid] += v;
    __syncthreads();
  }
  int pos = scan[tid] - cnt;
  for (int j = j0; j < j1; ++j)
    if (!mask[j]) rows[pos++] = j;
  // entries past the last pruned row name no row (a unit of such an entry does nothing): the job's row count comes
  // from the host's record of the kept count, which a caller-supplied mask need not match
  const int total = scan[1023];
  for (int j = total + tid; j < f; j += 1024) rows[j] = -1;
}

// scalar slots of strp_module_state::scalars
// bits of strp_module_state::sums_cached: which token sums cv.rowsums holds for EVERY row of the current state
enum { SUMS_G = 1, SUMS_EU = 2, SUMS_V = 4 };
enum { SC_LAM1 = 0, SC_LAM2 = 1, SC_SUMA0 = 2, SC_TRH = 3, SC_T1 = 4, SC_T2 = 5, SC_T3 = 6, SC_T4 = 7, SC_T5 = 8,
       SC_TAU = 9, SC_ENERGY = 10, SC_W2SQ = 15, SC_W1SQ = 16, SC_COUNT = 32 };

// The end of an iteration, in one launch: the pruned rows' sums from the units of their pass, the kept rows' scoring sums from the strips that the a- and
// z-update epilogues wrote, the objective's terms from the workgroups' sums, and the report's read-back.  What bounds it is the round trips to memory
// that follow each other, so everything that is independent is another workgroup or is asked for at once, and the last workgroup to end puts it together.
// A launch for the strips' sums of either update and one workgroup that formed the objective's seven sums one after the other before: us of
// a step's end, 768 x 1536 units over 65536 tokens 30 -> 12, 1000 x 1013 over 30011 (GAIN) 28 -> 12, 64 x 128 over 512 8.7 -> 9.4 (a launch less), and 7.2 since
// wavefronts without a summand exchange nothing.
constexpr int FINISH_THREADS = 1024, FINISH_ROWS = FINISH_THREADS / 6, FINISH_SUMS = 7;
static inline int finish_row_blocks(int nrows) { return (nrows + 2 * FINISH_ROWS - 1) / (2 * FINISH_ROWS); }      // two rows one after the other
struct FinishP {
  double* sc;
  // pruned rows of a fused a/z pass (nrows = 0: none)
  const int32_t* rows;
  const double* partial;
  int nrows, segs, f, z0;
  double* rowsums;
  // the kept rows' strips: strips[q][slots][M], fp32, a value per row and 64 tokens, are sum q of row idx[m] (null: not collected)
  const float* strips[3];
  int slots, M, n_strips;
  const int32_t* idx;
  double* blk;                               // [row_blocks][2]
  double* sums;                              // [FINISH_SUMS]
  int row_blocks;
  unsigned int* ticket;
  // per-workgroup sums: terms 2 and 3 (kept rows, pruned rows when their pass was a kernel of its own), term 1, weights
  const double* red_z; int nz;               // pairs
  const double* red_p; int np;               // pairs
  const double* red_1; int n1, stride1;      // every stride1-th
  const double* w2; int nw2;
  const double* w1; int nw1;
  double c1, c2, c3;
  int do_z, do_1, do_w;
  double* host;                              // pinned: [SC_COUNT] scalars, then the status word; null: no report
  int32_t* status;
};
// sums of v over the workgroup, in out (LDS) for everybody; threads from `active` on hold zeros, and a wavefront of them exchanges nothing (the
// exchanges of sixteen wavefronts go through one LDS: 84 of each for seven sums)
template <int K>
__device__ __forceinline__ void finish_sums(double (&v)[K], double (&sh)[FINISH_SUMS][16], double* out, int active) {
  const int tid = threadIdx.x;
  if ((int)__builtin_amdgcn_readfirstlane(tid) < active) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int q = 0; q < K; ++q) v[q] += __shfl_down(v[q], o, 64);
  }
  if ((tid & 63) == 0)
#pragma unroll
    for (int q = 0; q < K; ++q) sh[q][tid >> 6] = v[q];
  __syncthreads();
  if (tid < K) {
    double a = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) a += sh[tid][w];
    out[tid] = a;
  }
  __syncthreads();
}
// a pruned row has six lanes, a sum each, added over its segments in their order
__device__ __forceinline__ void finish_rows(const FinishP& p, int b, double (&r)[2]) {
  const int e = threadIdx.x % 6, in = threadIdx.x / 6, q0 = 2 * b * FINISH_ROWS + in;
  r[0] = r[1] = 0.0;
  if (in >= FINISH_ROWS) return;
  double t[2] = {0.0, 0.0};
  int j[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int q = q0 + h * FINISH_ROWS;
    j[h] = q < p.nrows ? p.rows[q] : -1;
    if (q >= p.nrows) continue;
    const double* src = p.partial + (unsigned long long)q * p.segs * 6 + e;
#pragma unroll 8
    for (int g = 0; g < p.segs; ++g) t[h] += src[6 * g];
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (j[h] < 0) continue;
    r[0] += e == 0 ? t[h] : 0.0;
    r[1] += e == 1 ? t[h] : 0.0;
    if (e == 2 || (e > 2 && p.z0)) p.rowsums[(long long)(e - 2) * p.f + j[h]] = t[h];
  }
}
// One workgroup sums 64 kept rows: a wavefront takes every 16th strip (256 contiguous bytes of each), the sixteen sums are added in order.
__device__ __forceinline__ void finish_strips(const FinishP& p, int b, double (&sh)[16][64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, per = (p.M + 63) / 64, q = b / per;
  const int m = (b - q * per) * 64 + lane;
  const long long M = p.M;
  const float* strips = q == 0 ? p.strips[0] : q == 1 ? p.strips[1] : p.strips[2];
  const int sum = q == 0 ? 0 : q == 1 ? 1 : 2;
  const float* src = strips + (m < p.M ? m : p.M - 1);
  double a[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) a[u] = 0.0;
  int sidx = wave;
  for (; sidx + 7 * 16 < p.slots; sidx += 8 * 16) {       // eight loads in flight
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[(sidx + 16 * u) * M];
#pragma unroll
    for (int u = 0; u < 8; ++u) a[u] += (double)v[u];
  }
  for (; sidx < p.slots; sidx += 16) a[0] += (double)src[sidx * M];
  sh[wave][lane] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  __syncthreads();
  if (wave == 0 && m < p.M) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += sh[w][lane];
    p.rowsums[(long long)sum * p.f + p.idx[m]] = t;
    if (!(fabs(t) <= 1.79e308)) atomicCAS(p.status, 0, (int)STRP_ENONFINITE);
  }
}
__global__ __launch_bounds__(FINISH_THREADS) void step_finish_kernel(const FinishP p) {
  __shared__ double strips[16][64], sh[FINISH_SUMS][16], tot[FINISH_SUMS], rtot[2];
  __shared__ unsigned int flag;
  const int tid = threadIdx.x, b = blockIdx.x;
  const double scalar = tid < SC_COUNT ? p.sc[tid] : 0.0;
  double r[2] = {0.0, 0.0};
  if (b < p.row_blocks) {
    finish_rows(p, b, r);
    finish_sums<2>(r, sh, rtot, 6 * (p.nrows - 2 * b * FINISH_ROWS));
    if (tid < 2) agent_put(&p.blk[2 * b + tid], rtot[tid]);
  } else if (b == p.row_blocks) {
    double v[FINISH_SUMS];
#pragma unroll
    for (int q = 0; q < FINISH_SUMS; ++q) v[q] = 0.0;
    const auto pairs = [&](const double* x, int n, double& v0, double& v1) {
#pragma unroll 4
      for (int i = tid; i < n; i += FINISH_THREADS) {
        const double2 d = *(const double2*)(x + 2 * (long long)i);
        v0 += d.x;
        v1 += d.y;
      }
    };
    const auto every = [&](const double* x, int n, int stride, double& v0) {
#pragma unroll 4
      for (int i = tid; i < n; i += FINISH_THREADS) v0 += x[(long long)i * stride];
    };
    if (p.do_z) pairs(p.red_z, p.nz, v[0], v[1]);
    if (p.do_z && p.np) pairs(p.red_p, p.np, v[2], v[3]);
    if (p.do_1) every(p.red_1, p.n1, p.stride1, v[4]);
    if (p.do_w) {
      every(p.w2, p.nw2, 1, v[5]);
      every(p.w1, p.nw1, 1, v[6]);
    }
    int most = p.do_1 ? p.n1 : 0;
    if (p.do_z) most = max(most, max(p.nz, p.np));
    if (p.do_w) most = max(most, max(p.nw2, p.nw1));
    finish_sums<FINISH_SUMS>(v, sh, tot, most);
    if (gridDim.x > 1 && tid < FINISH_SUMS) agent_put(&p.sums[tid], tot[tid]);
  } else {
    finish_strips(p, b - p.row_blocks - 1, strips);
  }
  if (gridDim.x > 1) {
    if (!last_block(p.ticket, &flag)) return;
    if (tid == 0) *p.ticket = 0u;
    if (tid < FINISH_SUMS) tot[tid] = agent_get(&p.sums[tid]);
    r[0] = r[1] = 0.0;
    for (int i = tid; i < p.row_blocks; i += FINISH_THREADS) {
      r[0] += agent_get(&p.blk[2 * i]);
      r[1] += agent_get(&p.blk[2 * i + 1]);
    }
    finish_sums<2>(r, sh, rtot, p.row_blocks);
  }
  // one lane a scalar: those that are new go to the state, all of them to the report
  if (tid < SC_COUNT) {
    const double r0 = gridDim.x > 1 ? rtot[0] : 0.0, r1 = gridDim.x > 1 ? rtot[1] : 0.0;
    double v = scalar;
    bool fresh = true;
    if (p.do_z && tid == SC_T2) v = p.c2 * (tot[0] + (p.np ? tot[2] : r0));
    else if (p.do_z && tid == SC_T3) v = p.c3 * (tot[1] + (p.np ? tot[3] : r1));
    else if (p.do_1 && tid == SC_T1) v = p.c1 * tot[4];
    else if (p.do_w && tid == SC_W2SQ) v = tot[5];
    else if (p.do_w && tid == SC_W1SQ) v = tot[6];
    else fresh = false;
    if (fresh) p.sc[tid] = v;
    if (p.host) __hip_atomic_store(&p.host[tid], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (p.host && tid == SC_COUNT) __hip_atomic_store((int32_t*)(p.host + SC_COUNT), agent_get(p.status), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

static strp_status check_desc(strp_ctx* ctx, const strp_module_desc* d) {
  if (!d) return fail(ctx, STRP_EINVAL, "null module descriptor");
  if (d->d <= 0 || d->f <= 0 || d->T <= 0) return fail(ctx, STRP_EINVAL, "module: d, f, T must be positive");
  if (d->ldx < d->T || d->lda < d->T) return fail(ctx, STRP_EINVAL, "module: leading dimension below T");
  if (d->ldx % 8 || d->lda % 8 || d->d % 8 || d->f % 8) return fail(ctx, STRP_EINVAL, "module: d, f and leading dimensions must be multiples of 8");
  if ((d->x_dtype != STRP_BF16 && d->x_dtype != STRP_F32) || (d->w_dtype != STRP_BF16 && d->w_dtype != STRP_F32))
    return fail(ctx, STRP_EINVAL, "module: unknown dtype");
  if (d->k_max < 0 || d->k_max > d->f) return fail(ctx, STRP_EINVAL, "module: k_max outside [0, f]");
  return STRP_OK;
}

}  // namespace strp

using namespace strp;

extern "C" {

strp_status strp_create(strp_ctx** out, int device, void* hip_stream) {
  if (!out) return STRP_EINVAL;
  *out = nullptr;
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || device < 0 || device >= count) return STRP_EHIP;
  if (hipSetDevice(device) != hipSuccess) return STRP_EHIP;
  strp_ctx* c = new (std::nothrow) strp_ctx();
  if (!c) return STRP_ENOMEM;
  memset(c, 0, sizeof(*c));
  c->device = device;
  c->stream = (hipStream_t)hip_stream;
  c->precision = STRP_PREC_SPLIT;
  for (int i = 0; i < 8; ++i) c->prod_planes[i][0] = c->prod_planes[i][1] = 2;
  if (hipHostMalloc(&c->pinned, 4096, hipHostMallocDefault) != hipSuccess) {
    delete c;
    return STRP_EHIP;
  }
  // device address of this GPU's copy of the static select scratch (the device was made current above)
  if (device < MAX_DEVICES && !g_topk_scratch[device]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(topk_static_scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      (void)hipHostFree(c->pinned);
      delete c;
      return STRP_EHIP;
    }
    g_topk_scratch[device] = ptr;
  }
  void* tickets = nullptr;
  if (hipGetSymbolAddress(&tickets, HIP_SYMBOL(context_tickets)) != hipSuccess) {
    (void)hipGetLastError();
    tickets = nullptr;
  }
  c->tickets = (unsigned int*)tickets;
  c->ticket = next_ticket(c->tickets);
  *out = c;
  return STRP_OK;
}

strp_status strp_destroy(strp_ctx* ctx) {
  if (!ctx) return STRP_EINVAL;
  if (ctx->pinned) (void)hipHostFree(ctx->pinned);
  if (ctx->side_state > 0) {
    (void)hipStreamDestroy(ctx->side);
    for (hipEvent_t e : ctx->side_event) (void)hipEventDestroy(e);
  }
  delete ctx->prof;
  delete ctx;
  return STRP_OK;
}

const char* strp_last_error(const strp_ctx* ctx) { return ctx ? ctx->err : "null context"; }

strp_status strp_set_precision(strp_ctx* ctx, strp_precision prec) {
  if (!ctx) return STRP_EINVAL;
  if (prec != STRP_PREC_FAST && prec != STRP_PREC_SPLIT) return fail(ctx, STRP_EINVAL, "unknown precision %d", (int)prec);
  ctx->precision = prec;
  return STRP_OK;
}

strp_status strp_set_product_planes(strp_ctx* ctx, strp_product product, int32_t planes_p, int32_t planes_q) {
  if (!ctx) return STRP_EINVAL;
  if (product < 0 || product >= STRP_PROD_COUNT || planes_p < 1 || planes_p > 2 || planes_q < 1 || planes_q > 2)
    return fail(ctx, STRP_EINVAL, "set_product_planes: product in [0, %d), planes 1 or 2", (int)STRP_PROD_COUNT);
  ctx->prod_planes[product][0] = (unsigned char)planes_p;
  ctx->prod_planes[product][1] = (unsigned char)planes_q;
  return STRP_OK;
}

strp_status strp_profile_enable(strp_ctx* ctx, int on) {
  if (!ctx) return STRP_EINVAL;
  if (!ctx->prof) ctx->prof = new (std::nothrow) Profiler();
  if (!ctx->prof) return fail(ctx, STRP_ENOMEM, "profile: host allocation failed");
  STRP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  ctx->prof->clear();
  ctx->prof->on = on != 0;
  return STRP_OK;
}

strp_status strp_profile_read(strp_ctx* ctx, strp_profile_entry* out_host, int32_t max_entries, int32_t* n_out) {
  if (!ctx || !out_host || !n_out || max_entries <= 0) return ctx ? fail(ctx, STRP_EINVAL, "profile_read: bad argument") : STRP_EINVAL;
  *n_out = 0;
  if (!ctx->prof) return STRP_OK;
  STRP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  int n = 0;
  for (auto& r : ctx->prof->recs) {
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, r.e0, r.e1) != hipSuccess) continue;
    int j = 0;
    for (; j < n; ++j)
      if (strncmp(out_host[j].name, r.name, sizeof(out_host[j].name)) == 0) break;
    if (j == n) {
      if (n == max_entries) continue;
      memset(&out_host[n], 0, sizeof(out_host[n]));
      strncpy(out_host[n].name, r.name, sizeof(out_host[n].name) - 1);
      ++n;
    }
    out_host[j].launches += 1;
    out_host[j].ms += ms;
    out_host[j].flops += r.flops;
    out_host[j].bytes += r.bytes;
  }
  *n_out = n;
  return STRP_OK;
}

strp_status strp_profile_launches(strp_ctx* ctx, strp_profile_entry* out_host, int32_t max_entries, int32_t* n_out) {
  if (!ctx || !out_host || !n_out || max_entries <= 0) return ctx ? fail(ctx, STRP_EINVAL, "profile_launches: bad argument") : STRP_EINVAL;
  *n_out = 0;
  if (!ctx->prof) return STRP_OK;
  STRP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  int n = 0;
  for (auto& r : ctx->prof->recs) {
    if (n == max_entries) break;
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, r.e0, r.e1) != hipSuccess) ms = -1.0f;
    memset(&out_host[n], 0, sizeof(out_host[n]));
    strncpy(out_host[n].name, r.name, sizeof(out_host[n].name) - 1);
    out_host[n].launches = 1;
    out_host[n].ms = ms;
    out_host[n].flops = r.flops;
    out_host[n].bytes = r.bytes;
    ++n;
  }
  *n_out = n;
  return STRP_OK;
}

strp_status strp_set_workspace(strp_ctx* ctx, void* dev_ptr, size_t bytes) {
  if (!ctx) return STRP_EINVAL;
  if (!dev_ptr || bytes < 4096) return fail(ctx, STRP_EINVAL, "workspace: null or smaller than 4096 bytes");
  if ((uintptr_t)dev_ptr & 255u) return fail(ctx, STRP_EINVAL, "workspace: pointer not 256-byte aligned");
  if (ctx->ws && ctx->ws != (char*)dev_ptr) ctx->ticket_due = 1;
  ctx->ws = (char*)dev_ptr;
  ctx->ws_bytes = bytes;
  ctx->status_dev = (int32_t*)dev_ptr;
  return fill_zero(ctx, dev_ptr, 256);
}

strp_status strp_poll(strp_ctx* ctx) {
  if (!ctx) return STRP_EINVAL;
  if (!ctx->ws) return fail(ctx, STRP_ENOMEM, "no workspace set");
  STRP_HIP(ctx, hipMemcpyAsync(ctx->pinned, ctx->status_dev, sizeof(int32_t), hipMemcpyDeviceToHost, ctx->stream));
  STRP_HIP(ctx, hipStreamSynchronize(ctx->stream));
  const int32_t st = *(int32_t*)ctx->pinned;
  if (st != 0) {
    fail(ctx, (strp_status)st, "device status word = %d", st);
    STRP_TRY(fill_zero(ctx, ctx->status_dev, 256));
  }
  return (strp_status)st;
}

strp_status strp_score_alloc(strp_ctx* ctx, const strp_score_in* in, float* unit_score, double* energies, int32_t layer_idx,
                             int32_t L, const int32_t* n_units, const int32_t* group_id, double rbar, double temperature,
                             double rmax, double* r_out, int32_t* nprune_out) {
  if (!ctx) return STRP_EINVAL;
  if (!in || !unit_score || !energies) return fail(ctx, STRP_EINVAL, "score_alloc: null argument");
  if (!in->A || in->n_channels <= 0 || in->group <= 0 || in->T <= 0) return fail(ctx, STRP_EINVAL, "score_alloc: bad input block");
  if (in->n_channels % in->group) return fail(ctx, STRP_EINVAL, "score_alloc: n_channels %% group != 0");
  if (in->ld < in->T || in->ld % 8 || !aligned16(in->A)) return fail(ctx, STRP_EINVAL, "score_alloc: bad leading dimension or alignment");
  if (in->mode < STRP_SCORE_WANDA || in->mode > STRP_SCORE_GAIN) return fail(ctx, STRP_EINVAL, "score_alloc: unknown mode");
  if (in->mode != STRP_SCORE_WANDA && (!in->Z || !in->Z0)) return fail(ctx, STRP_EINVAL, "score_alloc: LEMMA/GAIN need Z and Z0");
  if (!in->n2 && !in->What) return fail(ctx, STRP_EINVAL, "score_alloc: need n2 or What");
  if (L <= 0 || layer_idx < 0 || layer_idx >= L) return fail(ctx, STRP_EINVAL, "score_alloc: layer_idx outside [0, L)");
  if (r_out && (!nprune_out || !n_units)) return fail(ctx, STRP_EINVAL, "score_alloc: allocation needs n_units and nprune_out");
  if (r_out && (!(temperature > 0.0) || !(rbar >= 0.0) || !(rmax > 0.0))) return fail(ctx, STRP_EINVAL, "score_alloc: bad rbar/temperature/rmax");
  if (!ctx->ws) return fail(ctx, STRP_ENOMEM, "score_alloc: no workspace set");
  Arena arena(ctx);
  STRP_TAKE(ctx, arena, sums, double, 4 * (size_t)in->n_channels);
  const double* n2 = in->n2;
  if (!n2) {
    STRP_TAKE(ctx, arena, n2buf, double, (size_t)in->n_channels);
    STRP_TRY(launch_colnorm2(ctx, in->What, in->w_dtype, in->w_rows, in->n_channels, in->ldw, n2buf));
    n2 = n2buf;
  }
  STRP_TRY(launch_row_sums(ctx, in->A, in->a_dtype, in->Z, in->Z0, in->ld, in->T, in->n_channels, in->mode, sums));
  STRP_TRY(launch_unit_scores(ctx, sums, n2, in->n_channels, in->group, in->mode, unit_score, energies + layer_idx));
  if (r_out) STRP_TRY(launch_alloc(ctx, energies, L, n_units, group_id, rbar, temperature, rmax, 0, r_out, nprune_out));
  return STRP_OK;
}

strp_status strp_mask_topk(strp_ctx* ctx, const float* score, int32_t n, int32_t k, int32_t group, uint8_t* mask, int32_t* idx,
                           float* tau) {
  if (!ctx) return STRP_EINVAL;
  if (!score || !mask || !idx) return fail(ctx, STRP_EINVAL, "mask_topk: null argument");
  if (n <= 0 || k < 0 || k > n || group <= 0) return fail(ctx, STRP_EINVAL, "mask_topk: need n > 0, 0 <= k <= n, group > 0");
  const size_t need = (k > 0 && k < n) ? topk_scratch_bytes(n) : 0;
  void* scratch = nullptr;
  if (need) {
    Arena arena(ctx);
    scratch = arena.take(need);
    if (!scratch && group == 1) return fail(ctx, STRP_ENOMEM, "mask_topk: %d scores need %zu bytes of workspace (strp_topk_workspace_bytes)", n, need + 256);
  }
  return launch_topk(ctx, score, n, k, group, mask, idx, tau, scratch, need);
}

strp_status strp_weight_energy(strp_ctx* ctx, const strp_weight_ref* mats, int32_t n_mats, double var_coef, double l2_coef,
                               double scale, double* energy) {
  if (!ctx) return STRP_EINVAL;
  if (!mats || n_mats <= 0 || !energy) return fail(ctx, STRP_EINVAL, "weight_energy: null or empty matrix list");
  for (int i = 0; i < n_mats; ++i) {
    const strp_weight_ref& m = mats[i];
    if (!m.W || m.rows <= 0 || m.cols <= 0 || m.ld < m.cols) return fail(ctx, STRP_EINVAL, "weight_energy: bad matrix %d", i);
    if (m.dtype != STRP_BF16 && m.dtype != STRP_F32) return fail(ctx, STRP_EINVAL, "weight_energy: unknown dtype");
  }
  Arena arena(ctx);
  STRP_TAKE(ctx, arena, partial, double, weight_energy_scratch_bytes() / sizeof(double));
  if (ctx->ticket_due) {
    ctx->ticket = next_ticket(ctx->tickets);
    ctx->ticket_due = 0;
  }
  return launch_weight_energy(ctx, mats, n_mats, var_coef, l2_coef, scale, energy, partial);
}

strp_status strp_alloc_inverse(strp_ctx* ctx, const double* energies, int32_t L, const int32_t* n_units, const int32_t* group_id,
                               double rbar, double temperature, double rmax, double* r_out, int32_t* nprune_out) {
  if (!ctx) return STRP_EINVAL;
  if (!energies || !n_units || !r_out || !nprune_out) return fail(ctx, STRP_EINVAL, "alloc_inverse: null argument");
  if (L <= 0) return fail(ctx, STRP_EINVAL, "alloc_inverse: L must be positive");
  if (!(temperature > 0.0) || !(rbar >= 0.0 && rbar <= 1.0) || !(rmax > 0.0 && rmax <= 1.0))
    return fail(ctx, STRP_EINVAL, "alloc_inverse: need temperature > 0, 0 <= rbar <= 1, 0 < rmax <= 1");
  return launch_alloc(ctx, energies, L, n_units, group_id, rbar, temperature, rmax, 1, r_out, nprune_out);
}

strp_status strp_alloc_softmax(strp_ctx* ctx, const double* energies, int32_t L, const int32_t* n_units, const int32_t* group_id,
                               double rbar, double temperature, double rmax, double* r_out, int32_t* nprune_out) {
  if (!ctx) return STRP_EINVAL;
  if (!energies || !n_units || !r_out || !nprune_out) return fail(ctx, STRP_EINVAL, "alloc_softmax: null argument");
  if (L <= 0) return fail(ctx, STRP_EINVAL, "alloc_softmax: L must be positive");
  if (!(temperature > 0.0) || !(rbar >= 0.0 && rbar <= 1.0) || !(rmax > 0.0 && rmax <= 1.0))
    return fail(ctx, STRP_EINVAL, "alloc_softmax: need temperature > 0, 0 <= rbar <= 1, 0 < rmax <= 1");
  return launch_alloc(ctx, energies, L, n_units, group_id, rbar, temperature, rmax, 0, r_out, nprune_out);
}

size_t strp_topk_workspace_bytes(int32_t n) {
  const size_t b = n > 0 ? topk_scratch_bytes(n) : 0;
  return b ? b + 512 : 0;
}

strp_status strp_mask_topk_static(strp_ctx* ctx, const float* score, int32_t n, int32_t k, uint8_t* mask, int32_t* idx, float* tau) {
  if (!ctx) return STRP_EINVAL;
  if (!score || !mask || !idx) return fail(ctx, STRP_EINVAL, "mask_topk_static: null argument");
  if (n <= 0 || k < 0 || k > n) return fail(ctx, STRP_EINVAL, "mask_topk_static: need n > 0 and 0 <= k <= n");
  if (n > STRP_TOPK_STATIC_MAX_N)
    return fail(ctx, STRP_EINVAL, "mask_topk_static: %d scores exceed the static scratch (at most %d); use strp_mask_topk with a workspace",
                n, (int)STRP_TOPK_STATIC_MAX_N);
  const size_t need = (k > 0 && k < n) ? topk_scratch_bytes(n) : 0;
  if (need > TOPK_STATIC_BYTES) return fail(ctx, STRP_EINVAL, "mask_topk_static: %zu bytes of scratch needed, %zu held", need, TOPK_STATIC_BYTES);
  void* scratch = ctx->device < MAX_DEVICES ? g_topk_scratch[ctx->device] : nullptr;
  if (need && !scratch) return fail(ctx, STRP_ESTATE, "mask_topk_static: no static scratch resolved for device %d", ctx->device);
  // no timing records here: they would create HIP events
  Profiler* pr = ctx->prof;
  const bool was_on = pr && pr->on;
  if (pr) pr->on = false;
  const strp_status st = launch_topk(ctx, score, n, k, 1, mask, idx, tau, scratch, need);
  if (pr) pr->on = was_on;
  return st;
}

}  // extern "C"

namespace strp {

static inline int planes_for(int dtype, int prec) { return (dtype == STRP_F32 && prec == STRP_PREC_SPLIT) ? 2 : 1; }
// the operand as product `prod` of strp_admm_step is set to see it: without its lo plane when one plane was asked for
static inline PlaneOp operand_for(const strp_ctx* ctx, int prod, int side, const PlaneOp& op) {
  PlaneOp o = op;
  if (ctx->prod_planes[prod][side] < 2) o.lo = nullptr;
  return o;
}

// Planes of `rows` (optionally gathered) activation rows for a product that contracts over the tokens.
static strp_status make_t_planes(strp_ctx* ctx, Arena& arena, const void* src, int dtype, long long lds, const int* idx, int rows,
                                 long long T, int relu, int np, PlaneOp* out) {
  const size_t n = plane_elems(rows, T);
  STRP_TAKE(ctx, arena, hi, unsigned short, n);
  unsigned short* lo = nullptr;
  if (np == 2) {
    STRP_TAKE(ctx, arena, lo2, unsigned short, n);
    lo = lo2;
  }
  STRP_TRY(split_act(ctx, src, dtype, lds, idx, rows, T, relu, 0, hi, lo, nullptr, nullptr));
  *out = PlaneOp{hi, lo, plane_kg(T), (rows + 127) / 128, nullptr};
  return STRP_OK;
}

// Planes of `rows` (optionally gathered) activation rows for a product that contracts over those rows.
static strp_status make_c_planes(strp_ctx* ctx, Arena& arena, const void* src, int dtype, long long lds, const int* idx, int rows,
                                 long long T, int relu, int np, PlaneOp* out) {
  const size_t n = plane_elems(T, rows);
  STRP_TAKE(ctx, arena, hi, unsigned short, n);
  unsigned short* lo = nullptr;
  if (np == 2) {
    STRP_TAKE(ctx, arena, lo2, unsigned short, n);
    lo = lo2;
  }
  STRP_TRY(split_act(ctx, src, dtype, lds, idx, rows, T, 0, relu, nullptr, nullptr, hi, lo));
  *out = PlaneOp{hi, lo, plane_kg(rows), (int)((T + 127) / 128), nullptr};
  return STRP_OK;
}

// Room for the planes of a small matrix (weights; k = column, r = row), scaled by the power of two that *maxbits calls for.
static strp_status weight_planes(strp_ctx* ctx, Arena& arena, const void* src, int src_kind, long long lds, int rows, int cols,
                                 int transpose, int np, const unsigned int* maxbits, PlaneOp* out, SplitJob* job) {
  const size_t n = plane_elems(rows, cols);
  STRP_TAKE(ctx, arena, hi, unsigned short, n);
  unsigned short* lo = nullptr;
  if (np == 2) {
    STRP_TAKE(ctx, arena, lo2, unsigned short, n);
    lo = lo2;
  }
  *out = PlaneOp{hi, lo, plane_kg(cols), (rows + 127) / 128, maxbits};
  *job = SplitJob{src, lds, src_kind, rows, cols, transpose, maxbits, hi, lo};
  return STRP_OK;
}

// The fewest K splits a token-contraction product may have, and with them its longest accumulation chain.  The partials are
// added in fp64, so the error of a Gram matrix or right-hand side is that of one fp32 accumulation chain, which grows with its
// length, and the ridge system passes it on to the weights by its condition: with chains of 5472, 3872 and 2752 tokens the
// Gram of 1536 rows over 65536 tokens is 2.1e-7, 1.6e-7 and 1.1e-7 from the fp64 sum, and the fc2 weights of that module
// 1.31e-5, 0.99e-5 and 0.66e-5.  So a chain has at most 8192 tokens, and no more than the splits leave it that give
// the chip 1024 workgroups, down to 256 tokens (up to a quarter more splits where that makes fewer or shorter rounds of a
// grid of at most two).
static int fewest_splits(const GemmP& p, long long* chain) {
  GemmP q = p;
  gemm_plan_tiles(q, 1, 4);
  const long long n4 = q.ntiles;
  const bool ok4 = gemm_tile256_ok(p);
  gemm_plan_tiles(q, 1, 2);
  const long long n2 = q.ntiles, n = ok4 && n4 >= 192 ? n4 : n2;
  const long long s_chain = (p.K + 8191) / 8192, s_fill = (1024 + n - 1) / n, s_max = p.K >= 512 ? p.K / 256 : 1;
  long long s = s_chain > s_fill ? s_chain : s_fill;
  if (s > s_max) s = s_max;
  // rounds x chain of s splits
  auto plan = [&](long long s_) {
    gemm_plan_tiles(q, (int)s_, ok4 && n4 * s_ >= 192 ? 4 : 2);
    const long long slots = q.wt == 4 ? 256 : 512;
    return (double)(((long long)q.ntiles * q.splits + slots - 1) / slots) * (double)q.kchunk;
  };
  double cost = plan(s);
  long long best = s;
  if (s > 1 && (long long)q.ntiles * q.splits <= (q.wt == 4 ? 512 : 1024))
    for (long long c = s + 1; c <= s + s / 4; ++c) {
      const double cc = plan(c);
      if (cc < cost * 0.995) {
        cost = cc;
        best = c;
      }
    }
  plan(best);
  *chain = q.kchunk;
  return q.splits;
}

// Tile shape and K splits of a token-contraction product: fewest_splits or more.  Beyond that the split count is a matter of
// how well the workgroups fill the chip: 256 run at a time with 256x256 tiles, 512 with 128x128 ones, so the candidates are
// the counts that just fill a number of rounds, and the cheapest of them is taken.  Costs are in contraction steps of 32 by one workgroup with 256x256 tiles (about 2.1 us with
// four operand planes), fitted to sweeps over 126 .. 2048 workgroups: such a workgroup spends 7 of them on its first loads
// and its epilogue; one of two with 128x128 tiles takes 1.5 times as long for the same area (its operands pass through
// registers) and loses 4 steps of 64; a partial costs what it takes to read it back.  Against every allowed count with either
// tile, Gram matrices of 16 shapes from 128 x 2000 to 4915 x 32768 are within 5 % of the best (1536 x 65536: 431 us with 24
// splits, 455 with 21; 832 x 65536 201 with 50, 206 with 46), but for 300 rows, which 256-row tiles pad to 512 (300 x 100000:
// 133 us, 106 with 128-row tiles).
static void plan_nt_product(GemmP& p) {
  long long chain;
  const long long s_min = fewest_splits(p, &chain), s_max = p.K / 256 > s_min ? p.K / 256 : s_min;
  const double area = 16384.0 * (double)((p.M + 127) / 128) * (double)((p.N + 127) / 128) * (p.triangle ? 0.5 : 1.0);
  double best_cost = 0.0;
  GemmP best;
  for (int wt = 4; wt >= 2; wt -= 2) {
    if (wt == 4 && !gemm_tile256_ok(p)) continue;
    const long long slots = wt == 4 ? 256 : 512;
    GemmP q = p;
    gemm_plan_tiles(q, 1, wt);
    const long long r0 = (q.ntiles * s_min + slots - 1) / slots;
    for (long long r = r0 - 1; r < r0 + 8; ++r) {     // the first is fewest_splits itself
      long long s = r * slots / q.ntiles;
      s = s < s_min ? s_min : (s > s_max ? s_max : s);
      // a chunk is rounded up to stages of the tile
      do gemm_plan_tiles(q, (int)s++, wt); while (q.kchunk > chain && q.kchunk > 64);
      const double rounds = (double)(((long long)q.ntiles * q.splits + slots - 1) / slots);
      const double steps = wt == 4 ? (double)q.kchunk / 32.0 + 7.0 : 1.5 * ((double)q.kchunk / 64.0 + 4.0);
      const double cost = rounds * steps + (double)q.splits * area / 1.2e6;
      if (best_cost == 0.0 || cost < best_cost * 0.995) {
        best_cost = cost;
        best = q;
      }
    }
  }
  p = best;
}

static size_t nt_splits(int M, int N, long long K, int triangle) {
  GemmP p;
  memset(&p, 0, sizeof(p));
  p.M = M; p.N = N; p.K = K; p.triangle = triangle;
  plan_nt_product(p);
  return (size_t)p.splits;
}
static size_t nt_partial_elems(int M, int N, long long K, int triangle) { return nt_splits(M, N, K, triangle) * (size_t)M * (size_t)N; }
// Most elements the split partials take where M or N or both (given as 0) are kept units, at most km of them.  The split count
// is not monotone in their number; it changes between steps of 128 and at 256 (gemm_tile256_ok).
static size_t nt_partial_most(int M, int N, long long K, int km) {
  size_t most = 0;
  for (int k0 = 0; k0 < km; k0 += 128) {
    const int k1 = k0 + 128 < km ? k0 + 128 : km;
    auto at = [&](int k) {
      const size_t e = nt_splits(M ? M : k, N ? N : k, K, !M && !N) * (size_t)(M ? M : k1) * (size_t)(N ? N : k1);
      most = e > most ? e : most;
    };
    at(k1);
    if (k1 == 256) at(255);
  }
  return most;
}
// The same for W W^T of d rows, a contraction over the kept units rounded up to 8: chunks go by stages of 32, the most splits by 256.
static size_t nt_partial_most_over(int d, long long km) {
  size_t most = 0;
  auto at = [&](long long k) {
    const size_t e = nt_partial_elems(d, d, k, 1);
    most = e > most ? e : most;
  };
  for (long long k = 32; k < km + 32; k += 32) {
    at(k);
    if (k % 256 == 0) at(k - 8);
  }
  return most;
}

// C = P Q^T over K (ROW planes), planned; `room` elements for its partials
static GemmP nt_plan(const PlaneOp& P, const PlaneOp& Q, int M, int N, long long K, int triangle, size_t room) {
  GemmP p;
  memset(&p, 0, sizeof(p));
  p.P = P; p.Q = Q; p.M = M; p.N = N; p.K = K; p.triangle = triangle;
  p.epi = EPI_PARTIAL;
  plan_nt_product(p);
  // a workspace below strp_workspace_bytes may hold fewer partials than the plan's: as many as fit, but no chain longer than
  // 8192 tokens
  const long long chain = (K + 8191) / 8192, fit = (long long)room / ((long long)M * N);
  if (fit < p.splits && p.splits > chain) gemm_plan_tiles(p, (int)(fit > chain ? fit : chain), p.wt);
  gemm_small_tiles(p);
  return p;
}
static void reduce_of(const GemmP& p, ReduceP* r) {
  r->part = p.out; r->splits = p.splits; r->M = p.M; r->N = p.N; r->triangle = p.triangle;
}
// The product's partials in the arena (by value: released on return), fp64 reduction into what r names.
static strp_status nt_product(strp_ctx* ctx, Arena arena, const PlaneOp& P, const PlaneOp& Q, int M, int N, long long K, int triangle, ReduceP r) {
  GemmP p = nt_plan(P, Q, M, N, K, triangle, arena.room() / sizeof(float));
  STRP_TAKE(ctx, arena, part, float, (size_t)p.splits * M * N);
  p.out = part;
  STRP_TRY(launch_gemm(ctx, p));
  reduce_of(p, &r);
  return launch_splitk_reduce(ctx, r);
}
// Whether n <= 3 such products can share their launches: all are small ones and the arena holds all their partials.  Places these.
static bool group_fits(Arena arena, GemmP* p, ReduceP* r, int n) {
  for (int i = 0; i < n; ++i) {
    p[i].out = gemm_is_small(p[i]) ? (float*)arena.take(sizeof(float) * (size_t)p[i].splits * p[i].M * p[i].N) : nullptr;
    if (!p[i].out) return false;
    reduce_of(p[i], &r[i]);
  }
  return true;
}
static ReduceP reduce_to(double* outd, long long ldod) {
  ReduceP r;
  memset(&r, 0, sizeof(r));
  r.outd = outd; r.ldod = ldod;
  return r;
}
// a system that factor_and_invert takes next: with the zeros that chol_inverse wants, where the one launch keeps its counters
static ReduceP reduce_to_system(double* sys, long long ld) {
  ReduceP r = reduce_to(sys, ld);
  r.factored = 1;
  return r;
}

// Leading dimension of the fc2 system of a step, its factor and both sides of its solve.  The pruned rows' pass runs beside the
// factorisation, and tiles that share cache lines are read past the caches, from the memory that the pass is bound by; so rows are whole
// lines wherever the workspace holds them beside the partials of every product's plan (np: planes per operand).  us of the
// factorisation with its pass, rows padded to 8 / 16, and as a launch per panel:  kept 1000 of 2312 over 30011 tokens 331 / 193, 290;
// 1160 of 3072 over 65536 512 / 357, 527; 1544 of 4096 744 / 498, 728; 2056 648 / 633, 857; 3281 of 8192 2113 / 1691, 2043; 4915 of 16384 over
// 131072 5589 / 5501, 7054.  The factor's bits are the same.
static long long system_ld(Arena a, int d, int s, long long T, int np) {
  const long long ld = round_up(s, 16);
  if (ld == f64_ld(s)) return ld;
  bool fits = true;
  auto take = [&](Arena& from, size_t bytes) { fits = from.take(bytes) && fits; };
  take(a, 8 * (size_t)s * ld);
  for (int i = 0; i < np; ++i) take(a, 2 * plane_elems(s, T));
  Arena gram = a;
  take(gram, 4 * nt_partial_elems(s, s, T, 1));
  take(a, 8 * (size_t)s * ld);
  take(a, 8 * (size_t)d * ld);
  Arena chain = a;
  take(chain, 8 * chol_scratch_elems(s));
  take(a, 8 * (size_t)d * ld);
  take(a, 4 * nt_partial_elems(d, s, T, 0));
  return fits ? ld : f64_ld(s);
}

// Work of one call on the context's second stream, beside what the call's own stream does meanwhile.  A factorisation is a chain of
// dependent pivots that holds a few dozen CUs; in one launch it keeps them while the kernels of the other stream run on the rest,
// where its launches per panel would each wait for CUs again.  Which of the two a system takes is chol_inverse's to say, with company or without, so that
// the factor's bits depend neither on the room in the workspace nor on whether there is a second stream.  An order that takes launches per panel where no pass
// rides along (chol_by_order) stays in turn (us, in turn / beside those launches:  an initialisation of 4096 x 16384 over 2048 tokens 3299 / 3273, 5504 x 8000
// over 8000 6795 / 6839, refits of 512 x 4096 over 5000 2271 / 2251, 4096 x 4096 over 65536 8381 / 8435), but for M's, beside which E runs in any case
// (d = 4096, 4915 kept units over 2048 and 16384 tokens 13.04 / 12.99 and 20.22 / 20.16 ms).  HIP maps all streams of a process to four hardware queues; where both
// of a context's come to lie on one, what is meant to be beside runs in turn, with the fewer workgroups: slower, with the same results.
// The call's own stream has waited for the other one when the call returns, so that to the caller everything is on his stream, captured or not.
struct Aside {
  strp_ctx* const ctx;
  hipStream_t const own;
  bool open = false;
  explicit Aside(strp_ctx* c) : ctx(c), own(c->stream) {}
  ~Aside() {
    (void)join();
  }
  Aside(const Aside&) = delete;
  Aside& operator=(const Aside&) = delete;
  // whether there is a second stream; none is made while the call is being captured
  bool ready() const {
    if (ctx->side_state == 0) {
      hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
      if (hipStreamIsCapturing(own, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return false;
      }
      // streams and events belong to the device that is current in the calling thread as they are made, which need not be the context's
      int current = 0;
      const bool known = hipGetDevice(&current) == hipSuccess;
      ctx->side_state = known && hipSetDevice(ctx->device) == hipSuccess && make() ? 1 : -1;
      if (known) (void)hipSetDevice(current);
      if (ctx->side_state < 0) (void)hipGetLastError();
    }
    return ctx->side_state > 0;
  }
  // The events order kernels of one device: no fence for the host or for other devices.  What makes the results of one stream visible to the other is then
  // what does so from kernel to kernel within a stream, the release at device scope as a kernel ends and the acquire as the next begins: that is relied on.
  // us a call with this flag / with hipEventReleaseToDevice / with neither:  a step of 440 x 600 over 9000 tokens 457 / 465 / 461, a head pruning of
  // 1280 x 512 over 20000 283 / 290 / 289.
  bool make() const {
    const unsigned int flags = hipEventDisableTiming | hipEventDisableSystemFence;
    if (hipStreamCreateWithFlags(&ctx->side, hipStreamNonBlocking) != hipSuccess) return false;
    if (hipEventCreateWithFlags(&ctx->side_event[0], flags) == hipSuccess) {
      if (hipEventCreateWithFlags(&ctx->side_event[1], flags) == hipSuccess) return true;
      (void)hipEventDestroy(ctx->side_event[0]);
    }
    (void)hipStreamDestroy(ctx->side);
    return false;
  }
  // what follows on `to` waits for what `from` has been given so far
  strp_status order(hipStream_t from, hipStream_t to, int e) {
    if (hipEventRecord(ctx->side_event[e], from) != hipSuccess || hipStreamWaitEvent(to, ctx->side_event[e], 0) != hipSuccess)
      STRP_HIP(ctx, hipStreamSynchronize(from));
    return STRP_OK;
  }
  strp_status follow() {          // the second stream waits for the call's own
    open = true;
    return order(own, ctx->side, 0);
  }
  strp_status await() { return order(ctx->side, own, 1); }
  strp_status join() {            // ... and this is all it was given
    leave();
    const bool had = open;
    open = false;
    return had ? await() : STRP_OK;
  }
  void enter() { ctx->stream = ctx->side; }
  void leave() { ctx->stream = own; }
};

// How long things take, in us, as far as the choice between two ways of doing them needs it.
// Factor + inverse in one launch of that many workgroups, alone: the chain of its pivots, and tasks that grow as the cube of the order.  Measured / so, with 64, 128,
// 192 and 256 of them:  1000 192 / 206, 179 / 181, 181 / 172, 179 / 168;  2048 830 / 798, 540 / 561, 427 / 481, 377 / 441;  3277 2541 / 2652, 1584 / 1609, 1297 / 1260, 1100 /
// 1086;  4915 7400 / 7707, 4459 / 4320, 3359 / 3191, 2736 / 2626;  6144 13889 / 14377, 7622 / 7804, 6787 / 5613, 5149 / 4517;  7800 28.0 / 28.9, 14.7 / 15.2, 11.1 / 10.7, 9.2 / 8.5 ms.
// It goes in steps, by how many stages of tasks the workgroups hold at a time.
static double flow_us(int n, int workers) {
  const double N = (n + NB - 1) / NB;
  return 16.0 + 7.5 * N + 0.06 * N * N + 0.95 * N * N * N / workers;
}
constexpr double LAUNCH_US = 8.0;      // a small one with its gap
static double pass_us(double bytes) { return bytes / 5e6; }
static double product_us(double m, double n, double k, int passes) { return 2.0 * passes * m * n * k / 1.2e9; }      // 1.2 PFLOP/s executed
// ... over the tokens, which are split, with its reduction; over units or channels, which are not: a tile takes 0.9 us for 64 of them
static double nt_us(double m, double n, double T, int passes) { return product_us(m, n, T, passes) + 2.0 * LAUNCH_US; }
static double nn_us(double m, double T, double k, int passes) {
  const double us = product_us(m, T, k, passes);
  return (us > 0.014 * k ? us : 0.014 * k) + LAUNCH_US;
}
// planes of Z_S both ways, right-hand side, the two triangular products with H's factor, planes of the weights
static double fc1_us(int d, int s, long long T, int planes, int planes_x) {
  return pass_us(12.0 * s * (double)T) + nt_us(s, d, (double)T, planes + planes_x - 1) + 2.0 * s * (double)d * d / 5.5e7 + 4.0 * LAUNCH_US;
}
// the weights' largest magnitudes and planes, Z0 with A and Z, Y and its planes
static double targets_us(int d, int f, long long T, int planes_w, int planes_x, int planes_a) {
  return pass_us(24.0 * f * (double)T + 12.0 * planes_w * f * (double)d) + nn_us(f, (double)T, d, planes_w + planes_x - 1) +
         nn_us(d, (double)T, f, planes_w + planes_a - 1) + 3.0 * LAUNCH_US;
}
// E, one plane of it turned, E E^T
static double residual_us(int d, int s, long long T, int planes) {
  return nn_us(d, (double)T, s, 2 * planes - 1) + pass_us(4.0 * d * (double)T) + 0.5 * product_us(d, d, (double)T, 1) + 3.0 * LAUNCH_US;
}

// Workgroups of a factorisation that has other_us of kernels beside it: a workgroup holds a CU, waiting or not, and the others work on the rest.  So
// it ends no earlier than it would alone on that many, nor before the others have had their time on what CUs it left them.  Four a tile row or 128 are enough for
// the chain of pivots, 192 where an order has work for more; 0: all of them, where what fewer cost is more than what they let the others hide.  A choice has to
// be ahead of the one before by a twentieth of the factorisation (step of 1000 x 1000 over 1000, 64 / 192 workgroups, 640 / 660).  us, all / 128 / 192 / this rule's:
//   refits, rows x order over the tokens:  64 x 1500, 20000 395 / 367 / 344 / 192;  512 x 2500, 5000 820 / 988 / 860 / all;  2048 x 2500, 8000 1236 / 1283 / 1152 / 192;  64 x 5000, 4000
//   3224 / 5006 / 3842 / all;  2048 x 3000, 30000 2185 / 2041 / 2158 / 128;  4096 x 5000, 16000 7566 / 8496 / 6790 / 192;  128 x 7168, 8000 7790 / 12160 / 9633 / all;
//   initialisations, d x f:  2048 x 8192, 2048 838 / 697 / 791 / 128;  3968 x 8000, 4000 2624 / 3187 / 2464 / 192;  5120 x 20480, 2048 5427 / 5756 / 4967 / 192, over
//   8192 8970 / 7642 / 7960 / 128;  6144 x 6144, 2048 6189 / 8209 / 7299 / all;  7168 x 28672, 8000 18.2 / 16.1 / 16.2 / 128 ms;
//   steps, d x kept units:  2048 x 3277, 4096 4229 / 3912 / 3897 / 128;  2560 x 5000, 10000 11403 / 10972 / 10577 / 128;  3000 x 7800, 5000 23.6 / 26.6 / 21.7 / 192 ms;
//   1024 x 8000, 3000 14.1 / 21.1 / 15.5 / all.
// Up to some 1600 four a tile row:  440 alone with 16, 32, 64, 128 and 255 of them 83 / 83 / 82 / 82 / 82, 600 139 / 115 / 112 / 112 / 112, 1000 392 / 262 / 191 / 175 / 174;
// a step with 48, 64, 80, 96, 128 and 192 for the fc2 system  768 x 1536 over 16384 1389 / 1312 / 1288 / 1323 / 1328 / 1392, 1600 x 2500 over 8000 3574 / 3274 / 3227 /
// 2946 / 2877 / 2908, 2048 x 3277 over 65536 15728 / 15539 / 15531 / 15521 / 15574 / 15900.
static int flow_workers_beside(int n, double other_us) {
  const int few = 4 * ((n + NB - 1) / NB);
  const int choice[2] = {few < 128 ? few : 128, 192};
  const double sure = 0.05 * flow_us(n, 256);
  double least = flow_us(n, 256) + other_us;
  int workers = 0;
  for (int w : choice) {
    const double alone = flow_us(n, w), both = other_us + alone * w / 256.0, us = alone > both ? alone : both;
    if (us < least - sure) {
      least = us;
      workers = w;
    }
  }
  return workers;
}
struct FlowWorkers {
  strp_ctx* const ctx;
  FlowWorkers(strp_ctx* c, int w) : ctx(c) { c->flow_workers = w; }
  ~FlowWorkers() { ctx->flow_workers = 0; }
};

// Solve Wsub (Gram + lam I) = R with R = Lhs Rhs^T over the tokens.
struct RefitIn {
  const float* Gram; long long ldg;       // fp32 Gram (used when sys_ready == 0)
  long long ld;                           // leading dimension of sys and R
  double* sys; int sys_ready;             // [n x ld] fp64 scratch: 0 = empty, 1 = holds Gram + lam I
  double* Linv; long long ldl; int linv_ready;   // [n x ldl] fp64 inverse of the Cholesky factor (output, or input if linv_ready)
  double lam; const double* lam_dev;
  PlaneOp Lhs, Rhs;
  int m, n; long long T;
  double* R; int r_ready;                 // [m x ld] the right-hand side (null: taken from the arena); 1: it has been formed
};

// Factor the system in `sys` (leading dimension ld, holds Gram + lam I from reduce_to_system or f32_to_f64_ridge) and leave the inverse of its Cholesky factor in Linv.
static strp_status factor_and_invert(strp_ctx* ctx, Arena arena, double* sys, int n, long long ld, double* Linv, long long ldl) {
  STRP_TAKE(ctx, arena, sub, double, chol_scratch_elems(n));
  return chol_inverse(ctx, sys, n, ld, sub, Linv, ldl, ctx->status_dev);
}

// clear: bytes of out.W to zero first, once everything of the caller's has been read (W may be the array that holds Gram)
static strp_status ridge_solve(strp_ctx* ctx, Arena& arena, const RefitIn& in, const WeightsOut& out, size_t clear = 0) {
  const int n = in.n, m = in.m;
  const long long ld = in.ld;
  const bool factor = !in.linv_ready;
  if (factor) {
    if (in.sys_ready == 0) STRP_TRY(f32_to_f64_ridge(ctx, in.Gram, in.ldg, in.sys, ld, n, in.lam, in.lam_dev));
    STRP_TRY(factor_and_invert(ctx, arena, in.sys, n, ld, in.Linv, in.ldl));
  }
  double* R = in.R;
  if (!R) {
    STRP_TAKE(ctx, arena, R_, double, (size_t)m * ld);
    R = R_;
  }
  STRP_TAKE(ctx, arena, tmp, double, (size_t)m * ld);
  if (!in.r_ready) STRP_TRY(nt_product(ctx, arena, in.Lhs, in.Rhs, m, n, in.T, 0, reduce_to(R, ld)));
  if (clear) STRP_TRY(fill_zero(ctx, out.W, clear));
  return apply_inverse_right(ctx, in.Linv, n, in.ldl, R, m, ld, tmp, out);
}

// Both refits of a small module: their products, reductions and solves are independent of each other, and each leaves most of the
// chip idle, so they share launches: 26 instead of 32 in an iteration of a 64 x 256 module over 512 tokens, 218 -> 190 us.
// One refit after the other / both together, us a step of d x kept units over the tokens, fp32 inputs:  64 x 128, 512 206 / 174;
// 128 x 256, 2048 281 / 248;  200 x 400, 1500 380 / 339;  256 x 512, 2048 399 / 355;  512 x 512, 512 463 / 416;  512 x 1000, 1024 622 / 583;
// 64 x 1000, 512 456 / 423;  768 x 600, 768 596 / 553.  The same with bf16 inputs, and 4 to 12 % with one plane per operand.  More tokens
// have products that fill the chip by themselves (gemm_is_small): 256 x 512, 8192 take them one by one.
// Y, X: the cached planes; Linv1: the inverse factor of the fc1 system.
struct RefitsIn {
  const float* A; const float* Z; long long lda; const int* idx;
  int s, d; long long T;
  int planes;
  PlaneOp Y, X;
  const double* Linv1; const double* lam2_dev;
  const FillRange* clear;      // three ranges that the step needs cleared (refit_both)
};
// *done: 0 = not small, or no room for what both hold at a time (the workspace of one refit after the other stays enough);
// nothing was launched and nothing taken.  Otherwise *Zk: the planes of relu(Z_S) by channels, kept in the arena.
static strp_status refit_both(strp_ctx* ctx, Arena& arena, const RefitsIn& in, const WeightsOut& w2, const WeightsOut& w1, PlaneOp* Zk, int* done) {
  const int s = in.s, d = in.d;
  const long long T = in.T, lds = f64_ld(s), ldd = f64_ld(d);
  *done = 0;
  if (!solve_is_small(d, s) || !solve_is_small(s, d)) return STRP_OK;
  Arena keep = arena;
  bool ok = true;
  auto planes = [&](Arena& from, long long r, long long k) {
    PlaneOp op{(unsigned short*)from.take(2 * plane_elems(r, k)), nullptr, plane_kg(k), (int)((r + 127) / 128), nullptr};
    if (in.planes == 2) op.lo = (unsigned short*)from.take(2 * plane_elems(r, k));
    ok = ok && op.hi && (op.lo || in.planes < 2);
    return op;
  };
  const PlaneOp Zc = planes(keep, T, s);
  Arena a2 = keep;
  auto matrix = [&](int rows, long long ld) {
    double* m = (double*)a2.take(sizeof(double) * (size_t)rows * ld);
    ok = ok && m;
    return m;
  };
  const PlaneOp At = planes(a2, s, T), Zt = planes(a2, s, T);
  double* const G = matrix(s, lds);
  double* const Ginv = matrix(s, lds);
  double* const R2 = matrix(d, lds);
  double* const R1 = matrix(s, ldd);
  double* const tmp2 = matrix(d, lds);
  double* const tmp1 = matrix(s, ldd);
  if (!ok || a2.room() < chol_scratch_elems(s) * sizeof(double)) return STRP_OK;
  const size_t room = a2.room() / sizeof(float);
  GemmP p[3] = {nt_plan(operand_for(ctx, STRP_PROD_GRAM, 0, At), operand_for(ctx, STRP_PROD_GRAM, 1, At), s, s, T, 1, room),
                nt_plan(operand_for(ctx, STRP_PROD_RHS2, 0, in.Y), operand_for(ctx, STRP_PROD_RHS2, 1, At), d, s, T, 0, room),
                nt_plan(operand_for(ctx, STRP_PROD_RHS1, 0, Zt), operand_for(ctx, STRP_PROD_RHS1, 1, in.X), s, d, T, 0, room)};
  ReduceP r[3] = {reduce_to_system(G, lds), reduce_to(R2, lds), reduce_to(R1, ldd)};
  r[0].ridge_dev = in.lam2_dev;
  if (!group_fits(a2, p, r, 3)) return STRP_OK;
  *done = 1;
  arena = keep;
  *Zk = Zc;
  STRP_TRY(split_act_pair(ctx, in.A, in.Z, in.lda, in.idx, s, T, At, Zt, Zc, in.clear));
  STRP_TRY(launch_gemm_group(ctx, p, 3));
  STRP_TRY(launch_splitk_reduce_group(ctx, r, 3));
  STRP_TRY(factor_and_invert(ctx, a2, G, s, lds, Ginv, lds));
  return apply_inverse_right_pair(ctx, SolveIn{Ginv, s, lds, R2, d, lds, tmp2, w2}, SolveIn{in.Linv1, d, d, R1, s, ldd, tmp1, w1});
}

// A refit by itself: what runs beside the factorisation is the planes of both sides and their product, where they take longer (25 us) than the
// two waits.  us of a head pruning's four calls, one after the other / so:  2048 rows x 832 kept over 65536 tokens, bf16 1112 / 1016, 2240 x 960, 20000
// 701 / 614, 800 x 320, 40000, fp32 433 / 398, 2560 x 1152, 100000 2314 / 2198, 1024 x 512, 3000 204 / 204.
static double refit_beside_us(int m, int n, long long T, int planes_l, int planes_r) {
  return nt_us(m, n, (double)T, planes_l + planes_r - 1) + pass_us(4.0 * ((double)planes_l * m + (double)planes_r * n) * (double)T);
}
// the block of the M^-1 chain: partials of W W^T, scratch of the factorisation, planes of M^-1
static size_t m_chain_bytes(int d, long long sp) {
  auto al = [](size_t bytes) { return (bytes + 255) & ~size_t(255); };
  return al(nt_partial_elems(d, d, sp, 1) * 4) + al(chol_scratch_elems(d) * 8) + 2 * al(plane_elems(d, d) * 2) + 4096;
}
// What strp_admm_step takes of the arena behind the refits: planes of the weights and of B, M^-1 and what comes of it, sums, E, and E by tokens
static size_t bytes_after_refits(int d, int s, long long T, int np) {
  auto al = [](size_t bytes) { return (bytes + 255) & ~size_t(255); };
  const size_t D = d, S = s, slots = (size_t)((T + 63) / 64);
  return np * (al(2 * plane_elems(D, S)) + 3 * al(2 * plane_elems(S, D))) + al(8 * (size_t)reduce_blocks(d, d)) + 2 * al(8 * D * D) + al(4 * S * D) +
         al(4 * D * D) + al(m_chain_bytes(d, round_up(s, 8))) + al(8 * slots * S) + al(4 * slots * S) + np * al(2 * plane_elems(T, D)) +
         al(2 * plane_elems(D, T)) + al(64 * ((S + 127) / 128) * ((size_t)(T + 127) / 128));
}
// Both refits of a larger module: while the fc2 system is factored on the call's own stream, the second one has the pruned rows' pass, the
// right-hand side of fc2, and all of the fc1 refit.  The own stream waits for R2 and goes on to W2; what the other one has left then runs beside
// that and beside what comes of W2.  us of a step, one after the other / so:  440 x 600 over 9000 tokens 604 / 489, 768 x 1536 over 16384 1564 / 1318, 1600 x 2500
// over 8000 2991 / 2652, 1000 x 1013 over 30011 (fp32, GAIN) 1949 / 1729, 768 x 1536 over 65536 3547 / 3387, 2048 x 3277 over 65536 15740 / 15520.
// What it hides is the factorisations' time, so not where the products' is many times that: 2048 x 3277 over 262144 52.2 / 52.3 ms, 4096 x 4915 over
// 131072 79.3 / 79.8.  Nor where the factorisation is so much that it had better have all of the chip (flow_workers_beside), since the pass can then ride
// along.  The bits are the same.
static bool refits_beside_pay(int d, int s, long long T, int workers) {
  const double N = (s + NB - 1) / NB, factor_us = 11.0 * N + N * N * N / 260.0;
  return product_us(d, s, (double)T, 3) <= 4.0 * factor_us && (workers || !chol_flow_ok(s, 0.0));
}
// later: bytes of the arena that the rest of the step takes.  *done: 0 = nothing was launched or taken.  Otherwise *Zk as in refit_both, *W1p: the
// planes of W1's kept rows, *part: room for partials on the second stream.
static strp_status refits_beside(strp_ctx* ctx, Aside& aside, Arena& arena, const RefitsIn& in, const WeightsOut& w2, const WeightsOut& w1, size_t later,
                                 PlaneOp* Zk, PlaneOp* W1p, Arena* part, int* done) {
  const int s = in.s, d = in.d;
  const long long T = in.T, lds = round_up(s, 16), ldd = f64_ld(d);
  *done = 0;
  const int workers = flow_workers_beside(s, nt_us(d, s, (double)T, 2 * in.planes - 1) + fc1_us(d, s, T, in.planes, in.X.lo ? 2 : 1));
  if (!chol_by_order(s) || !refits_beside_pay(d, s, T, workers) || !aside.ready()) return STRP_OK;
  Arena a = arena;
  bool ok = true;
  auto take = [&](size_t bytes) {
    void* p = a.take(bytes);
    ok = ok && p;
    return p;
  };
  auto planes = [&](long long r, long long k) {
    PlaneOp op{(unsigned short*)take(2 * plane_elems(r, k)), nullptr, plane_kg(k), (int)((r + 127) / 128), nullptr};
    if (in.planes == 2) op.lo = (unsigned short*)take(2 * plane_elems(r, k));
    return op;
  };
  auto matrix = [&](int rows, long long ld) { return (double*)take(sizeof(double) * (size_t)rows * ld); };
  const PlaneOp Zc = planes(T, s), At = planes(s, T), Zt = At;      // A's planes are read by the two products before Z's are written
  double* const G = matrix(s, lds);
  double* const Ginv = matrix(s, lds);
  double* const R2 = matrix(d, lds);
  double* const R1 = matrix(s, ldd);
  double* const tmp2 = matrix(d, lds);
  double* const tmp1 = matrix(s, ldd);
  double* const sub = (double*)take(sizeof(double) * chol_scratch_elems(s));
  const size_t most = ~size_t(0) >> 8;
  const PlaneOp none{nullptr, nullptr, 0, 0, nullptr};
  GemmP p[3] = {nt_plan(operand_for(ctx, STRP_PROD_GRAM, 0, At), operand_for(ctx, STRP_PROD_GRAM, 1, At), s, s, T, 1, most),
                nt_plan(operand_for(ctx, STRP_PROD_RHS2, 0, in.Y), operand_for(ctx, STRP_PROD_RHS2, 1, At), d, s, T, 0, most),
                nt_plan(operand_for(ctx, STRP_PROD_RHS1, 0, Zt), operand_for(ctx, STRP_PROD_RHS1, 1, in.X), s, d, T, 0, most)};
  // The right-hand sides have not all of the CUs: a grid that fills the chip once would take two rounds, of half as high tiles one and a third.  us of a
  // step with 256x256 / 128x256 tiles, the same splits:  440 x 600 over 9000 tokens 484 / 479, 600 x 800 over 9000 714 / 689, 768 x 1536 over 16384
  // 1374 / 1348, 1000 x 1013 over 30011 1811 / 1818, 768 x 1536 over 65536 3512 / 3517.
  for (int i = 1; i < 3; ++i)
    if (p[i].wt == 4) gemm_plan_tiles(p[i], p[i].splits, 3);
  size_t partials = sizeof(float) * (size_t)nt_plan(none, none, d, d, T, 1, most).splits * d * d;      // E E^T
  for (const GemmP& q : p) {
    const size_t b = sizeof(float) * (size_t)q.splits * q.M * q.N;
    partials = b > partials ? b : partials;
  }
  partials = (partials + 255) & ~size_t(255);
  float* const pt = (float*)take(partials);
  if (!ok || a.room() < later) return STRP_OK;
  *done = 1;
  arena = a;
  *Zk = Zc;
  *part = Arena(pt, partials);
  auto product = [&](GemmP& q, ReduceP r) {
    q.out = pt;
    STRP_TRY(launch_gemm(ctx, q));
    reduce_of(q, &r);
    return launch_splitk_reduce(ctx, r);
  };
  STRP_TRY(split_act(ctx, in.A, STRP_F32, in.lda, in.idx, s, T, 0, 0, (unsigned short*)At.hi, (unsigned short*)At.lo, nullptr, nullptr));
  ReduceP g = reduce_to_system(G, lds);
  g.ridge_dev = in.lam2_dev;
  STRP_TRY(product(p[0], g));
  const CoJob* const pass = ctx->cojob;
  ctx->cojob = nullptr;
  // the factorisation first, so that it finds its CUs free
  STRP_TRY(aside.follow());
  {
    const FlowWorkers few(ctx, workers);
    STRP_TRY(factor_and_invert(ctx, Arena(sub, sizeof(double) * chol_scratch_elems(s)), G, s, lds, Ginv, lds));
  }
  aside.enter();
  if (pass) STRP_TRY(launch_cojob(ctx, *pass));
  STRP_TRY(product(p[1], reduce_to(R2, lds)));
  STRP_TRY(aside.await());
  STRP_TRY(split_act(ctx, in.Z, STRP_F32, in.lda, in.idx, s, T, 0, 1, (unsigned short*)Zt.hi, (unsigned short*)Zt.lo, (unsigned short*)Zc.hi, (unsigned short*)Zc.lo));
  STRP_TRY(product(p[2], reduce_to(R1, ldd)));
  STRP_TRY(apply_inverse_right(ctx, in.Linv1, d, d, R1, s, ldd, tmp1, w1));
  SplitJob job;
  STRP_TRY(weight_planes(ctx, arena, w1.Wc, SRC_F32, w1.ldc, s, d, 0, in.planes, w1.maxbits, W1p, &job));
  STRP_TRY(split_small(ctx, &job, 1));
  aside.leave();
  return apply_inverse_right(ctx, Ginv, s, lds, R2, d, lds, tmp2, w2);
}

// Persistent per-module planes (caller-owned strp_module_state::cache), fixed at initialisation:
// Y as ROW planes, X as ROW planes and as K8 planes.
struct CacheView {
  int nx, ny;
  double* rowsums;     // [4][f] scoring sums of the pruned rows, valid as strp_module_state::sums_cached says
  PlaneOp Yt, Xt, Xc;   // Y and X for token-contraction products; X for the channel-contraction product W1 X
};
static size_t cache_layout(const strp_module_desc* desc, int prec, char* base, CacheView* v) {
  const long long d = desc->d, T = desc->T;
  const int nx = planes_for(desc->x_dtype, prec), ny = planes_for(STRP_F32, prec);
  size_t off = 256;
  double* rowsums = (double*)(base ? base + off : nullptr);
  off += ((size_t)desc->f * 4 * sizeof(double) + 255) & ~size_t(255);
  auto take = [&](size_t elems) {
    char* p = base ? base + off : nullptr;
    off += (elems * 2 + 255) & ~size_t(255);
    return (unsigned short*)p;
  };
  unsigned short* yh = take(plane_elems(d, T));
  unsigned short* yl = ny == 2 ? take(plane_elems(d, T)) : nullptr;
  unsigned short* xh = take(plane_elems(d, T));
  unsigned short* xl = nx == 2 ? take(plane_elems(d, T)) : nullptr;
  unsigned short* kh = take(plane_elems(T, d));
  unsigned short* kl = nx == 2 ? take(plane_elems(T, d)) : nullptr;
  if (v) {
    v->nx = nx; v->ny = ny;
    v->rowsums = rowsums;
    v->Yt = PlaneOp{yh, yl, plane_kg(T), (int)((d + 127) / 128), nullptr};
    v->Xt = PlaneOp{xh, xl, plane_kg(T), (int)((d + 127) / 128), nullptr};
    v->Xc = PlaneOp{kh, kl, plane_kg(d), (int)((T + 127) / 128), nullptr};
  }
  return off;
}

}  // namespace strp

extern "C" {

size_t strp_module_cache_bytes(const strp_module_desc* desc) {
  if (!desc || desc->d <= 0 || desc->f <= 0 || desc->T <= 0) return 0;
  return cache_layout(desc, STRP_PREC_SPLIT, nullptr, nullptr);
}

size_t strp_workspace_bytes(const strp_module_desc* desc) {
  if (!desc || desc->d <= 0 || desc->f <= 0 || desc->T <= 0) return 0;
  const size_t d = desc->d, f = desc->f;
  const size_t km = desc->k_max > 0 ? (size_t)desc->k_max : f;
  const size_t kp = (size_t)round_up((long long)km, 8);
  const long long T = desc->T;
  auto al = [](size_t bytes) { return (bytes + 255) & ~size_t(255); };
  const size_t nmax = km > d ? km : d;
  const size_t invd_max = chol_scratch_elems((long long)nmax) * 8;
  const size_t tilesT = (size_t)((T + 127) / 128);
  const size_t red = al((((f + 127) / 128) * tilesT + f + 4096) * 16);
  // initialisation: weight planes, relu(Z0) planes, H partials
  size_t init = 256 + al(256) + 2 * al(plane_elems(f, d) * 2) + 2 * al(plane_elems(d, f) * 2) + 2 * al(plane_elems(T, f) * 2) + red +
                al(nt_partial_elems((int)d, (int)d, T, 1) * 4) + al(d * 8) + al(invd_max) + 2 * al(d * d * 8);
  // one iteration: everything every stage carves (stages reuse the arena, so this is an upper bound)
  size_t part = 0;
  auto upd = [&](size_t e) { if (e > part) part = e; };
  upd(nt_partial_most(0, 0, T, (int)km));
  upd(nt_partial_most((int)d, 0, T, (int)km));
  upd(nt_partial_most(0, (int)d, T, (int)km));
  upd(nt_partial_elems((int)d, (int)d, T, 1));   // H; E E^T of the objective
  const size_t wwt = nt_partial_most_over((int)d, (long long)kp);
  upd(wwt);
  // a small product's partials beside another's (group_fits): at most 256 tiles of 128 x 128
  const size_t part_small = part < ((size_t)256 << 14) ? part : (size_t)256 << 14;
  const size_t segs = (size_t)((T + 8191) / 8192), slots = (size_t)((T + 63) / 64);
  const size_t w_blocks = ((d + 63) / 64 + 1) * ((km + 31) / 32 + 1) + ((km + 63) / 64 + 1) * ((d + 31) / 32 + 1) + 2048;
  size_t step = 256 + al(256) + al(4 * f * 8) +
                /* the refitted weights of the kept units and their sums of squares */
                al(d * kp * 4) + al(km * d * 4) + al(w_blocks * 8) +
                /* the pruned rows' pass: the row list, the units' partial sums, the workgroups' (or the rows') sums */
                al(f * 4) + al(f * segs * 6 * 8) + al(2 * f * 8) +
                /* planes of the kept weights (both orders of W2) and of B */
                2 * al(plane_elems(d, km) * 2) + 3 * 2 * al(plane_elems(km, d) * 2) + al(km * d * 4) +
                /* fc2 and fc1 refit: system and factor, their rows padded to 8, scratch of the chain, right-hand side and solve */
                al(part * 4) + al(part_small * 4) + 3 * al(nmax * (nmax + 8) * 8) + 2 * al(invd_max) + 4 * al(d * km * 8) + 2 * al((d + km) * 8 * 8) + 2 * al(d * d * 8) +
                2 * al(plane_elems(km, T) * 2) /* kept rows, token contraction */ +
                2 * al(plane_elems(T, km) * 2) /* kept rows, channel contraction */ +
                2 * al(plane_elems(T, d) * 2) /* E */ + red +
                /* objective: E by tokens, M^-2, the reduction's sums; without the identity A's plane */
                al(plane_elems(d, T) * 2) + al(d * d * 4) + al((size_t)reduce_blocks((int)d, (int)d) * 8) + al(plane_elems(T, km) * 2) +
                /* M, its factor's inverse, and the block of the M-inverse chain, which stays while the fc1 refit runs */
                2 * al(d * d * 8) + al(wwt * 4) + al(invd_max) + 2 * al(plane_elems(d, d) * 2) + 8192 +
                /* strip sums of the kept rows from the a- and z-update epilogues */
                al(2 * slots * km * 4) + al(slots * km * 4);
  return (init > step ? init : step) + (2 << 20);
}

strp_status strp_gram(strp_ctx* ctx, const void* A, strp_dtype dt, int32_t C, int64_t T, int64_t ldA, const int32_t* idx,
                      int32_t s, float* G, int32_t ldG, double* diag, int accumulate) {
  if (!ctx) return STRP_EINVAL;
  if (!A || !G) return fail(ctx, STRP_EINVAL, "gram: null A or G");
  if (dt != STRP_BF16 && dt != STRP_F32) return fail(ctx, STRP_EINVAL, "gram: unknown dtype");
  if (C <= 0 || s <= 0 || s > C || T <= 0) return fail(ctx, STRP_EINVAL, "gram: need 0 < s <= C and T > 0");
  if (!idx && s != C) return fail(ctx, STRP_EINVAL, "gram: idx == NULL requires s == C");
  if (ldA < T || ldA % 8 || ldG < s) return fail(ctx, STRP_EINVAL, "gram: bad leading dimension");
  if (!aligned16(A)) return fail(ctx, STRP_EINVAL, "gram: A not 16-byte aligned");
  if (!ctx->ws) return fail(ctx, STRP_ENOMEM, "gram: no workspace set");
  Arena arena(ctx);
  PlaneOp op;
  STRP_TRY(make_t_planes(ctx, arena, A, dt, ldA, idx, s, T, 0, planes_for(dt, ctx->precision), &op));
  ReduceP r = reduce_to(nullptr, 0);
  r.outf = G; r.ldof = ldG; r.diag = diag; r.accumulate = accumulate;
  return nt_product(ctx, arena, op, op, s, s, T, 1, r);
}

strp_status strp_refit(strp_ctx* ctx, strp_side side, const float* Gram, int32_t ldg, double lambda, double* chol, int chol_valid,
                       const void* Lhs, strp_dtype lhs_dtype, int64_t ld_lhs, const void* Rhs, strp_dtype rhs_dtype,
                       int64_t ld_rhs, int64_t T, const int32_t* idx, int32_t s, float* W, int32_t out, int32_t in) {
  if (!ctx) return STRP_EINVAL;
  if (side != STRP_SIDE_FC1 && side != STRP_SIDE_FC2) return fail(ctx, STRP_EINVAL, "refit: unknown side");
  if (!Lhs || !Rhs || !W || !idx) return fail(ctx, STRP_EINVAL, "refit: null argument");
  if (out <= 0 || in <= 0 || T <= 0 || s <= 0) return fail(ctx, STRP_EINVAL, "refit: non-positive size");
  if (side == STRP_SIDE_FC2 && s > in) return fail(ctx, STRP_EINVAL, "refit: s > in");
  if (side == STRP_SIDE_FC1 && s > out) return fail(ctx, STRP_EINVAL, "refit: s > out");
  if (ld_lhs < T || ld_rhs < T || ld_lhs % 8 || ld_rhs % 8) return fail(ctx, STRP_EINVAL, "refit: bad leading dimension");
  if (!aligned16(Lhs) || !aligned16(Rhs)) return fail(ctx, STRP_EINVAL, "refit: operands not 16-byte aligned");
  if (chol_valid && !chol) return fail(ctx, STRP_EINVAL, "refit: chol_valid without chol");
  if (!chol_valid && !Gram) return fail(ctx, STRP_EINVAL, "refit: need Gram or a valid factor");
  const int n = side == STRP_SIDE_FC2 ? s : in;
  const int m = side == STRP_SIDE_FC2 ? out : s;
  if (!chol_valid && ldg < n) return fail(ctx, STRP_EINVAL, "refit: ldg below the order of Gram");
  if (!(lambda >= 0.0)) return fail(ctx, STRP_EINVAL, "refit: negative lambda");
  if (!ctx->ws) return fail(ctx, STRP_ENOMEM, "refit: no workspace set");
  Arena arena(ctx);
  RefitIn ri;
  memset(&ri, 0, sizeof(ri));
  ri.Gram = Gram; ri.ldg = ldg; ri.lam = lambda; ri.lam_dev = nullptr;
  // the factorisation wants aligned rows of even length: a caller's cache of odd order gets a copy of the result
  const bool chol_direct = chol && (chol_valid || (n % 2 == 0 && aligned16(chol)));
  if (chol_direct) {
    ri.Linv = chol;
    ri.ldl = n;
  } else {
    STRP_TAKE(ctx, arena, Linv, double, (size_t)n * f64_ld(n));
    ri.Linv = Linv;
    ri.ldl = f64_ld(n);
  }
  ri.linv_ready = chol_valid ? 1 : 0;
  if (!chol_valid) {
    STRP_TAKE(ctx, arena, sys, double, (size_t)n * f64_ld(n));
    ri.sys = sys;
  }
  const int prec = ctx->precision, npl = planes_for(lhs_dtype, prec), npr = planes_for(rhs_dtype, prec);
  ri.m = m; ri.n = n; ri.ld = f64_ld(n); ri.T = T;
  // Neither the planes nor the right-hand side need the factor: they are made on the second stream beside it.  Where the workspace
  // holds everything at once, with all of the product's partials: what is summed in which order does not depend on it.
  Aside aside(ctx);
  const double beside_us = refit_beside_us(m, n, T, npl, npr);
  if (!chol_valid && n >= 2 * NB && chol_by_order(n) && beside_us >= 25.0) {
    Arena a = arena;
    bool fits = true;
    auto take = [&](size_t bytes) { fits = a.take(bytes) && fits; };
    double* const sub = (double*)a.take(sizeof(double) * chol_scratch_elems(n));
    double* const R = (double*)a.take(sizeof(double) * (size_t)m * ri.ld);
    const Arena rest = a;
    for (int i = 0; i < npl; ++i) take(2 * plane_elems(m, T));
    for (int i = 0; i < npr; ++i) take(2 * plane_elems(n, T));
    take(sizeof(double) * (size_t)m * ri.ld);
    take(sizeof(float) * nt_partial_elems(m, n, T, 0));
    if (sub && R && fits && aside.ready()) {
      STRP_TRY(f32_to_f64_ridge(ctx, Gram, ldg, ri.sys, ri.ld, n, lambda, nullptr));
      STRP_TRY(aside.follow());
      {
        const FlowWorkers few(ctx, flow_workers_beside(n, beside_us));
        STRP_TRY(factor_and_invert(ctx, Arena(sub, sizeof(double) * chol_scratch_elems(n)), ri.sys, n, ri.ld, ri.Linv, ri.ldl));
      }
      ri.linv_ready = ri.r_ready = 1;
      ri.R = R;
      arena = rest;
      aside.enter();
    }
  }
  if (side == STRP_SIDE_FC2) {
    STRP_TRY(make_t_planes(ctx, arena, Lhs, lhs_dtype, ld_lhs, nullptr, out, T, 0, npl, &ri.Lhs));
    STRP_TRY(make_t_planes(ctx, arena, Rhs, rhs_dtype, ld_rhs, idx, s, T, 0, npr, &ri.Rhs));
  } else {
    STRP_TRY(make_t_planes(ctx, arena, Lhs, lhs_dtype, ld_lhs, idx, s, T, 0, npl, &ri.Lhs));
    STRP_TRY(make_t_planes(ctx, arena, Rhs, rhs_dtype, ld_rhs, nullptr, in, T, 0, npr, &ri.Rhs));
  }
  if (ri.r_ready) {
    STRP_TRY(nt_product(ctx, arena, ri.Lhs, ri.Rhs, m, n, T, 0, reduce_to(ri.R, ri.ld)));
    STRP_TRY(aside.join());
  }
  STRP_TRY(ridge_solve(ctx, arena, ri, WeightsOut{side, idx, W, in, nullptr, 0, nullptr, nullptr}, sizeof(float) * (size_t)out * (size_t)in));
  return chol && !chol_direct ? copy_f64(ctx, ri.Linv, ri.ldl, chol, n, n) : STRP_OK;
}

strp_status strp_module_init(strp_ctx* ctx, const strp_module_desc* desc, strp_module_state* st, const strp_params* params) {
  if (!ctx) return STRP_EINVAL;
  STRP_TRY(check_desc(ctx, desc));
  if (!st || !params) return fail(ctx, STRP_EINVAL, "module_init: null state or params");
  if (!st->X || !st->W1hat || !st->W2hat || !st->Z || !st->A || !st->Z0 || !st->Y || !st->W1 || !st->W2 || !st->H || !st->cholH ||
      !st->n2 || !st->score || !st->mask || !st->idx || !st->scalars || !st->cache)
    return fail(ctx, STRP_EINVAL, "module_init: null buffer in state");
  if (!aligned16(st->X) || !aligned16(st->W1hat) || !aligned16(st->W2hat) || !aligned16(st->Z) || !aligned16(st->A) ||
      !aligned16(st->Z0) || !aligned16(st->Y) || ((uintptr_t)st->cache & 255u))
    return fail(ctx, STRP_EINVAL, "module_init: buffers must be 16-byte aligned (cache: 256)");
  if (!(params->delta >= 0.0)) return fail(ctx, STRP_EINVAL, "module_init: negative delta");
  if (!ctx->ws) return fail(ctx, STRP_ENOMEM, "module_init: no workspace set");
  const int d = desc->d, f = desc->f;
  const long long T = desc->T, lda = desc->lda;
  const int prec = ctx->precision;
  const int npw = planes_for(desc->w_dtype, prec), npa = planes_for(STRP_F32, prec);
  const int wkind = desc->w_dtype == STRP_BF16 ? SRC_BF16 : SRC_F32;
  CacheView cv;
  cache_layout(desc, prec, (char*)st->cache, &cv);
  Arena arena(ctx);
  double* sc = st->scalars;
  STRP_TAKE(ctx, arena, wmax, unsigned int, 64);
  {
    const FillRange z[2] = {{sc, SC_COUNT * sizeof(double)}, {wmax, 256}};
    STRP_TRY(fill_zero(ctx, z, 2));
  }
  STRP_TRY(launch_colnorm2(ctx, st->W2hat, desc->w_dtype, d, f, f, st->n2));
  // X planes (persistent)
  STRP_TRY(split_act(ctx, st->X, desc->x_dtype, desc->ldx, nullptr, d, T, 0, 0, (unsigned short*)cv.Xt.hi, (unsigned short*)cv.Xt.lo,
                     (unsigned short*)cv.Xc.hi, (unsigned short*)cv.Xc.lo));
  auto al = [](size_t bytes) { return (bytes + 255) & ~size_t(255); };
  const size_t targets_bytes = npw * (al(2 * plane_elems(f, d)) + al(2 * plane_elems(d, f))) + npa * al(2 * plane_elems(T, f)) +
                               al(64 * (((size_t)f + 127) / 128) * (((size_t)T + 127) / 128));
  // Z0, A, Y and Y's planes
  auto targets = [&](Arena a2) -> strp_status {
    PlaneOp W1p, W2p, A0k8;
    SplitJob jobs[2];
    STRP_TRY(weight_planes(ctx, a2, st->W1hat, wkind, d, f, d, 0, npw, wmax, &W1p, &jobs[0]));
    STRP_TRY(weight_planes(ctx, a2, st->W2hat, wkind, f, d, f, 0, npw, wmax + 1, &W2p, &jobs[1]));
    const MaxJob mj[2] = {{st->W1hat, d, wkind, f, d, wmax}, {st->W2hat, f, wkind, d, f, wmax + 1}};
    STRP_TRY(abs_max(ctx, mj, 2));
    STRP_TRY(split_small(ctx, jobs, 2));
    STRP_TAKE(ctx, a2, a0h, unsigned short, plane_elems(T, f));
    unsigned short* a0l = nullptr;
    if (npa == 2) {
      STRP_TAKE(ctx, a2, a0l2, unsigned short, plane_elems(T, f));
      a0l = a0l2;
    }
    A0k8 = PlaneOp{a0h, a0l, plane_kg(f), (int)((T + 127) / 128), nullptr};
    {  // Z0 = W1hat X, Z = Z0, A = relu(Z0) (+ K8 planes of A), sum A^2
      GemmP p;
      memset(&p, 0, sizeof(p));
      p.P = W1p; p.Q = cv.Xc;
      p.M = f; p.N = (int)T; p.K = d;
      p.epi = EPI_INITZ; p.Zs = st->Z; p.As = st->A; p.Z0s = st->Z0; p.lda = lda;
      p.k8_hi = a0h; p.k8_lo = a0l; p.k8_kg = plane_kg(f);
      gemm_plan_tiles(p, 1);
      STRP_TAKE(ctx, a2, red, double, 2 * (size_t)gemm_grid_blocks(p));
      p.red = red;
      STRP_TRY(launch_gemm(ctx, p));
      hipLaunchKernelGGL(scaled_sum_kernel, dim3(1), dim3(1024), 0, ctx->stream, (const double*)red, 2, gemm_grid_blocks(p), params->delta / (double)f,
                         sc + SC_SUMA0, sc + SC_LAM2, (double*)nullptr, 0LL, 0);
    }
    {  // Y = W2hat A
      GemmP p;
      memset(&p, 0, sizeof(p));
      p.P = W2p; p.Q = A0k8;
      p.M = d; p.N = (int)T; p.K = f;
      p.epi = EPI_STORE; p.out = st->Y; p.ldo = lda;
      gemm_plan_tiles(p, 1);
      STRP_TRY(launch_gemm(ctx, p));
    }
    return split_act(ctx, st->Y, STRP_F32, lda, nullptr, d, T, 0, 0, (unsigned short*)cv.Yt.hi, (unsigned short*)cv.Yt.lo, nullptr, nullptr);
  };
  // H = X X^T (fp32 copy and fp64 system), lam1 = delta tr(H)/d
  auto gram = [&](Arena a2, double* diag, double* Hd) -> strp_status {
    ReduceP r = reduce_to_system(Hd, d);
    r.outf = st->H; r.ldof = d; r.diag = diag;
    STRP_TRY(nt_product(ctx, a2, cv.Xt, cv.Xt, d, d, T, 1, r));
    hipLaunchKernelGGL(scaled_sum_kernel, dim3(1), dim3(1024), 0, ctx->stream, (const double*)diag, 1, d, params->delta / (double)d, sc + SC_TRH,
                       sc + SC_LAM1, Hd, (long long)d, d);
    return STRP_OK;
  };
  // factor of H + lam1 I; the chain wants its result 16-byte aligned, cholH need not be: then it goes to scratch first
  auto factor = [&](Arena a2, double* Hd, double* scratch) -> strp_status {
    double* const Linv = scratch ? scratch : st->cholH;
    STRP_TRY(factor_and_invert(ctx, a2, Hd, d, d, Linv, d));
    return scratch ? copy_f64(ctx, Linv, d, st->cholH, d, d) : STRP_OK;
  };
  // The factor needs nothing of the targets, nor they of it: where the workspace holds both they are made beside it on the second stream,
  // behind the product, so that it finds its CUs free (us of the initialisation, 128 x 520 over 1000 tokens 90 -> 85, 440 x 1440, 9000 259 -> 200, 768 x
  // 3072, 16384 639 -> 546, 1000 x 3000, 30000, fp32 1696 -> 1553; 64 x 256, 512 65 either way).
  Aside aside(ctx);
  Arena ah = arena;
  double* const diag = (double*)ah.take(sizeof(double) * (size_t)d);
  double* const Hd = (double*)ah.take(sizeof(double) * (size_t)d * d);
  if (!diag || !Hd) return fail(ctx, STRP_ENOMEM, "workspace too small for H");
  const bool copied = !aligned16(st->cholH);
  Arena both = ah;
  double* const sub = (double*)both.take(sizeof(double) * chol_scratch_elems(d));
  double* scratch = copied ? (double*)both.take(sizeof(double) * (size_t)d * d) : nullptr;
  if (d >= 2 * NB && chol_by_order(d) && sub && (scratch || !copied) && both.room() >= targets_bytes && both.room() >= sizeof(float) * nt_partial_elems(d, d, T, 1) && aside.ready()) {
    STRP_TRY(gram(both, diag, Hd));
    STRP_TRY(aside.follow());
    {
      const FlowWorkers few(ctx, flow_workers_beside(d, targets_us(d, f, T, npw, cv.Xt.lo ? 2 : 1, npa)));
      STRP_TRY(factor(Arena(sub, sizeof(double) * chol_scratch_elems(d)), Hd, scratch));
    }
    aside.enter();
    STRP_TRY(targets(both));
    STRP_TRY(aside.join());
  } else {
    STRP_TRY(targets(arena));
    STRP_TRY(gram(ah, diag, Hd));
    if (copied) {
      STRP_TAKE(ctx, ah, linv, double, (size_t)d * d);
      scratch = linv;
    }
    STRP_TRY(factor(ah, Hd, scratch));
  }
  {  // last: fp32 weights may be refitted in the arrays of the dense ones
    const FillRange z[3] = {{st->W1, sizeof(float) * (size_t)f * d}, {st->W2, sizeof(float) * (size_t)f * d}, {st->mask, (size_t)f}};
    STRP_TRY(fill_zero(ctx, z, 3));
  }
  STRP_HIP(ctx, hipGetLastError());
  st->s = 0;
  st->iter = 0;
  st->sums_cached = 0;
  st->precision = 1 + prec;
  return STRP_OK;
}

strp_status strp_admm_step(strp_ctx* ctx, const strp_module_desc* desc, strp_module_state* st, const strp_params* params,
                           strp_report* report_host) {
  if (!ctx) return STRP_EINVAL;
  STRP_TRY(check_desc(ctx, desc));
  if (!st || !params) return fail(ctx, STRP_EINVAL, "admm_step: null state or params");
  if (!st->X || !st->W2hat || !st->Z || !st->A || !st->Z0 || !st->Y || !st->W1 || !st->W2 || !st->cholH || !st->n2 || !st->score ||
      !st->mask || !st->idx || !st->scalars || !st->cache)
    return fail(ctx, STRP_EINVAL, "admm_step: null buffer in state");
  const int d = desc->d, f = desc->f;
  const long long T = desc->T, lda = desc->lda;
  const int stages = params->stages ? params->stages : 63;
  const bool do_select = (stages & STRP_STAGE_SELECT) && (params->reselect || st->s == 0);
  if (do_select && (params->k <= 0 || params->k > f)) return fail(ctx, STRP_EINVAL, "admm_step: k outside [1, f]");
  if (desc->k_max > 0 && do_select && params->k > desc->k_max) return fail(ctx, STRP_EINVAL, "admm_step: k above desc.k_max");
  if (do_select && f > SELECT_MAX && params->k < f) return fail(ctx, STRP_EINVAL, "admm_step: selects among at most %d units", SELECT_MAX);
  if (!do_select && st->s <= 0) return fail(ctx, STRP_ESTATE, "admm_step: no mask selected yet");
  if (!(params->alpha > 0.0) || !(params->beta > 0.0)) return fail(ctx, STRP_EINVAL, "admm_step: alpha, beta must be positive");
  if (params->mode < STRP_SCORE_WANDA || params->mode > STRP_SCORE_GAIN) return fail(ctx, STRP_EINVAL, "admm_step: unknown score mode");
  if (!ctx->ws) return fail(ctx, STRP_ENOMEM, "admm_step: no workspace set");
  const int prec = ctx->precision;
  // the plane cache was laid out and written under the precision of strp_module_init: another one would read other offsets
  if (st->precision == 0) return fail(ctx, STRP_ESTATE, "admm_step: strp_module_init has not run on this state");
  if (st->precision != 1 + prec)
    return fail(ctx, STRP_ESTATE, "admm_step: the context's precision (%d) differs from the one the module was initialised with (%d)",
                prec, st->precision - 1);
  const int npa = planes_for(STRP_F32, prec);
  CacheView cv;
  cache_layout(desc, prec, (char*)st->cache, &cv);
  double* sc = st->scalars;
  const float alpha = (float)params->alpha, beta = (float)params->beta;
  Arena arena(ctx);

  // ---- S2/S4: scores and top-k ---------------------------------------------------------
  // The token sums every score is built from live in the module cache (cv.rowsums, [4][f]): sum A^2, sum A relu(Z0),
  // sum Z0 Z, sum Z0^2.  A full iteration leaves them there for every row -- the pruned rows' from the pass that writes
  // those rows, the kept rows' from the epilogues of the a- and z-update products (sum Z0^2 never changes after it has
  // been streamed once) -- so that only a selection on a state the library did not produce streams the rows.
  const bool wanda = params->mode == STRP_SCORE_WANDA;
  const bool fuse_pruned = (stages & STRP_STAGE_AUPD) && (stages & STRP_STAGE_ZUPD);
  int32_t* prow = nullptr;
  bool prow_done = false;
  if (fuse_pruned) {
    STRP_TAKE(ctx, arena, prow_, int32_t, (size_t)f);
    prow = prow_;
  }
  if (do_select) {
    const bool have = (st->sums_cached & SUMS_G) && (wanda || ((st->sums_cached & SUMS_EU) && (st->sums_cached & SUMS_V)));
    if (!have) {
      STRP_TRY(launch_row_sums(ctx, st->A, STRP_F32, st->Z, st->Z0, lda, T, f, params->mode, cv.rowsums));
      st->sums_cached = wanda ? (st->sums_cached & SUMS_V) | SUMS_G : SUMS_G | SUMS_EU | SUMS_V;
    }
    STRP_TRY(launch_select(ctx, cv.rowsums, st->n2, params->mode, f, params->k, st->score, sc + SC_ENERGY, st->mask, st->idx, (float*)(sc + SC_TAU), prow));
    st->s = params->k;
    prow_done = true;
  }
  // the sums describe the state as it is now: void them before an update changes it (sum Z0^2 stays valid)
  if (stages & (STRP_STAGE_AUPD | STRP_STAGE_ZUPD)) st->sums_cached &= SUMS_V;
  const int s = st->s;
  const long long sp = round_up(s, 8);

  // ---- everything the step needs cleared, in one launch (that of the small refits' first planes, or its own): the refitted weights outside the kept rows and columns, the
  // maxima of the weights' planes, the finishing kernel's counter
  enum { MAX_W2 = 0, MAX_MI = 1, MAX_B = 2, MAX_W1 = 3 };
  STRP_TAKE(ctx, arena, wmax, unsigned int, 64);
  unsigned int* const ticket = wmax + 32;
  const size_t wbytes = sizeof(float) * (size_t)f * d;
  const FillRange clear[3] = {{wmax, 256}, {st->W2, (stages & STRP_STAGE_REFIT2) ? wbytes : 0}, {st->W1, (stages & STRP_STAGE_REFIT1) ? wbytes : 0}};

  // ---- the pruned rows' fused a/z pass as a ride-along job ------------------------------------------------------
  // It touches only rows outside S, which nothing else in the step reads or writes, so it may run any time from
  // here to the end of the step: the first launch of the step's first factorisation chain carries it (chol_inverse takes
  // ctx->cojob; the a-update, which this pass is fused with, always factors a system).
  struct CoJobGuard {
    strp_ctx* c;
    ~CoJobGuard() { c->cojob = nullptr; }
  } cojob_guard{ctx};
  CoJob pjob;
  memset(&pjob, 0, sizeof(pjob));
  double* finish_blk = nullptr;
  if (fuse_pruned && s < f) {
    constexpr long long SEG = 8192;
    const int segs = (int)((T + SEG - 1) / SEG);
    STRP_TAKE(ctx, arena, partial, double, (size_t)(f - s) * segs * 6);
    STRP_TAKE(ctx, arena, blk, double, 2 * (size_t)finish_row_blocks(f - s));
    finish_blk = blk;
    if (!prow_done) hipLaunchKernelGGL(pruned_list_kernel, dim3(1), dim3(1024), 0, ctx->stream, st->mask, f, prow);
    pjob.units = (unsigned int)(f - s) * (unsigned int)segs;
    pjob.rows = prow; pjob.nrows = f - s; pjob.segs = segs; pjob.seg_tokens = SEG;
    pjob.Z = st->Z; pjob.A = st->A; pjob.Z0 = wanda ? nullptr : st->Z0;
    pjob.lda = lda; pjob.T = T; pjob.alpha = alpha; pjob.beta = beta; pjob.partial = partial;
    ctx->cojob = &pjob;
  }
  // compact kept weights: written by the refits' last products when those run in this call, gathered otherwise
  float* W2S = nullptr;
  float* W1S = nullptr;
  double* w2sq = nullptr;
  double* w1sq = nullptr;
  int nw2 = 0, nw1 = 0;
  if (stages & (STRP_STAGE_AUPD | STRP_STAGE_OBJ)) {
    nw2 = (stages & STRP_STAGE_REFIT2) ? weights_out_blocks(d, s) : gather_blocks(d, s);
    STRP_TAKE(ctx, arena, w2s, float, (size_t)d * sp);
    STRP_TAKE(ctx, arena, w2sq_, double, (size_t)nw2);
    W2S = w2s;
    w2sq = w2sq_;
  }
  if (stages & (STRP_STAGE_ZUPD | STRP_STAGE_OBJ)) {
    nw1 = (stages & STRP_STAGE_REFIT1) ? weights_out_blocks(s, d) : gather_blocks(s, d);
    STRP_TAKE(ctx, arena, w1s, float, (size_t)s * d);
    STRP_TAKE(ctx, arena, w1sq_, double, (size_t)nw1);
    W1S = w1s;
    w1sq = w1sq_;
  }
  const WeightsOut w2out{STRP_SIDE_FC2, st->idx, st->W2, f, W2S, sp, W2S ? wmax + MAX_W2 : nullptr, w2sq};
  const WeightsOut w1out{STRP_SIDE_FC1, st->idx, st->W1, d, W1S, d, W1S ? wmax + MAX_W1 : nullptr, w1sq};
  // ---- S1/S5: Gram of the kept A rows, fc2 refit -------------------------------------------
  // Z_S is needed by tokens (fc1 refit) and, with relu, by channels (a-update): when both stages run, one pass over
  // the kept rows of Z writes both sets of planes; the second set stays in the base arena until the a-update.
  PlaneOp Zk8pre;
  memset(&Zk8pre, 0, sizeof(Zk8pre));
  const bool z_planes_once = (stages & STRP_STAGE_REFIT1) && (stages & STRP_STAGE_AUPD);
  int refits_done = 0, beside = 0;
  PlaneOp W2Sp, W2Tp, W1Sp;      // planes of the kept weights, shared by the stages below
  memset(&W2Sp, 0, sizeof(W2Sp));
  memset(&W2Tp, 0, sizeof(W2Tp));
  memset(&W1Sp, 0, sizeof(W1Sp));
  Aside aside(ctx);
  Arena side_part;
  if (z_planes_once && (stages & STRP_STAGE_REFIT2)) {
    const RefitsIn in{st->A, st->Z, lda, st->idx, s, d, T, npa, cv.Yt, cv.Xt, st->cholH, sc + SC_LAM2, clear};
    STRP_TRY(refit_both(ctx, arena, in, w2out, w1out, &Zk8pre, &refits_done));
    if (!refits_done) STRP_TRY(fill_zero(ctx, clear, 3));
    if (!refits_done && W1S) {
      STRP_TRY(refits_beside(ctx, aside, arena, in, w2out, w1out, bytes_after_refits(d, s, T, npa), &Zk8pre, &W1Sp, &side_part, &beside));
      refits_done = beside;
    }
  }
  else STRP_TRY(fill_zero(ctx, clear, 3));
  if (refits_done) {
    // the fc2 weights are there
  } else if (stages & STRP_STAGE_REFIT2) {
    Arena a2 = arena;
    const long long lds = system_ld(arena, d, s, T, npa);
    STRP_TAKE(ctx, a2, Gd, double, (size_t)s * lds);
    PlaneOp Arow;
    STRP_TRY(make_t_planes(ctx, a2, st->A, STRP_F32, lda, st->idx, s, T, 0, npa, &Arow));
    ReduceP r = reduce_to_system(Gd, lds);
    r.ridge_dev = sc + SC_LAM2;
    const Arena first = a2;                 // of a Gram product by itself: its partials are gone before the factor and R2 are written
    RefitIn ri;
    memset(&ri, 0, sizeof(ri));
    STRP_TAKE(ctx, a2, Ginv, double, (size_t)s * lds);
    ri.sys = Gd; ri.sys_ready = 1; ri.Linv = Ginv; ri.ldl = lds; ri.linv_ready = 0;
    ri.Lhs = operand_for(ctx, STRP_PROD_RHS2, 0, cv.Yt);
    ri.Rhs = operand_for(ctx, STRP_PROD_RHS2, 1, Arow);
    ri.m = d; ri.n = s; ri.ld = lds; ri.T = T;
    STRP_TAKE(ctx, a2, R2, double, (size_t)d * lds);
    const PlaneOp Gp = operand_for(ctx, STRP_PROD_GRAM, 0, Arow), Gq = operand_for(ctx, STRP_PROD_GRAM, 1, Arow);
    const size_t room = a2.room() / sizeof(float);
    GemmP prod[2] = {nt_plan(Gp, Gq, s, s, T, 1, room), nt_plan(ri.Lhs, ri.Rhs, d, s, T, 0, room)};
    ReduceP red[2] = {r, reduce_to(R2, lds)};
    if (group_fits(a2, prod, red, 2)) {
      STRP_TRY(launch_gemm_group(ctx, prod, 2));
      STRP_TRY(launch_splitk_reduce_group(ctx, red, 2));
      ri.r_ready = 1;
    }
    ri.R = R2;
    if (!ri.r_ready) STRP_TRY(nt_product(ctx, first, Gp, Gq, s, s, T, 1, r));
    STRP_TRY(ridge_solve(ctx, a2, ri, w2out));
  } else if (W2S) {
    STRP_TRY(gather_weights(ctx, w2out, d, s));
  }
  if (W2S) {
    SplitJob jobs[3];
    STRP_TRY(weight_planes(ctx, arena, W2S, SRC_F32, sp, d, s, 0, npa, wmax + MAX_W2, &W2Sp, &jobs[0]));
    const bool both = (stages & STRP_STAGE_AUPD) != 0;
    if (both) STRP_TRY(weight_planes(ctx, arena, W2S, SRC_F32, sp, s, d, 1, npa, wmax + MAX_W2, &W2Tp, &jobs[1]));
    int n = both ? 2 : 1;
    if (refits_done && !beside && W1S) STRP_TRY(weight_planes(ctx, arena, W1S, SRC_F32, d, s, d, 0, npa, wmax + MAX_W1, &W1Sp, &jobs[n++]));
    STRP_TRY(split_small(ctx, jobs, n));
  }
  // ---- a-update, part 1: B = W^T M^-1 with M = (beta/alpha) I + W W^T, W = W2[:, S] -------------------------
  // Needs only the refitted W2.  Its buffers come from the base arena and stay until the step ends.
  PlaneOp Bp;
  memset(&Bp, 0, sizeof(Bp));
  // First objective term when the a-update runs in the same call: the update solves its least-squares problem exactly, so
  //   Y - W A_S = E - W W^T M^-1 E = (M - W W^T) M^-1 E = (beta/alpha) M^-1 E,   E = Y - W relu(Z_S),
  // and |Y - W A_S|_F^2 = (beta/alpha)^2 <M^-2, E E^T>: a d x d Gram of E over the tokens (half the work of the product
  // W A_S) and two d x d matrices.  One fp16 plane of E is ample for a sum reported to 1e-3.
  const bool term1_identity = (stages & STRP_STAGE_AUPD) && (stages & STRP_STAGE_OBJ);
  bool residual_aside = false, residual_shared = false;
  float* M2f = nullptr;
  double* red_t1 = nullptr;
  unsigned short *ekh = nullptr, *ekl = nullptr, *eth = nullptr;      // planes of E by channels, one of them by tokens
  GemmP eet;                                                          // E E^T
  auto take_residual = [&](Arena& from) {
    ekh = (unsigned short*)from.take(2 * plane_elems(T, d));
    ekl = npa == 2 ? (unsigned short*)from.take(2 * plane_elems(T, d)) : nullptr;
    return ekh && (ekl || npa < 2);
  };
  auto residual = [&](const PlaneOp& Zk) {      // E = Y - W relu(Z_S), kept only as K8 planes
    GemmP p;
    memset(&p, 0, sizeof(p));
    p.P = operand_for(ctx, STRP_PROD_RESID, 0, W2Sp);
    p.Q = operand_for(ctx, STRP_PROD_RESID, 1, Zk);
    p.M = d; p.N = (int)T; p.K = s;
    p.epi = EPI_RESID; p.Yin = st->Y; p.ldy = lda;
    p.k8_hi = ekh; p.k8_lo = ekl; p.k8_kg = plane_kg(d);
    gemm_plan_tiles(p, 1);
    return p;
  };
  if (term1_identity) {
    STRP_TAKE(ctx, arena, rt1, double, (size_t)reduce_blocks(d, d));
    red_t1 = rt1;
  }
  auto term1 = [&](const GemmP& p) {            // <M^-2, E E^T>
    ReduceP r = reduce_to(nullptr, 0);
    r.dot = M2f; r.red = red_t1;
    reduce_of(p, &r);
    return r;
  };
  if (stages & STRP_STAGE_AUPD) {
    STRP_TAKE(ctx, arena, Md, double, (size_t)d * d);
    STRP_TAKE(ctx, arena, Linv, double, (size_t)d * d);
    STRP_TAKE(ctx, arena, Bf, float, (size_t)s * d);
    if (term1_identity) {
      STRP_TAKE(ctx, arena, m2, float, (size_t)d * d);
      M2f = m2;
    }
    const size_t cbytes = m_chain_bytes(d, sp);
    STRP_TAKE(ctx, arena, cblock, char, cbytes);
    Arena a2(cblock, cbytes);
    ReduceP r = reduce_to_system(Md, d);
    r.ridge = params->beta / params->alpha;
    Arena a3 = a2;
    GemmP first[2] = {nt_plan(W2Sp, W2Sp, d, d, sp, 1, a3.room() / sizeof(float))};
    STRP_TAKE(ctx, a3, part, float, (size_t)first[0].splits * d * d);
    first[0].out = part;
    // A small module's chain is launches of a few workgroups, so E, its turned plane, E E^T and the sum with M^-2 share them: E that of W W^T, the
    // plane that of M^-1's planes, E E^T that of B, the sum that of B's planes: four launches fewer, the same bits.  us a step of d x kept units over
    // the tokens, in launches of their own (at d <= 64) or on the second stream / shared:  64 x 128, 512 173.8 / 157.0;  64 x 128, 30000 260 / 240;
    // 48 x 90, 3000 177 / 159;  72 x 128, 512 182 / 173;  128 x 256, 2048 223 / 213;  200 x 400, 4000 310 / 300;  256 x 512, 2048 307 / 298;
    // 512 x 1000, 1024 517 / 514;  768 x 600, 768 473 / 469.
    if (term1_identity && refits_done && !beside) {
      Arena a4 = arena;
      eth = take_residual(a4) ? (unsigned short*)a4.take(2 * plane_elems(d, T)) : nullptr;
      const PlaneOp Et{eth, nullptr, plane_kg(T), (int)((d + 127) / 128), nullptr};
      eet = nt_plan(Et, Et, d, d, T, 1, ~size_t(0) >> 8);
      eet.out = eth ? (float*)a4.take(sizeof(float) * (size_t)eet.splits * d * d) : nullptr;
      first[1] = residual(Zk8pre);
      residual_shared = eet.out && a4.room() >= bytes_after_refits(d, s, T, npa) && gemm_is_small(first[0]) && gemm_is_small(first[1]) && gemm_is_small(eet);
      if (residual_shared) arena = a4;
    }
    // below some 500 kept units there is one partial, and the product of a small module writes the system by itself, with no reduction behind it
    // (us a step of d x kept units over the tokens  64 x 128, 512 151.4 / 148.8;  200 x 400, 4000 302.4 / 299.2;  768 x 300, 768 389.7 / 386.5)
    const bool direct = gemm_is_small(first[0]) && first[0].splits == 1;
    if (direct) {
      first[0].epi = EPI_SYSTEM; first[0].sys = Md; first[0].ldo = d; first[0].ridge = r.ridge;
    }
    STRP_TRY(residual_shared ? launch_gemm_group(ctx, first, 2) : launch_gemm(ctx, first[0]));
    reduce_of(first[0], &r);
    if (!direct) STRP_TRY(launch_splitk_reduce(ctx, r));
    // With both refits done E is next, which needs nothing of this chain.  Where it could not share the chain's launches it runs on the second
    // stream, from where M is factored on (us a step, 440 x 600 over 9000 tokens 546 -> 496; with one tile of M the two waits cost what there is
    // to hide: 64 x 128 over 512 172.7 / 173.7).
    residual_aside = refits_done && !residual_shared && (beside || d > NB) && aside.ready();
    if (residual_aside) STRP_TRY(aside.follow());
    {
      const double beside_us = residual_us(d, s, T, npa) + (beside ? fc1_us(d, s, T, npa, cv.Xt.lo ? 2 : 1) : 0.0);      // what the second stream has left
      const FlowWorkers few(ctx, residual_aside ? flow_workers_beside(d, beside_us) : 0);
      STRP_TRY(factor_and_invert(ctx, a2, Md, d, d, Linv, d));
    }
    // M is well conditioned (its spectrum lies in [beta/alpha, beta/alpha + |W|^2]): form M^-1 = Linv^T Linv
    // (lower half, fp64) and B = W^T M^-1 on the fp16-split matrix cores instead of a third fp64 solve
    STRP_TRY(gram_of_inverse(ctx, Linv, d, d, Md, d, wmax + MAX_MI));
    SplitJob job;
    PlaneOp Mi;
    STRP_TRY(weight_planes(ctx, a2, Md, SRC_F64, d, d, d, 2, npa, wmax + MAX_MI, &Mi, &job));
    STRP_TRY(residual_shared ? split_small_turn(ctx, job, ekh, eth, d, T) : split_small(ctx, &job, 1));
    GemmP p;
    memset(&p, 0, sizeof(p));
    p.P = W2Tp; p.Q = Mi;
    p.M = s; p.N = d; p.K = d;
    p.epi = EPI_STORE; p.out = Bf; p.ldo = d; p.maxbits = wmax + MAX_B;
    gemm_plan_tiles(p, 1);
    if (term1_identity) {   // M^-2 for the first objective term (see the a-update below)
      GemmP q;
      memset(&q, 0, sizeof(q));
      q.P = Mi; q.Q = Mi;
      q.M = d; q.N = d; q.K = d;
      q.epi = EPI_STORE; q.out = M2f; q.ldo = d;
      gemm_plan_tiles(q, 1);
      GemmP group[3] = {p, q, eet};
      STRP_TRY(launch_gemm_group(ctx, group, residual_shared ? 3 : 2));
    } else {
      STRP_TRY(launch_gemm(ctx, p));
    }
    STRP_TRY(weight_planes(ctx, arena, Bf, SRC_F32, d, s, d, 0, npa, wmax + MAX_B, &Bp, &job));
    STRP_TRY(residual_shared ? split_small_reduce(ctx, job, term1(eet)) : split_small(ctx, &job, 1));
  }
  if (z_planes_once && !refits_done) {
    STRP_TAKE(ctx, arena, zch, unsigned short, plane_elems(T, s));
    unsigned short* zcl = nullptr;
    if (npa == 2) {
      STRP_TAKE(ctx, arena, zcl2, unsigned short, plane_elems(T, s));
      zcl = zcl2;
    }
    Zk8pre = PlaneOp{zch, zcl, plane_kg(s), (int)((T + 127) / 128), nullptr};
  }
  // ---- S6: fc1 refit with the cached factor of H + lam1 I ------------------------------------
  if (refits_done) {
    // the fc1 weights are there
  } else if (stages & STRP_STAGE_REFIT1) {
    Arena a2 = arena;
    PlaneOp Zrow;
    if (z_planes_once) {
      STRP_TAKE(ctx, a2, zth, unsigned short, plane_elems(s, T));
      unsigned short* ztl = nullptr;
      if (npa == 2) {
        STRP_TAKE(ctx, a2, ztl2, unsigned short, plane_elems(s, T));
        ztl = ztl2;
      }
      STRP_TRY(split_act(ctx, st->Z, STRP_F32, lda, st->idx, s, T, 0, 1, zth, ztl, (unsigned short*)Zk8pre.hi, (unsigned short*)Zk8pre.lo));
      Zrow = PlaneOp{zth, ztl, plane_kg(T), (s + 127) / 128, nullptr};
    } else {
      STRP_TRY(make_t_planes(ctx, a2, st->Z, STRP_F32, lda, st->idx, s, T, 0, npa, &Zrow));
    }
    RefitIn ri;
    memset(&ri, 0, sizeof(ri));
    ri.Linv = st->cholH; ri.ldl = d; ri.linv_ready = 1;
    ri.Lhs = operand_for(ctx, STRP_PROD_RHS1, 0, Zrow);
    ri.Rhs = operand_for(ctx, STRP_PROD_RHS1, 1, cv.Xt);
    ri.m = s; ri.n = d; ri.ld = f64_ld(d); ri.T = T;
    STRP_TRY(ridge_solve(ctx, a2, ri, w1out));
  } else if (W1S) {
    STRP_TRY(gather_weights(ctx, w1out, s, d));
  }
  if (W1S && !refits_done) {
    SplitJob job;
    STRP_TRY(weight_planes(ctx, arena, W1S, SRC_F32, d, s, d, 0, npa, wmax + MAX_W1, &W1Sp, &job));
    STRP_TRY(split_small(ctx, &job, 1));
  }

  // scoring sums of the kept rows, collected by the two epilogues that write those rows (64-column strips, fp32)
  const int rs_slots = (int)((T + 63) / 64);
  float* rsA = nullptr;
  float* rsZ = nullptr;
  if (fuse_pruned) {
    STRP_TAKE(ctx, arena, rsa_, float, (size_t)(wanda ? 1 : 2) * rs_slots * s);
    rsA = rsa_;
    if (!wanda) {
      STRP_TAKE(ctx, arena, rsz_, float, (size_t)rs_slots * s);
      rsZ = rsz_;
    }
  }
  FinishP fin;
  memset(&fin, 0, sizeof(fin));
  fin.sc = sc;
  // ---- S7: a-update in residual (Woodbury) form ------------------------------------------------
  //   A_S = relu(Z_S) + W^T M^-1 (Y - W relu(Z_S)),  M = (beta/alpha) I + W W^T,  W = W2[:, S];  A_j = relu(Z_j) for pruned j
  if (stages & STRP_STAGE_AUPD) {
    Arena a2 = arena;
    PlaneOp Zk8 = Zk8pre;
    if (!z_planes_once) {
      STRP_TRY(make_c_planes(ctx, a2, st->Z, STRP_F32, lda, st->idx, s, T, 1, npa, &Zk8));
    }
    if (!residual_shared) {
      if (!take_residual(a2)) return fail(ctx, STRP_ENOMEM, "workspace too small for the residual");
      if (residual_aside) aside.enter();
      GemmP p = residual(Zk8);
      STRP_TRY(launch_gemm(ctx, p));
    }
    if (term1_identity) {   // (alpha/T) |Y - W A_S|^2 = (alpha/T) (beta/alpha)^2 <M^-2, E E^T>
      if (!residual_shared) {
        Arena a3 = a2;
        STRP_TAKE(ctx, a3, et, unsigned short, plane_elems(d, T));
        STRP_TRY(plane_c_to_t(ctx, ekh, et, d, T));
        const PlaneOp Et{et, nullptr, plane_kg(T), (int)((d + 127) / 128), nullptr};
        if (beside) a3 = side_part;
        eet = nt_plan(Et, Et, d, d, T, 1, a3.room() / sizeof(float));
        STRP_TAKE(ctx, a3, part, float, (size_t)eet.splits * d * d);
        eet.out = part;
        STRP_TRY(launch_gemm(ctx, eet));
        STRP_TRY(aside.join());        // the sum below is with M^-2
        STRP_TRY(launch_splitk_reduce(ctx, term1(eet)));
      }
      const double c = params->beta / params->alpha;
      fin.do_1 = 1; fin.red_1 = red_t1; fin.n1 = reduce_blocks(d, d); fin.stride1 = 1; fin.c1 = params->alpha / (double)T * c * c;
    }
    STRP_TRY(aside.join());
    {  // A_S = relu(Z_S) + B E
      GemmP p;
      memset(&p, 0, sizeof(p));
      p.P = operand_for(ctx, STRP_PROD_AUPD, 0, Bp);
      p.Q = operand_for(ctx, STRP_PROD_AUPD, 1, PlaneOp{ekh, ekl, plane_kg(d), (int)((T + 127) / 128), nullptr});
      p.M = s; p.N = (int)T; p.K = d;
      p.epi = EPI_AUPD; p.Zs = st->Z; p.As = st->A; p.lda = lda; p.oidx = st->idx;
      p.rs_out = rsA; p.rs_z0 = (rsA && !wanda) ? st->Z0 : nullptr; p.rs_slots = rs_slots;
      gemm_plan_tiles(p, 1);
      STRP_TRY(launch_gemm(ctx, p));
    }
    if (!fuse_pruned) {
      ProfScope ps(ctx, "pruned_rows_a", 0.0, 8.0 * (double)(f - s) * (double)T);
      hipLaunchKernelGGL(pruned_rows_kernel, dim3(f), dim3(256), 0, ctx->stream, st->mask, st->Z, st->A, lda, T, 0, alpha, beta, 1, (double*)nullptr);
    }
  }
  // ---- S8 (+ objective terms 2, 3): z-update fused on Z1 = W1 X --------------------------------
  const bool zupd = (stages & STRP_STAGE_ZUPD) != 0;
  if (zupd || (stages & STRP_STAGE_OBJ)) {
    GemmP p;
    memset(&p, 0, sizeof(p));
    p.P = operand_for(ctx, STRP_PROD_ZUPD, 0, W1Sp);
    p.Q = operand_for(ctx, STRP_PROD_ZUPD, 1, cv.Xc);
    p.M = s; p.N = (int)T; p.K = d;
    p.epi = EPI_ZUPD; p.Zs = st->Z; p.As = st->A; p.lda = lda; p.oidx = st->idx; p.alpha = alpha; p.beta = beta;
    p.write_out = zupd ? 1 : 0;
    p.rs_out = (zupd && rsZ) ? rsZ : nullptr; p.rs_z0 = p.rs_out ? st->Z0 : nullptr; p.rs_slots = rs_slots;
    gemm_plan_tiles(p, 1);
    const int nb = gemm_grid_blocks(p);
    STRP_TAKE(ctx, arena, red, double, 2 * (size_t)nb);
    p.red = red;
    STRP_TRY(launch_gemm(ctx, p));
    fin.do_z = 1; fin.red_z = red; fin.nz = nb; fin.c2 = params->beta / (double)T; fin.c3 = params->alpha / (double)T;
    if (fuse_pruned) {
      if (pjob.units) {      // the rows' sums are added at the end
        fin.rows = prow; fin.partial = pjob.partial; fin.nrows = pjob.nrows; fin.segs = pjob.segs; fin.z0 = pjob.Z0 != nullptr;
        fin.blk = finish_blk;
      }
      // every row's sums are then in place: the kept rows' from the two epilogues, the pruned rows' from this pass
      // (which also rewrites their sum Z0^2; the kept rows' is only there if it was streamed before)
      st->sums_cached = (st->sums_cached & SUMS_V) | SUMS_G | (wanda ? 0 : SUMS_EU);
    } else {
      STRP_TAKE(ctx, arena, redp, double, 2 * (size_t)f);
      ProfScope ps(ctx, "pruned_rows_z", 0.0, 8.0 * (double)(f - s) * (double)T);
      hipLaunchKernelGGL(pruned_rows_kernel, dim3(f), dim3(256), 0, ctx->stream, st->mask, st->Z, st->A, lda, T, 1, alpha, beta,
                         zupd ? 1 : 0, redp);
      fin.red_p = redp; fin.np = f;
    }
  }
  // ---- S9: objective term 1 (one fp16 plane per operand is ample for a 1e-3 sum) and ridge terms ----
  if (stages & STRP_STAGE_OBJ) {
    if (!term1_identity) {   // A is whatever the caller left: the product itself
      Arena a3 = arena;
      PlaneOp Ak8;
      GemmP p;
      memset(&p, 0, sizeof(p));
      p.P = W2Sp; p.P.lo = nullptr;
      p.M = d; p.N = (int)T; p.K = s;
      p.epi = EPI_RESID; p.Yin = st->Y; p.ldy = lda;
      gemm_plan_tiles(p, 1);
      const int nb = gemm_grid_blocks(p);
      STRP_TAKE(ctx, a3, redg, double, 2 * (size_t)nb);
      STRP_TRY(make_c_planes(ctx, a3, st->A, STRP_F32, lda, st->idx, s, T, 0, 1, &Ak8));
      p.Q = Ak8;
      p.red = redg;
      STRP_TRY(launch_gemm(ctx, p));
      fin.do_1 = 1; fin.red_1 = redg; fin.n1 = nb; fin.stride1 = 2; fin.c1 = params->alpha / (double)T;
    }
    fin.do_w = 1; fin.w2 = w2sq; fin.nw2 = nw2; fin.w1 = w1sq; fin.nw1 = nw1;
  }
  if (report_host) {
    fin.host = (double*)ctx->pinned;
  }
  if (fin.nrows || fin.do_z || fin.do_1 || fin.do_w || fin.host) {
    if (rsA) {
      fin.strips[0] = rsA;
      fin.strips[1] = rsA + (size_t)rs_slots * s;
      fin.strips[2] = rsZ;
      fin.n_strips = wanda ? 1 : 3;
    }
    fin.slots = rs_slots; fin.M = s; fin.idx = st->idx; fin.rowsums = cv.rowsums; fin.f = f;
    fin.row_blocks = finish_row_blocks(fin.nrows);
    fin.ticket = ticket;
    fin.sums = (double*)(wmax + 40);
    fin.status = ctx->status_dev;
    ProfScope ps(ctx, fin.nrows ? "pruned_rows_drain" : "step_finish", 0.0, 0.0);
    const int strips = fin.n_strips ? prof_begin(ctx, "rowsum_reduce", 0.0, 4.0 * (double)fin.n_strips * (double)rs_slots * (double)s) : -1;
    hipLaunchKernelGGL(step_finish_kernel, dim3(fin.row_blocks + 1 + fin.n_strips * ((s + 63) / 64)), dim3(FINISH_THREADS), 0, ctx->stream, fin);
    prof_end(ctx, strips);
  }
  STRP_HIP(ctx, hipGetLastError());
  st->iter += 1;

  if (report_host) {
    double* h = (double*)ctx->pinned;
    STRP_HIP(ctx, hipStreamSynchronize(ctx->stream));
    memset(report_host, 0, sizeof(*report_host));
    report_host->lam1 = h[SC_LAM1];
    report_host->lam2 = h[SC_LAM2];
    report_host->terms[0] = h[SC_T1];
    report_host->terms[1] = h[SC_T2];
    report_host->terms[2] = h[SC_T3];
    report_host->terms[3] = params->alpha * h[SC_LAM2] * h[SC_W2SQ] / (double)T;
    report_host->terms[4] = params->alpha * h[SC_LAM1] * h[SC_W1SQ] / (double)T;
    report_host->J = report_host->terms[0] + report_host->terms[1] + report_host->terms[2];
    report_host->J_ridge = report_host->J + report_host->terms[3] + report_host->terms[4];
    report_host->tau = *(float*)(h + SC_TAU);
    report_host->s = s;
    report_host->status = *(int32_t*)(h + SC_COUNT);
    if (report_host->status != 0) {
      fail(ctx, (strp_status)report_host->status, "device status word = %d", report_host->status);
      STRP_TRY(fill_zero(ctx, ctx->status_dev, 256));
    }
  }
  return STRP_OK;
}

}  // extern "C"
