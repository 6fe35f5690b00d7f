// Internal declarations shared by the HIP translation units of libstrp.so (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "strp.h"

namespace strp {
struct CoJob;
}

struct strp_ctx {
  int device;
  hipStream_t stream;
  char* ws;            // caller-owned device workspace
  size_t ws_bytes;
  int precision;       // strp_precision
  int32_t* status_dev; // first word of the workspace
  void* pinned;        // small pinned host buffer for report read-back
  char err[512];
  struct Profiler* prof;  // optional per-kernel event timing (host object)
  unsigned char prod_planes[8][2];  // fp16 planes (1 or 2) of the P and Q operand per strp_product of strp_admm_step
  // Set by strp_admm_step while a streaming job waits for a launch to ride along with (see cojob.h); null everywhere else.
  // The next chol_inverse takes it.
  const strp::CoJob* cojob;
  // A device counter that only this context's weight statistics on its present workspace use: zero between calls, reset by the
  // workgroup that reads its last count.  Null when the process has taken all there are.
  unsigned int* ticket;
  unsigned int* tickets;  // all of them, on this device
  int ticket_due;         // another workspace has been set: the next weight statistics take the next counter
  // A second stream for work that a call's latency-bound part leaves the chip to (see Aside in strp_api.hip), and the events that order the two.
  // Made by the first call that can use them, on the context's device; side_state: 0 not yet, 1 there, -1 not to be had.
  hipStream_t side;
  hipEvent_t side_event[2];
  int side_state;
  int flow_workers;       // workgroups of the next factorisation in one launch, which has other kernels beside it; 0: as many as it has use for
};

struct Profiler;

namespace strp {

// ---- optional per-kernel timing with HIP events on the context's stream -----------------------
// prof_begin returns a record index (or -1 when profiling is off); prof_end closes it.
int prof_begin(strp_ctx* ctx, const char* name, double flops, double bytes);
void prof_end(strp_ctx* ctx, int rec);
struct ProfScope {
  strp_ctx* ctx;
  int rec;
  ProfScope(strp_ctx* c, const char* name, double flops, double bytes) : ctx(c), rec(prof_begin(c, name, flops, bytes)) {}
  ~ProfScope() { prof_end(ctx, rec); }
};

// ---- error helpers -------------------------------------------------------------------
strp_status fail(strp_ctx* ctx, strp_status st, const char* fmt, ...);
#define STRP_HIP(ctx, call)                                                              \
  do {                                                                                   \
    hipError_t e_ = (call);                                                              \
    if (e_ != hipSuccess)                                                                \
      return strp::fail((ctx), STRP_EHIP, "%s failed: %s", #call, hipGetErrorString(e_)); \
  } while (0)
#define STRP_TRY(expr)                  \
  do {                                  \
    strp_status s_ = (expr);            \
    if (s_ != STRP_OK) return s_;       \
  } while (0)

// ---- workspace bump arena (256-byte granules); the first granule holds the status word, the only thing in the workspace
// that lasts from one call to the next ----
struct Arena {
  char* base;
  size_t off, cap;
  Arena() : base(nullptr), off(0), cap(0) {}
  explicit Arena(strp_ctx* ctx) : base(ctx->ws), off(256), cap(ctx->ws_bytes) {}
  Arena(void* block, size_t bytes) : base((char*)block), off(0), cap(bytes) {}   // sub-arena over a block taken elsewhere
  size_t room() const { return base && off < cap ? (cap - off) & ~size_t(255) : 0; }
  void* take(size_t bytes) {
    size_t b = (bytes + 255) & ~size_t(255);
    if (!base || off + b > cap) return nullptr;
    void* p = base + off;
    off += b;
    return p;
  }
};
#define STRP_TAKE(ctx, arena, var, type, count)                                                     \
  type* var = (type*)(arena).take(sizeof(type) * (size_t)(count));                                  \
  if (!var) return strp::fail((ctx), STRP_ENOMEM, "workspace too small for %s (%zu bytes more)",    \
                              #var, sizeof(type) * (size_t)(count))

// ---- MFMA GEMM family on 16-bit operand planes (gemm_mfma.hip, split_planes.hip) -----------------
// An operand as the matrix cores see it: one (hi) or two (hi, lo) fp16 planes in the panel-major chunk layout
//   offset(k, r) = (((r / 128) * kg + k / 8) * 128 + r % 128) * 8 + k % 8
// k = contraction index, r = output row (P) or output column (Q); npan panels of 128 rows, kg k-groups of 8
// (kg = plane_kg(K): a multiple of four, padding zero).
// maxbits (device, optional): the bits of max|x|; the planes hold x * scale_of_max(*maxbits), the GEMM epilogue divides it out.
struct PlaneOp {
  const unsigned short* hi;
  const unsigned short* lo;
  long long kg;
  int npan;
  const unsigned int* maxbits;
};
// Power of two that brings a maximum (given by its bits) into [2^11, 2^12): keeps fp16 hi far from overflow and lo out of
// the subnormals.  1 for zero, infinity and NaN.
__device__ __forceinline__ float scale_of_max(unsigned int bits) {
  if (bits == 0u || bits > 0x7f61b1e6u) return 1.0f;       // above 3e38
  const unsigned int e = 265u - (bits >> 23);              // max = q 2^(E - 126), q in [1/2, 1): 2^(12 - (E - 126))
  return __builtin_bit_cast(float, (e > 254u ? 254u : e) << 23);
}
// k-groups allocated for a contraction of length K: a multiple of four, the pad groups zero-filled (the pipelined
// kernel moves two k-groups per stage and multiplies four per matrix-core instruction, both without tail logic)
__host__ __device__ static inline long long plane_kg(long long K) { return (((K + 7) / 8) + 3) & ~3LL; }
static inline size_t plane_elems(long long rows, long long K) {
  return (size_t)((rows + 127) / 128) * (size_t)plane_kg(K) * 1024;
}

enum { EPI_PARTIAL = 0, EPI_STORE = 1, EPI_INITZ = 2, EPI_RESID = 3, EPI_AUPD = 4, EPI_ZUPD = 5, EPI_SYSTEM = 6 };
enum { SRC_F64 = 0, SRC_F32 = 1, SRC_BF16 = 2 };

struct GemmP {
  PlaneOp P, Q;        // C[m, n] = sum_k P(k, m) Q(k, n)
  int M, N;
  long long K;
  int wt;              // 32x32 MFMA tiles per wavefront per dimension: 2 (128x128 blocks) or 4 (256x256), set by gemm_plan_tiles; 3: 128x256, 5: 64x256; 1: the
                       // plan of 2 with each tile cut into subM x subN blocks of 64x64 (gemm_small_tiles)
  int subM, subN;
  int tilesM, tilesN, ntiles;
  int gridM, gridN;    // tile grid the blocks are laid over: tilesM x tilesN, or the folded triangle (see decode_tile)
  int gm, gn;          // tile group (gm x gn = tiles that are resident on one XCD together)
  int triangle;        // P == Q, only tiles with tn <= tm are computed
  int splits;
  long long kchunk;    // K range per split (multiple of the K tile)
  int epi;
  float* out;          // PARTIAL: [splits][M][N]; STORE: [M x ldo]
  long long ldo;
  const float* Yin;    // RESID: Y
  long long ldy;
  float* Zs;           // INITZ / AUPD / ZUPD state pointers, leading dimension lda
  float* As;
  float* Z0s;
  long long lda;
  const int* oidx;     // AUPD / ZUPD: output row m is state row oidx[m]
  float alpha, beta;
  double* red;         // per-block partial sums [gridDim.x][2] (INITZ, RESID, ZUPD)
  int write_out;       // ZUPD: 1 = update Z, 0 = only accumulate the objective sums
  unsigned int* maxbits;  // STORE, optional: atomic maximum of the bits of |C|
  unsigned short* k8_hi;  // optional operand planes of the produced values with k = output row, r = output column
  unsigned short* k8_lo;  //   (STORE: C, INITZ: relu(C), RESID: Y - C; not offered by AUPD / ZUPD); k8_kg = plane_kg(M) groups, ceil(N/128) panels
  long long k8_kg;
  // AUPD / ZUPD, optional: scoring sums of the rows being written, one fp32 partial per output row and 64-column strip,
  //   rs_out[(q * rs_slots + strip) * M + m];  AUPD: q = 0 sum a^2, q = 1 sum a relu(z0) (iff rs_z0); ZUPD: q = 0 sum z0 z
  //   (iff rs_z0).  rs_z0 = the Z0 state tensor (leading dimension lda, rows gathered like Zs).  rs_slots = ceil(N / 64).
  float* rs_out;
  const float* rs_z0;
  int rs_slots;
  // SYSTEM (64x64 blocks only): what the reduction of a single partial by reduce_to_system would write, leading dimension ldo
  double* sys;
  double ridge;
};

strp_status launch_gemm(strp_ctx* ctx, GemmP& p);
// n <= 3 products, none of which reads what another writes; launch_splitk_reduce_group: n <= 3 reductions
strp_status launch_gemm_group(strp_ctx* ctx, GemmP* p, int n);
bool gemm_is_small(const GemmP& p);
int gemm_grid_blocks(const GemmP& p);
// tile shape (wt = 0: by the number of tiles), tile grid and K splits of a product
void gemm_plan_tiles(GemmP& p, int want_splits, int wt = 0);
// smaller blocks for a plan that leaves the chip idle (part of gemm_plan_tiles with wt = 0)
void gemm_small_tiles(GemmP& p);
static inline bool gemm_tile256_ok(const GemmP& p) { return p.M >= 256 && p.N >= 256 && p.K >= 256; }

// Sum split-K partials in fp64; optional symmetric completion from the computed lower half.
// outf / outd (either may be null): [M x ldo]; accumulate adds to outf's previous content; ridge (or *ridge_dev) is added
// to outd's diagonal.  dot (symmetric products only, instead of any output): [M x N] fp32, red[workgroup] = its share of
// <dot, C>; reduce_blocks(M, N) workgroups.
struct ReduceP {
  const float* part;
  int splits, M, N, triangle;
  float* outf; long long ldof;
  double* outd; long long ldod;
  int factored;          // outd is for chol_inverse: zeros in columns 64 .. of rows 0 .. 63 (reduce_to_system)
  double* diag;
  int accumulate;
  double ridge; const double* ridge_dev;
  const float* dot; double* red;
};
strp_status launch_splitk_reduce(strp_ctx* ctx, const ReduceP& r);
strp_status launch_splitk_reduce_group(strp_ctx* ctx, const ReduceP* r, int n);
constexpr int REDUCE_TILE_M = 16, REDUCE_TILE_N = 64;      // output tile of one workgroup of the split-K reduction
static inline int reduce_blocks(int M, int N) { return ((M + REDUCE_TILE_M - 1) / REDUCE_TILE_M) * ((N + REDUCE_TILE_N - 1) / REDUCE_TILE_N); }
// fp32 / bf16 activation rows (optionally gathered by idx) -> fp16 planes; any output pair may be null.
//   t_* : contraction over tokens   (k = token,   r = row):   plane_elems(rows, T)
//   c_* : contraction over channels (k = row,     r = token): plane_elems(T, rows)
strp_status split_act(strp_ctx* ctx, const void* src, int src_dtype, long long lds, const int* idx, int rows, long long T,
                      int relu_t, int relu_c, unsigned short* t_hi, unsigned short* t_lo, unsigned short* c_hi,
                      unsigned short* c_lo);
// Rows idx of two fp32 matrices in one launch: a -> t_* (At), z -> t_* (Zt) and, with relu, c_* (Zc); all of one plane or all of two.
// clear: three ranges that the same launch clears.
struct FillRange;
strp_status split_act_pair(strp_ctx* ctx, const float* a, const float* z, long long lds, const int* idx, int rows, long long T, const PlaneOp& At,
                           const PlaneOp& Zt, const PlaneOp& Zc, const FillRange* clear);
// One fp16 plane of a [C x T] quantity with k = channel, r = token (plane_elems(T, C)) -> the plane with k = token,
// r = channel (plane_elems(C, T)); padding tokens zero.
strp_status plane_c_to_t(strp_ctx* ctx, const unsigned short* src, unsigned short* dst, int C, long long T);
// Small matrices (weights) -> planes with k = column, r = row: plane_elems(rows, cols); kind = SRC_*.
// transpose: 1 = the source is stored transposed, 2 = symmetric, only its lower triangle is valid.
struct SplitJob {
  const void* src;
  long long lds;
  int kind, rows, cols, transpose;
  const unsigned int* maxbits;
  unsigned short* hi;
  unsigned short* lo;
};
strp_status split_small(strp_ctx* ctx, const SplitJob* jobs, int n);      // n <= 3, one launch
// The planes of one matrix, and in the same launch plane_c_to_t of something else / the reduction of a symmetric product with an inner product.
strp_status split_small_turn(strp_ctx* ctx, const SplitJob& job, const unsigned short* src, unsigned short* dst, int C, long long T);
strp_status split_small_reduce(strp_ctx* ctx, const SplitJob& job, const ReduceP& r);
// *maxbits[i] = max(*maxbits[i], bits of max|src_i|) for fp32 / bf16 matrices; n <= 2, one launch
struct MaxJob {
  const void* src;
  long long lds;
  int kind, rows, cols;
  unsigned int* maxbits;
};
strp_status abs_max(strp_ctx* ctx, const MaxJob* jobs, int n);

// ---- fp64 dense kernels (dense_f64.hip) ---------------------------------------------------
constexpr int NB = 64;  // block order of the factorisation
// leading dimension of the fp64 work matrices: rows 16-byte aligned whatever the order
static inline long long f64_ld(long long n) { return (n + 7) & ~7LL; }
// doubles of scratch of a factorisation: the tiles of two launches that the next panel reads, two each
static inline size_t chol_scratch_elems(long long n) {
  const long long tiles = (n + NB - 1) / NB;
  return (size_t)(tiles < 4 ? tiles : 4) * NB * NB;
}
// Linv [n x n, ldv] = L^-1 (upper part zero) of the SPD matrix A [n x n, ld] = L L^T whose lower triangle is given (the
// caller has added the ridge) and destroyed.  Columns 64 .. of rows 0 .. 63 of A hold zeros, which become counters: with anything else
// there tiles are taken for finished and the factor is wrong, so A comes from a reduction with `factored` or from
// f32_to_f64_ridge.  sub: chol_scratch_elems(n) doubles of scratch.  ld and ldv even, A and Linv 16-byte aligned.  A pivot that
// is not positive sets ENOTPD in status (device word); a wait that takes ten seconds, EHIP.
strp_status chol_inverse(strp_ctx* ctx, double* A, int n, long long ld, double* sub, double* Linv, long long ldv, int32_t* status);
// The same in one launch, for the orders that are faster so beside a pass of these bytes (0: none).
bool chol_flow_ok(int n, double pass_bytes);
// whether the order alone decides that
bool chol_by_order(int n);
strp_status chol_flow(strp_ctx* ctx, double* A, int n, long long ld, double* Linv, long long ldv, int32_t* status, const CoJob& job);
// a pass that rides with nothing: a launch of its own
strp_status launch_cojob(strp_ctx* ctx, const CoJob& job);
// X (L L^T)^-1 = (X Linv^T) Linv for X [m x n] (ldx), as refitted weights; tmp: m x ldx scratch.
//   FC2: W[i, idx[j]] = result[i, j] (m rows of W);  FC1: W[idx[i], j] = result[i, j];  other entries of W are not written.
//   Wc (optional): the result itself, [m x ldc]; maxbits (optional): atomic maximum of the bits of its magnitudes; sumsq
//   (optional): [weights_out_blocks(m, n)] sums of squares.
struct WeightsOut {
  int side;
  const int32_t* idx;
  float* W; long long ldw;
  float* Wc; long long ldc;
  unsigned int* maxbits;
  double* sumsq;
};
strp_status apply_inverse_right(strp_ctx* ctx, const double* Linv, int n, long long ldl, const double* X, int m, long long ldx, double* tmp,
                                const WeightsOut& out);
// Two solves of which neither reads what the other writes, in two launches; both of solve_is_small: less than a wave of tiles each
bool solve_is_small(int m, int n);
struct SolveIn {
  const double* Linv; int n; long long ldl;
  const double* X; int m; long long ldx;
  double* tmp;
  WeightsOut out;
};
strp_status apply_inverse_right_pair(strp_ctx* ctx, const SolveIn& a, const SolveIn& b);
int weights_out_blocks(int m, int n);
// The compact weights Wc [m x ldc] of an earlier refit out of W, with the same by-products (gather_blocks(m, n) sums).
strp_status gather_weights(strp_ctx* ctx, const WeightsOut& io, int m, int n);
int gather_blocks(int m, int n);
// Tiles on or below the diagonal of S [n x n, lds] = Linv^T Linv; maxbits: atomic maximum of the bits of its magnitudes.
strp_status gram_of_inverse(strp_ctx* ctx, const double* Linv, int n, long long ldl, double* S, long long lds, unsigned int* maxbits);
// dst [n x n, ldd] = src [n x n, lds]
strp_status copy_f64(strp_ctx* ctx, const double* src, long long lds, double* dst, long long ldd, int n);
// Ad[i*ld+j] = (double)Af[i*ldf+j] + (i==j ? lam (or *lam_dev if non-null) : 0), for chol_inverse: zeros in columns 64 .. of rows 0 .. 63
strp_status f32_to_f64_ridge(strp_ctx* ctx, const float* Af, long long ldf, double* Ad, long long ld, int n,
                             double lam, const double* lam_dev);

// ---- reductions, scores, allocation, select (score_select.hip) ------------------------------
strp_status launch_row_sums(strp_ctx* ctx, const void* A, int a_dtype, const float* Z, const float* Z0,
                            long long ld, long long T, int rows, int mode, double* sums /*[4][rows]*/);
strp_status launch_colnorm2(strp_ctx* ctx, const void* W, int w_dtype, int rows, int cols, long long ldw,
                            double* n2);
strp_status launch_unit_scores(strp_ctx* ctx, const double* sums, const double* n2, int n_channels, int group,
                               int mode, float* score, double* energy_out);
strp_status launch_alloc(strp_ctx* ctx, const double* energies, int L, const int32_t* n_units,
                         const int32_t* group_id, double rbar, double temperature, double rmax, int rule, double* r_out,
                         int32_t* nprune_out);
strp_status launch_weight_energy(strp_ctx* ctx, const strp_weight_ref* mats, int n_mats, double var_coef, double l2_coef,
                                 double scale, double* energy, double* partial);
size_t weight_energy_scratch_bytes();
strp_status launch_topk(strp_ctx* ctx, const float* score, int n, int k, int group, uint8_t* mask, int32_t* idx,
                        float* tau, void* scratch, size_t scratch_bytes);
size_t topk_scratch_bytes(int n);
// One module's selection in one launch: unit scores from the token sums (layout of launch_row_sums), their mean, and the k
// best of them; rest (optional): the n - k other indices, ascending.  n <= SELECT_MAX unless k = n.
constexpr int SELECT_MAX = 65536;     // scores one block selects from (64 per thread)
strp_status launch_select(strp_ctx* ctx, const double* sums, const double* n2, int mode, int n, int k, float* score, double* energy_out,
                          uint8_t* mask, int32_t* idx, float* tau, int32_t* rest);

// ---- small helpers -----------------------------------------------------------------------------
strp_status fill_zero(strp_ctx* ctx, void* ptr, size_t bytes);
struct FillRange {
  void* ptr;
  size_t bytes;      // multiple of 4
};
strp_status fill_zero(strp_ctx* ctx, const FillRange* ranges, int n);     // n <= 3, one launch
// several ranges in one launch: a launch costs more than clearing most of what is cleared here
struct FillRanges {
  uint32_t* p[3];
  long long words[3];
};
// bytes of 4 or more -> *f, in words; the longest of them in *most
strp_status fill_ranges(strp_ctx* ctx, const FillRange* ranges, int n, FillRanges* f, long long* most);
// by workgroup `block` of `blocks` of 256 threads
__device__ __forceinline__ void fill_block(const FillRanges& f, unsigned int block, unsigned int blocks) {
  const long long stride = (long long)blocks * 256, e0 = (long long)block * 256 + threadIdx.x;
  for (int r = 0; r < 3; ++r) {
    uint32_t* p = f.p[r];
    const long long quads = ((uintptr_t)p & 15) == 0 ? f.words[r] >> 2 : 0;
    for (long long e = e0; e < quads; e += stride) ((uint4*)p)[e] = make_uint4(0u, 0u, 0u, 0u);
    for (long long e = 4 * quads + e0; e < f.words[r]; e += stride) p[e] = 0u;
  }
}

// "The last workgroup does the rest": true in every thread of the last workgroup of the grid to get here.  What the
// workgroups hand to it goes through agent-scope atomics (agent_put / agent_get / atomicAdd), which act at the level all
// XCDs share, so it is enough that they have completed before the counter moves: an agent-scope fence would
// write back and invalidate the XCD's L2 from every workgroup, which took 45 of a launch's 50 us.
template <typename T>
__device__ __forceinline__ void agent_put(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T agent_get(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ bool last_block(unsigned int* done, unsigned int* flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) *flag = atomicAdd(done, 1u) + 1u == gridDim.x;
  __syncthreads();
  return *flag != 0;
}

}  // namespace strp
