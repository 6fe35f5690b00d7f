// HBM-bound scoring reductions, the softmax sparsity allocation and the top-k structured select.
//   row_sums      : per-channel token sums (fp64 accumulation, one block per channel, float4 loads)
//   colnorm2      : squared column norms of the next linear layer
//   unit_scores   : WANDA / LEMMA / GAIN unit scores (+ group sums for heads) and the layer energy
//   alloc         : softmax allocation with clipping, rescale and largest-remainder prune counts
//   topk          : histogram select on order-preserving keys, ballot/prefix compaction, ties -> lower index
#include <stddef.h>

#include <type_traits>

#include "strp_internal.h"

namespace strp {

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_allsum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wave_allmax_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float bf16lo(unsigned int w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16hi(unsigned int w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// ---------------------------------------------------------------------------------------------
// per-channel token sums: sums[0][r] = sum A^2, [1][r] = sum A*relu(Z0), [2][r] = sum Z0*Z, [3][r] = sum Z0^2
// ---------------------------------------------------------------------------------------------
template <bool A_BF16, bool FULL>
__global__ __launch_bounds__(256) void row_sums_kernel(const void* Av, const float* Z, const float* Z0, long long ld,
                                                       long long T, int rows, double* sums, int32_t* status) {
  const int r = blockIdx.x;
  const int tid = threadIdx.x;
  double g = 0.0, e = 0.0, u = 0.0, v = 0.0;
  const long long T8 = T & ~7LL;
  if (A_BF16 && !FULL) {
    const uint4* a8 = (const uint4*)((const unsigned short*)Av + (long long)r * ld);
    for (long long c = tid; c < T8 / 8; c += 256) {
      const uint4 w = a8[c];
      const unsigned int ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double lo = (double)bf16lo(ww[q]), hi = (double)bf16hi(ww[q]);
        g = __builtin_fma(lo, lo, g);
        g = __builtin_fma(hi, hi, g);
      }
    }
    const unsigned short* as = (const unsigned short*)Av + (long long)r * ld;
    for (long long t = T8 + tid; t < T; t += 256) {
      const double x = (double)__builtin_bit_cast(float, (unsigned int)as[t] << 16);
      g = __builtin_fma(x, x, g);
    }
  } else {
    const float* a = (const float*)Av + (long long)r * ld;
    const float* z = FULL ? Z + (long long)r * ld : nullptr;
    const float* z0 = FULL ? Z0 + (long long)r * ld : nullptr;
    const float4* a4 = (const float4*)a;
    const float4* z4 = (const float4*)z;
    const float4* z04 = (const float4*)z0;
    const long long T4 = T & ~3LL;
    for (long long c = tid; c < T4 / 4; c += 256) {
      const float4 x = a4[c];
      const float xa[4] = {x.x, x.y, x.z, x.w};
      if (FULL) {
        const float4 y = z4[c], w = z04[c];
        const float ya[4] = {y.x, y.y, y.z, y.w}, wa[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double xd = xa[q], zd = ya[q], z0d = wa[q];
          g = __builtin_fma(xd, xd, g);
          e = __builtin_fma(xd, fmax(z0d, 0.0), e);
          u = __builtin_fma(z0d, zd, u);
          v = __builtin_fma(z0d, z0d, v);
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double xd = xa[q];
          g = __builtin_fma(xd, xd, g);
        }
      }
    }
    for (long long t = T4 + tid; t < T; t += 256) {
      const double xd = a[t];
      g = __builtin_fma(xd, xd, g);
      if (FULL) {
        const double zd = z[t], z0d = z0[t];
        e = __builtin_fma(xd, fmax(z0d, 0.0), e);
        u = __builtin_fma(z0d, zd, u);
        v = __builtin_fma(z0d, z0d, v);
      }
    }
  }
  __shared__ double sh[4][4];
  g = wave_sum_d(g);
  if (FULL) {
    e = wave_sum_d(e);
    u = wave_sum_d(u);
    v = wave_sum_d(v);
  }
  const int lane = tid & 63, wave = tid >> 6;
  if (lane == 0) {
    sh[wave][0] = g;
    sh[wave][1] = e;
    sh[wave][2] = u;
    sh[wave][3] = v;
  }
  __syncthreads();
  if (tid < 4) {
    const double s = sh[0][tid] + sh[1][tid] + sh[2][tid] + sh[3][tid];
    if (tid == 0 || FULL) sums[(long long)tid * rows + r] = s;
    if (!(fabs(s) <= 1.79e308)) atomicCAS(status, 0, (int)STRP_ENONFINITE);
  }
}

strp_status launch_row_sums(strp_ctx* ctx, const void* A, int a_dtype, const float* Z, const float* Z0, long long ld,
                            long long T, int rows, int mode, double* sums) {
  const bool full = mode != STRP_SCORE_WANDA;
  if (full && a_dtype != STRP_F32) return fail(ctx, STRP_EINVAL, "score: LEMMA/GAIN need fp32 auxiliaries");
  dim3 grid(rows), block(256);
  const double es = a_dtype == STRP_BF16 ? 2.0 : 4.0;
  ProfScope ps(ctx, full ? "row_sums_full" : "row_sums_wanda", (full ? 8.0 : 2.0) * (double)rows * (double)T,
               (full ? 12.0 : es) * (double)rows * (double)T);
  if (full)
    hipLaunchKernelGGL((row_sums_kernel<false, true>), grid, block, 0, ctx->stream, A, Z, Z0, ld, T, rows, sums, ctx->status_dev);
  else if (a_dtype == STRP_BF16)
    hipLaunchKernelGGL((row_sums_kernel<true, false>), grid, block, 0, ctx->stream, A, Z, Z0, ld, T, rows, sums, ctx->status_dev);
  else
    hipLaunchKernelGGL((row_sums_kernel<false, false>), grid, block, 0, ctx->stream, A, Z, Z0, ld, T, rows, sums, ctx->status_dev);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---------------------------------------------------------------------------------------------
// squared column norms: block = 64 columns, each wavefront 8 rows x 8 groups of 8 columns at a time (128 rows per trip of
// the block: a weight matrix has too few 64-column blocks to fill the chip, so the depth of one block's loop is what it
// takes: 3072 columns of 768 rows 75 -> 9 us).  vec: 16-byte loads of 8 bf16 or 2 x 4 fp32 columns.
// ---------------------------------------------------------------------------------------------
template <bool BF16>
__device__ __forceinline__ void load8(const void* W, long long off, float (&x)[8]) {
  if (BF16) {
    const uint4 w = *(const uint4*)((const unsigned short*)W + off);
    const unsigned int u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      x[2 * q] = bf16lo(u[q]);
      x[2 * q + 1] = bf16hi(u[q]);
    }
  } else {
    const float4 a = *(const float4*)((const float*)W + off), b = *(const float4*)((const float*)W + off + 4);
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w; x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  }
}
template <bool BF16>
__device__ __forceinline__ float load1(const void* W, long long off) {
  return BF16 ? __builtin_bit_cast(float, (unsigned int)((const unsigned short*)W)[off] << 16) : ((const float*)W)[off];
}

template <bool BF16>
__global__ __launch_bounds__(1024) void colnorm2_kernel(const void* W, int rows, int cols, long long ldw, int vec, double* n2) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c0 = blockIdx.x * 64 + 8 * (lane & 7);
  const int row0 = wave * 8 + (lane >> 3);
  double acc[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q] = 0.0;
  if (vec && c0 + 8 <= cols) {
#pragma unroll 4
    for (int r = row0; r < rows; r += 128) {
      float x[8];
      load8<BF16>(W, (long long)r * ldw + c0, x);
#pragma unroll
      for (int q = 0; q < 8; ++q) acc[q] = __builtin_fma((double)x[q], (double)x[q], acc[q]);
    }
  } else {
    for (int r = row0; r < rows; r += 128)
      for (int q = 0; q < 8 && c0 + q < cols; ++q) {
        const double x = load1<BF16>(W, (long long)r * ldw + c0 + q);
        acc[q] = __builtin_fma(x, x, acc[q]);
      }
  }
  __shared__ double sh[16][64];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    acc[q] += __shfl_xor(acc[q], 8, 64);
    acc[q] += __shfl_xor(acc[q], 16, 64);
    acc[q] += __shfl_xor(acc[q], 32, 64);
  }
  if (lane < 8)
#pragma unroll
    for (int q = 0; q < 8; ++q) sh[wave][8 * lane + q] = acc[q];
  __syncthreads();
  if (tid < 64 && blockIdx.x * 64 + tid < cols) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += sh[w][tid];
    n2[blockIdx.x * 64 + tid] = t;
  }
}

strp_status launch_colnorm2(strp_ctx* ctx, const void* W, int w_dtype, int rows, int cols, long long ldw, double* n2) {
  dim3 grid((cols + 63) / 64), block(1024);
  const int vec = ((uintptr_t)W & 15) == 0 && ldw % 8 == 0;
  if (w_dtype == STRP_BF16)
    hipLaunchKernelGGL((colnorm2_kernel<true>), grid, block, 0, ctx->stream, W, rows, cols, ldw, vec, n2);
  else
    hipLaunchKernelGGL((colnorm2_kernel<false>), grid, block, 0, ctx->stream, W, rows, cols, ldw, vec, n2);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---------------------------------------------------------------------------------------------
// unit scores + layer energy (single block, fixed summation order)
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ double score_of(int mode, double n2, double g, double e, double u, double v) {
  const double w = n2 * g;
  if (mode == STRP_SCORE_WANDA) return w;
  const double p = u + n2 * e, q = v + w;
  return mode == STRP_SCORE_LEMMA ? p / q : 2.0 * p - q;
}

__global__ __launch_bounds__(1024) void unit_scores_kernel(const double* sums, const double* n2, int n_channels, int group,
                                                          int mode, float* score, double* energy_out) {
  const int n = n_channels / group;
  const double* g = sums;
  const double* e = sums + (long long)n_channels;
  const double* u = sums + 2LL * n_channels;
  const double* v = sums + 3LL * n_channels;
  double esum = 0.0;
  for (int unit = threadIdx.x; unit < n; unit += 1024) {
    double sp = 0.0, sq = 0.0, sw = 0.0;
    for (int c = 0; c < group; ++c) {
      const int j = unit * group + c;
      const double w = n2[j] * g[j];
      sw += w;
      if (mode != STRP_SCORE_WANDA) {
        sp += u[j] + n2[j] * e[j];
        sq += v[j] + w;
      }
    }
    double sc;
    if (mode == STRP_SCORE_WANDA) sc = sw;
    else if (mode == STRP_SCORE_LEMMA) sc = sp / sq;
    else sc = 2.0 * sp - sq;
    score[unit] = (float)sc;
    esum += sc;
  }
  __shared__ double sh[16];
  esum = wave_sum_d(esum);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = esum;
  __syncthreads();
  if (threadIdx.x == 0 && energy_out) {
    double tot = 0.0;
    for (int w = 0; w < 16; ++w) tot += sh[w];
    *energy_out = tot / (double)n;
  }
}

strp_status launch_unit_scores(strp_ctx* ctx, const double* sums, const double* n2, int n_channels, int group, int mode,
                               float* score, double* energy_out) {
  hipLaunchKernelGGL(unit_scores_kernel, dim3(1), dim3(1024), 0, ctx->stream, sums, n2, n_channels, group, mode, score,
                     energy_out);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---------------------------------------------------------------------------------------------
// weight statistics of a parameter group (Alg. 2 step 1): sum |w|, sum w, sum w^2 over every entry of a list of
// matrices, folded into  energy += scale (|W|_1 + cv Var(W) + c2 |W|_2).
// A model has a few hundred small groups (a head's four slices are 0.4 MB), so a call costs its launches: one for up to eight
// matrices, whose last workgroup adds the partial sums in order.  The counter that tells it belongs to the context and its
// workspace, like the sums (strp_ctx::ticket), and is zero between calls; where none was left a second launch adds them.
// ---------------------------------------------------------------------------------------------
constexpr int WSTAT_BLOCKS = 256, WSTAT_MATS = 8;

struct WeightList {
  const void* W[WSTAT_MATS];
  long long ld[WSTAT_MATS];
  int rows[WSTAT_MATS], cols[WSTAT_MATS];
  int block0[WSTAT_MATS + 1];            // workgroups block0[m] .. block0[m + 1] - 1 take matrix m
  unsigned char bf16[WSTAT_MATS], vec[WSTAT_MATS];
  int n;
};

template <bool BF16>
__device__ __forceinline__ void weight_sums(const WeightList& l, int m, unsigned int b, unsigned int blocks, double& s1, double& s, double& s2) {
  const void* W = l.W[m];
  const int cols = l.cols[m];
  const long long ld = l.ld[m];
  const unsigned int step = blocks * 256u;
  auto add = [&](float x) {
    const double v = (double)x;
    s1 += fabs(v);
    s += v;
    s2 = __builtin_fma(v, v, s2);
  };
  if (l.vec[m]) {                        // groups of eight columns; below 2^35 entries
    const unsigned int per = (unsigned int)cols >> 3, n = (unsigned int)l.rows[m] * per;
#pragma unroll 4
    for (unsigned int g = b * 256u + threadIdx.x; g < n; g += step) {
      const unsigned int r = g / per;
      float x[8];
      load8<BF16>(W, (long long)r * ld + 8 * (long long)(g - r * per), x);
#pragma unroll
      for (int q = 0; q < 8; ++q) add(x[q]);
    }
  } else {
    // entry by entry; row and column go on by the step's own (a division per entry cost more than its load)
    const unsigned int e = b * 256u + threadIdx.x, dr = step / cols, dc = step % cols;
    unsigned int c = e % cols;
    for (long long r = e / cols; r < l.rows[m]; r += dr) {
      add(load1<BF16>(W, r * ld + c));
      c += dc;
      if (c >= (unsigned int)cols) {
        c -= cols;
        ++r;
      }
    }
  }
}

// what becomes of the sums
struct WeightEnd {
  double count, var_coef, l2_coef, scale;
  double* energy;
  unsigned int* ticket;                  // null: another launch follows
  int filled;                            // entries of partial once this launch is done
};
// by the first wavefront of a workgroup
__device__ __forceinline__ void weight_energy(const double* partial, const WeightEnd& e) {
  double a[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
  for (int b = threadIdx.x; b < e.filled; b += 64)
#pragma unroll
    for (int q = 0; q < 3; ++q) a[q] += agent_get(&partial[3 * b + q]);
#pragma unroll
  for (int q = 0; q < 3; ++q) a[q] = wave_allsum_d(a[q]);
  if (threadIdx.x != 0) return;
  const double mean = a[1] / e.count;
  const double var = a[2] / e.count - mean * mean;
  *e.energy += e.scale * (a[0] + e.var_coef * var + e.l2_coef * sqrt(a[2]));
}

// partial: [WSTAT_BLOCKS][3]; the first `filled` entries hold the sums of earlier launches of the same call
__global__ __launch_bounds__(256) void weight_sums_kernel(const WeightList l, int filled, double* partial, const WeightEnd end) {
  __shared__ unsigned int flag;
  double s1 = 0.0, s = 0.0, s2 = 0.0;
  int m = 0;
  while (m + 1 < l.n && (int)blockIdx.x >= l.block0[m + 1]) ++m;
  const unsigned int b = blockIdx.x - l.block0[m], blocks = l.block0[m + 1] - l.block0[m];
  if (l.bf16[m]) weight_sums<true>(l, m, b, blocks, s1, s, s2);
  else weight_sums<false>(l, m, b, blocks, s1, s, s2);
  __shared__ double red[4][3];
  s1 = wave_sum_d(s1);
  s = wave_sum_d(s);
  s2 = wave_sum_d(s2);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (lane == 0) {
    red[wave][0] = s1;
    red[wave][1] = s;
    red[wave][2] = s2;
  }
  __syncthreads();
  if (tid < 3) {
    double* p = &partial[3 * blockIdx.x + tid];
    const double before = (int)blockIdx.x < filled ? *p : 0.0;
    agent_put(p, before + (red[0][tid] + red[1][tid] + red[2][tid] + red[3][tid]));
  }
  if (!end.ticket || !last_block(end.ticket, &flag)) return;
  if (tid == 64) *end.ticket = 0u;
  if (tid < 64) weight_energy(partial, end);
}

__global__ __launch_bounds__(64) void weight_energy_kernel(const double* partial, const WeightEnd end) { weight_energy(partial, end); }

strp_status launch_weight_energy(strp_ctx* ctx, const strp_weight_ref* mats, int n_mats, double var_coef, double l2_coef, double scale,
                                 double* energy, double* partial) {
  WeightList l;
  WeightEnd end{0.0, var_coef, l2_coef, scale, energy, nullptr, 0};
  int filled = 0;
  for (int i = 0; i < n_mats; ++i) end.count += (double)mats[i].rows * (double)mats[i].cols;
  for (int i0 = 0; i0 < n_mats; i0 += WSTAT_MATS) {
    l.n = n_mats - i0 < WSTAT_MATS ? n_mats - i0 : WSTAT_MATS;
    double cost[WSTAT_MATS], total = 0.0;
    for (int i = 0; i < l.n; ++i) {
      const strp_weight_ref& m = mats[i0 + i];
      l.W[i] = m.W; l.rows[i] = m.rows; l.cols[i] = m.cols; l.ld[i] = m.ld;
      l.bf16[i] = m.dtype == STRP_BF16;
      l.vec[i] = ((uintptr_t)m.W & 15) == 0 && m.cols % 8 == 0 && m.ld % 8 == 0 && (double)m.rows * m.cols < 3.0e10;
      // workgroups' worth of work: four groups of eight entries per thread, all requested at once; an entry that comes by
      // itself takes about five times as long as one of a group (67 million: 298 us against 57 with 256 workgroups)
      cost[i] = (double)m.rows * m.cols / (32.0 * 256.0) * (l.vec[i] ? 1.0 : 5.0);
      if (cost[i] < 1.0) cost[i] = 1.0;
      total += cost[i];
    }
    // the workgroups are dealt out by the work: with an even share by place in the list, a matrix of 2048 x 8193 behind seven
    // small ones took 715 us instead of 81
    l.block0[0] = 0;
    for (int i = 0; i < l.n; ++i)
      l.block0[i + 1] = l.block0[i] + (total <= WSTAT_BLOCKS ? (int)cost[i] : 1 + (int)((WSTAT_BLOCKS - l.n) * (cost[i] / total)));
    end.filled = l.block0[l.n] > filled ? l.block0[l.n] : filled;
    if (i0 + WSTAT_MATS >= n_mats) end.ticket = ctx->ticket;
    hipLaunchKernelGGL(weight_sums_kernel, dim3(l.block0[l.n]), dim3(256), 0, ctx->stream, l, filled, partial, end);
    filled = end.filled;
  }
  if (!end.ticket) hipLaunchKernelGGL(weight_energy_kernel, dim3(1), dim3(64), 0, ctx->stream, (const double*)partial, end);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}
size_t weight_energy_scratch_bytes() { return sizeof(double) * 3 * WSTAT_BLOCKS; }

// ---------------------------------------------------------------------------------------------
// softmax allocation: one wavefront, fp64, layers strided over lanes
// ---------------------------------------------------------------------------------------------
constexpr int ALLOC_MAXL = 1024;

// rule 0: r = rbar L w, clip, conditional rescale (Alg. 1);  rule 1: r = rbar L (1 - w) / sum(1 - w), clip (Alg. 2)
__global__ __launch_bounds__(64) void alloc_kernel(const double* I, int L, const int32_t* n_units, const int32_t* group_id,
                                                   double rbar, double temperature, double rmax, int rule, double* r_out,
                                                   int32_t* nprune_out) {
  __shared__ double r[ALLOC_MAXL];
  __shared__ double frac[ALLOC_MAXL];
  __shared__ int base[ALLOC_MAXL];
  __shared__ int member[ALLOC_MAXL];
  __shared__ int gids[ALLOC_MAXL];
  const int lane = threadIdx.x;
  for (int l = lane; l < L; l += 64) gids[l] = group_id ? group_id[l] : 0;
  __syncthreads();
  for (int lead = 0; lead < L; ++lead) {
    // a group is handled by its first member; its members are collected in order, 64 layers at a time
    const int gid = gids[lead];
    int Lg = 0;
    bool is_lead = true;
    for (int j0 = 0; j0 < L; j0 += 64) {
      const int j = j0 + lane;
      const bool in = j < L && gids[j] == gid;
      const unsigned long long bal = __ballot(in);
      if (__ballot(in && j < lead)) is_lead = false;
      if (in) member[Lg + __popcll(bal & ((1ull << lane) - 1ull))] = j;
      Lg += __popcll(bal);
    }
    if (!is_lead) continue;                    // uniform across the wavefront
    __syncthreads();
    // scale by mean |I|, softmax of -I/T with the maximum subtracted
    double sabs = 0.0;
    for (int q = lane; q < Lg; q += 64) sabs += fabs(I[member[q]]);
    sabs = wave_allsum_d(sabs);
    const double scale = sabs / (double)Lg;
    double amax = -1.0e308;
    for (int q = lane; q < Lg; q += 64) {
      const double a = (scale > 0.0) ? -(I[member[q]] / scale) / temperature : 0.0;
      r[q] = a;
      amax = fmax(amax, a);
    }
    amax = wave_allmax_d(amax);
    double wsum = 0.0;
    for (int q = lane; q < Lg; q += 64) {
      const double w = exp(r[q] - amax);
      r[q] = w;
      wsum += w;
    }
    wsum = wave_allsum_d(wsum);
    int at_max = 0;
    double rsum = 0.0;
    for (int q = lane; q < Lg; q += 64) {
      const double w = r[q] / wsum;
      double rv = rbar * (double)Lg * w;
      if (rule == 1) rv = Lg > 1 ? rbar * (double)Lg * (1.0 - w) / (double)(Lg - 1) : rbar;   // sum(1 - w) = L - 1
      rv = fmin(fmax(rv, 0.0), rmax);
      r[q] = rv;
      at_max |= (rv == rmax);
      rsum += rv;
    }
    at_max = __any(at_max);
    rsum = wave_allsum_d(rsum);
    if (!at_max && rule == 0) {
      const double mu = rsum / (double)Lg;
      for (int q = lane; q < Lg; q += 64) r[q] = fmin(fmax(r[q] * (rbar / mu), 0.0), rmax);
    }
    // largest-remainder integer counts
    double xsum = 0.0;
    long long bsum = 0;
    for (int q = lane; q < Lg; q += 64) {
      const double x = r[q] * (double)n_units[member[q]];
      const double fl = floor(x);
      base[q] = (int)fl;
      frac[q] = x - fl;
      xsum += x;
      bsum += (long long)fl;
    }
    xsum = wave_allsum_d(xsum);
    bsum = (long long)wave_allsum_d((double)bsum);
    const int extra = (int)(rint(xsum) - (double)bsum);
    __syncthreads();
    for (int q = lane; q < Lg; q += 64) {
      int rank = 0;
      const double fq = frac[q];
      for (int j = 0; j < Lg; ++j) rank += (frac[j] > fq) || (frac[j] == fq && j < q);
      int b = base[q] + ((rank < extra) ? 1 : 0);
      const int nu = n_units[member[q]];
      b = b > nu - 1 ? nu - 1 : b;
      b = b < 0 ? 0 : b;
      r_out[member[q]] = r[q];
      nprune_out[member[q]] = b;
    }
    __syncthreads();
  }
}

strp_status launch_alloc(strp_ctx* ctx, const double* energies, int L, const int32_t* n_units, const int32_t* group_id,
                         double rbar, double temperature, double rmax, int rule, double* r_out, int32_t* nprune_out) {
  if (L <= 0 || L > ALLOC_MAXL) return fail(ctx, STRP_EINVAL, "alloc: L=%d outside [1, %d]", L, ALLOC_MAXL);
  hipLaunchKernelGGL(alloc_kernel, dim3(1), dim3(64), 0, ctx->stream, energies, L, n_units, group_id, rbar, temperature,
                     rmax, rule, r_out, nprune_out);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---------------------------------------------------------------------------------------------
// top-k select.  Scores are compared as order-preserving integer keys; equal keys keep the lower index.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ unsigned int score_key(float x) {
  const unsigned int u = __builtin_bit_cast(unsigned int, x + 0.0f);   // -0 and +0 are one value: both map to +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_score(unsigned int k) {
  const unsigned int u = (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
  return __builtin_bit_cast(float, u);
}

// nothing (k = 0) or everything (k = n) is kept
__global__ __launch_bounds__(1024) void topk_all_kernel(const float* score, int n, int keep, int group, uint8_t* mask, int32_t* idx, float* tau) {
  __shared__ float wmin[16];
  const int tid = threadIdx.x;
  float t = keep ? __builtin_nanf("") : __builtin_inff();     // fminf passes over NaN: the minimum is NaN only if every score is
  for (int i = tid; i < n; i += 1024) {
    mask[i] = (uint8_t)keep;
    if (keep) {
      t = fminf(t, score[i]);
      for (int c = 0; c < group; ++c) idx[(long long)i * group + c] = i * group + c;
    }
  }
  for (int o = 32; o > 0; o >>= 1) t = fminf(t, __shfl_down(t, o, 64));
  if ((tid & 63) == 0) wmin[tid >> 6] = t;
  __syncthreads();
  if (tid == 0 && tau) {
    for (int w = 1; w < 16; ++w) t = fminf(t, wmin[w]);
    *tau = t;
  }
}

// Wave-wide in registers: DPP moves instead of LDS permutes, which take 100 cycles a step where nothing else runs.
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned int dpp_move(unsigned int old, unsigned int x) {
  return (unsigned int)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROWS, 0xf, false);
}
// f over the lanes: the last one has all of them, and every lane those up to its own (inclusive scan); id is f's neutral element
template <typename F>
__device__ __forceinline__ unsigned int wave_scan(unsigned int x, unsigned int id, F f) {
  x = f(x, dpp_move<0x111, 0xf>(id, x));       // row_shr 1, 2, 4, 8
  x = f(x, dpp_move<0x112, 0xf>(id, x));
  x = f(x, dpp_move<0x114, 0xf>(id, x));
  x = f(x, dpp_move<0x118, 0xf>(id, x));
  x = f(x, dpp_move<0x142, 0xa>(id, x));       // row_bcast 15 into rows 1 and 3, 31 into rows 2 and 3
  x = f(x, dpp_move<0x143, 0xc>(id, x));
  return x;
}
__device__ __forceinline__ unsigned int wave_sum_scan(unsigned int x) {
  return wave_scan(x, 0u, [](unsigned int a, unsigned int b) { return a + b; });
}

// exclusive prefix, in thread order, of a per-thread count over the block; *total = the block's sum
__device__ __forceinline__ int block_scan(int cnt, int* wave_tot, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int inc = (int)wave_sum_scan((unsigned int)cnt);
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  int off = 0, tot = 0;
  const int nw = blockDim.x >> 6;
  for (int w = 0; w < nw; ++w) {
    const int c = wave_tot[w];
    if (w < wave) off += c;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return off + inc - cnt;
}

// Suffix scan of a histogram of B * 1024 bins (or B * 512, by blockDim) for the bin that holds the krem-th largest entry:
// thread t owns bins B t .. B t + B - 1.  out[0] = bin, out[1] = entries above it, out[2] = entries in it (LDS).
template <int B, int WAVES>
__device__ __forceinline__ void pick_bin(const unsigned int (&h)[B], unsigned int krem, unsigned int* wave_tot, unsigned int* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned int own = 0;
#pragma unroll
  for (int b = 0; b < B; ++b) own += h[b];
  const unsigned int inc = wave_sum_scan(own);
  if (lane == 63) wave_tot[wave] = inc;
  __syncthreads();
  unsigned int above = 0u - inc;      // entries in the bins of later threads
#pragma unroll
  for (int w = 0; w < WAVES; ++w) above += w >= wave ? wave_tot[w] : 0u;
#pragma unroll
  for (int b = B - 1; b >= 0; --b) {
    if (above < krem && above + h[b] >= krem) {
      out[0] = (unsigned int)(B * tid + b);
      out[1] = above;
      out[2] = h[b];
    }
    above += h[b];
  }
  __syncthreads();
}

// One vector of scores (0 < k < n) by one block of 1024 threads, which keeps their keys in registers (REGS, up to 4096 R of them; beyond 16 a
// thread each phase reads them again, from the L2, 4096 R at a time): thread t has elements 4096 j + 4 t + e, so that scores, masks and sums move 16 bytes a lane, and the ascending indices need one scan of four counts.
// What bounds it is the number of dependent block-wide phases, so the threshold is found in few of them: a histogram of 2048
// bins stretched over the keys that are there (real scores share a handful of exponents: bins at fixed bit positions
// would put them, and the LDS atomics that count them, in a few places), the bin with the k-th largest key, and the rank
// of each of the bin's keys among themselves; a bin of more than 128 keys is stretched again (ranking 900 took 25 us, a round 1.5).  The k-th key
// and its index decide every element: kept = larger, or equal with no higher index.
// Before (strided keys, a scan of 256 counts, LDS permutes, up to 1024 keys ranked) / now: 16384 scores 13.9 / 9.3 us with the launch;
// in a step, with the scores formed first, 2312 35.7 / 11.3 and 256 8.3 / 5.7; read again in each phase, 20480 23.1 / 18.9, 32768 31.7 / 19.9,
// 32769 35.7 / 26.9, 49152 44.4 / 27.5, 65536 57.9 / 39.2 (65537, in four launches, 29.1 / 21.3).
// With in.sums the scores (group = 1) are formed here first, with their mean; rest takes the indices that are not kept.
struct ScoreSource {
  const double* sums;       // [4][n], or null: the scores are given
  const double* n2;
  int mode;
  double* energy_out;
};
constexpr int SELECT_RANKED = 128;
template <int R, bool SCORED, bool REGS>
__global__ __launch_bounds__(1024) void topk_small_kernel(float* score, int n, int k, int group, int vec, uint8_t* mask, int32_t* idx, float* tau,
                                                          const ScoreSource in, int32_t* rest) {
  __shared__ unsigned int hist[2048];
  __shared__ unsigned int ckey[SELECT_RANKED];
  __shared__ int cidx[SELECT_RANKED];
  __shared__ unsigned int wt[2][16];
  __shared__ unsigned int sel[3], ncand, cut[2];
  __shared__ unsigned int wtot[16][(R + 1) / 2];
  __shared__ double esums[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  unsigned int key[R][4];
  const int rounds = REGS ? R : (n + 4096 * R - 1) / (4096 * R) * R;
  const auto at = [&](int j) { return 4096 * j + 4 * tid; };
  const auto load = [&](int j0) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      float x[4];
      if (vec && at(j0 + j) + 4 <= n) {
        const float4 v = *(const float4*)(score + at(j0 + j));
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = score[at(j0 + j) + e < n ? at(j0 + j) + e : n - 1];       // past the end: the last one again
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) key[j][e] = score_key(x[e]);
    }
  };
  if constexpr (SCORED) {
    const long long nn = n;
    const double* g = in.sums;
    const bool full = in.mode != STRP_SCORE_WANDA;
    double esum = 0.0;
    const auto form = [&](int j, unsigned int* keys) {
      double sc[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = at(j) + e < n ? at(j) + e : n - 1;
        sc[e] = score_of(in.mode, in.n2[i], g[i], full ? g[nn + i] : 0.0, full ? g[2 * nn + i] : 0.0, full ? g[3 * nn + i] : 0.0);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (REGS) keys[e] = score_key((float)sc[e]);
        if (at(j) + e < n) {
          esum += sc[e];
          score[at(j) + e] = (float)sc[e];
        }
      }
    };
    if constexpr (REGS) {
#pragma unroll
      for (int j = 0; j < R; ++j) form(j, key[j]);
    } else {
      for (int j = 0; j < rounds; ++j) form(j, nullptr);
    }
    esum = wave_sum_d(esum);
    if (lane == 0) esums[wave] = esum;
    if (!REGS) __syncthreads();          // the last score, which every thread may read
  } else if constexpr (REGS) {
    load(0);
  }
  // f(index, key, index < n) for each element
  const auto each = [&](auto f) {
    for (int j0 = 0; j0 < rounds; j0 += R) {
      if (!REGS) load(j0);
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) f(at(j0 + j) + e, key[j][e], at(j0 + j) + e < n);
    }
  };
  unsigned int lo = 0xffffffffu, hi = 0u;
  each([&](int, unsigned int x, bool) {
    lo = x < lo ? x : lo;
    hi = x > hi ? x : hi;
  });
  lo = wave_scan(lo, 0xffffffffu, [](unsigned int a, unsigned int b) { return a < b ? a : b; });
  hi = wave_scan(hi, 0u, [](unsigned int a, unsigned int b) { return a > b ? a : b; });
  if (lane == 63) {
    wt[0][wave] = lo;
    wt[1][wave] = hi;
  }
  hist[tid] = 0;
  hist[tid + 1024] = 0;
  if (tid == 0) ncand = 0;
  __syncthreads();
  if constexpr (SCORED) {
    if (tid == 0 && in.energy_out) {
      double tot = 0.0;
      for (int w = 0; w < 16; ++w) tot += esums[w];
      *in.energy_out = tot / (double)n;
    }
  }
  lo = 0xffffffffu;
  hi = 0u;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    lo = wt[0][w] < lo ? wt[0][w] : lo;
    hi = wt[1][w] > hi ? wt[1][w] : hi;
  }
  unsigned int krem = (unsigned int)k, count;
  int shift;
  for (;;) {
    // the keys in [lo, hi] by 2048 bins
    const unsigned int range = hi - lo;
    shift = range ? 32 - __builtin_clz(range) - 11 : 0;
    shift = shift > 0 ? shift : 0;
    each([&](int, unsigned int x, bool is) {
      if (is && x >= lo && x <= hi) atomicAdd(&hist[(x - lo) >> shift], 1u);
    });
    __syncthreads();
    const unsigned int h[2] = {hist[2 * tid], hist[2 * tid + 1]};
    pick_bin<2, 16>(h, krem, wt[0], sel);
    krem -= sel[1];
    count = sel[2];
    lo += sel[0] << shift;
    const unsigned int width = (1u << shift) - 1u;
    hi = hi - lo > width ? lo + width : hi;
    if (count <= SELECT_RANKED || shift == 0) break;
    hist[tid] = 0;
    hist[tid + 1024] = 0;
    __syncthreads();
  }
  // pre[j]: run and the sum of cnt over the elements before this thread's of the j-th of R rounds; run goes on.  Two rounds' counts in
  // the halves of a word
  const auto before = [&](const unsigned int (&cnt)[R], unsigned int (&pre)[R], unsigned int& run) {
    constexpr int Q = (R + 1) / 2;
    unsigned int own[Q], inc[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      own[q] = cnt[2 * q] | (2 * q + 1 < R ? cnt[2 * q + 1 < R ? 2 * q + 1 : 0] << 16 : 0u);
      inc[q] = wave_sum_scan(own[q]);
    }
    if (lane == 63)
#pragma unroll
      for (int q = 0; q < Q; ++q) wtot[wave][q] = inc[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      unsigned int low = inc[q] - own[q], all = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) {
        const unsigned int t = wtot[w][q];
        low += w < wave ? t : 0u;
        all += t;
      }
      pre[2 * q] = run + (low & 0xffffu);
      run += all & 0xffffu;
      if (2 * q + 1 < R) pre[2 * q + 1 < R ? 2 * q + 1 : 0] = run + (low >> 16);
      run += all >> 16;
    }
    if (!REGS) __syncthreads();
  };
  // the krem largest of the `count` keys in [lo, hi]
  if (count <= SELECT_RANKED) {
    each([&](int i, unsigned int x, bool is) {
      if (is && x >= lo && x <= hi) {
        const unsigned int q = atomicAdd(&ncand, 1u);
        ckey[q] = x;
        cidx[q] = i;
      }
    });
    __syncthreads();
    // rank of each candidate: eight lanes share one
    const int c = tid >> 3;
    if (c < (int)count) {
      const unsigned int kc = ckey[c];
      const int ic = cidx[c];
      int rank = 0;
      for (int q = tid & 7; q < (int)count; q += 8) rank += (ckey[q] > kc || (ckey[q] == kc && cidx[q] < ic)) ? 1 : 0;
      rank += __shfl_xor(rank, 1, 64);
      rank += __shfl_xor(rank, 2, 64);
      rank += __shfl_xor(rank, 4, 64);
      if (rank == (int)krem - 1) {
        cut[0] = kc;
        cut[1] = (unsigned int)ic;
      }
    }
    __syncthreads();
  } else {
    // more equal keys than that (lo == hi): the krem-th in index order
    unsigned int run = 0;
    for (int j0 = 0; j0 < rounds; j0 += R) {
      unsigned int cnt[R], pre[R];
      if (!REGS) load(j0);
#pragma unroll
      for (int j = 0; j < R; ++j) {
        cnt[j] = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) cnt[j] += at(j0 + j) + e < n && key[j][e] == lo ? 1u : 0u;
      }
      before(cnt, pre, run);
#pragma unroll
      for (int j = 0; j < R; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (at(j0 + j) + e < n && key[j][e] == lo && ++pre[j] == krem) {
            cut[0] = lo;
            cut[1] = (unsigned int)(at(j0 + j) + e);
          }
    }
    __syncthreads();
  }
  const unsigned int ckth = cut[0];
  const int ikth = (int)cut[1];
  if (tid == 0 && tau) *tau = key_score(ckth);
  unsigned int run = 0;
  for (int j0 = 0; j0 < rounds; j0 += R) {
    unsigned int keep[R], cnt[R], pre[R];
    if (!REGS) load(j0);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int i0 = at(j0 + j);
      keep[j] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) keep[j] |= (i0 + e < n && (key[j][e] > ckth || (key[j][e] == ckth && i0 + e <= ikth)) ? 1u : 0u) << e;
      cnt[j] = (unsigned int)__popc(keep[j]);
      if (vec && i0 + 4 <= n) {
        *(unsigned int*)(mask + i0) = (keep[j] & 1u) | (keep[j] & 2u) << 7 | (keep[j] & 4u) << 14 | (keep[j] & 8u) << 21;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (i0 + e < n) mask[i0 + e] = (uint8_t)((keep[j] >> e) & 1u);
      }
    }
    before(cnt, pre, run);
#pragma unroll
    for (int j = 0; j < R; ++j) {
      unsigned int pos = pre[j];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = at(j0 + j) + e;
        if ((keep[j] >> e) & 1u) {
          if (group == 1) idx[pos] = i;
          else
            for (int c = 0; c < group; ++c) idx[(long long)pos * group + c] = i * group + c;
          ++pos;
        } else if (SCORED && rest && i < n) {
          rest[i - (int)pos] = i;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// top-k select over a long score vector (all layers' scores at once for a global threshold, or a stress input), in four
// launches, each reading the scores once; the last workgroup of each of the first three (device counter) makes the choice
// that the next one needs, so no launch is spent on it:
//   hist 0   histogram of the top 13 key bits (sign, exponent, 4 mantissa bits); the bin of the k-th largest key
//   hist 1   of the keys in that bin, the next 13 bits
//   count    per workgroup: keys above the 26-bit prefix, and (few) keys that have it by their last 6 bits;
//            then the threshold itself, and per workgroup where its kept entries go and how many of its entries equal to
//            the threshold are kept (lower indices first)
//   write    mask and ascending indices
// Every input takes the same path, also one of equal scores.  48 x 28672 scores: 66 -> 34 us against eight launches, 31.7 with a trip's
// scores on their way while the one before is counted and the bins of a workgroup read and cleared 16 bytes or 16 counts at a time;
// 70 thousand 28.2 -> 20.4 by that and by the number of workgroups (big_plan).
// ---------------------------------------------------------------------------------------------
namespace big {
constexpr int BINS = 8192;          // 13 bits
constexpr int THREADS = 512;
constexpr int MAXBLOCKS = 512;
struct State {
  unsigned int ghist[2][BINS];      // these and the counters are cleared before every select
  unsigned int glow[64];            // keys with the 26-bit prefix, by their last 6 bits
  unsigned int done[3];             // workgroups that have finished, per launch
  unsigned int clear_end;
  unsigned int prefix[2];           // chosen 13-bit and 26-bit prefix
  unsigned int krem[2];             // keys still to keep among those that have it
  unsigned int thr;                 // the k-th largest key
  unsigned int gt[MAXBLOCKS];       // keys above the 26-bit prefix in the workgroup's chunk
  unsigned int suf[MAXBLOCKS][65];  // keys with the prefix whose last 6 bits are not below the index
  unsigned int kpre[MAXBLOCKS];     // kept entries before the chunk
  unsigned int eqkeep[MAXBLOCKS];   // entries equal to the threshold that the chunk keeps
};
}  // namespace big

static void big_plan(long long n, int* blocks, long long* chunk) {
  // A trip of a workgroup is 4096 scores.  More workgroups read faster, but each adds its counts of the same few hundred bins to the
  // global histogram, and adds to one address go one after another: about 0.02 us a workgroup and launch, against 5 us a trip for the
  // four together.  us, one trip / two: 300 thousand scores 22.9 / 24.5, 500 thousand 25.5 / 25.5, 1.04 million 32.4 / 29.3; two / three
  // at 2.09 million 36.6 / 35.7; 128 / 256 workgroups at 1.7 million 35.0 / 33.6, 256 / 512 at 6 million 53.4 / 60.8, at 12 million 76.9 (367) / 89.2.
  long long trips = 1;
  auto most = [&]() { return trips > 8 ? (long long)big::MAXBLOCKS : trips > 2 ? 256ll : 96 * trips; };
  while ((n + big::THREADS * 8 * trips - 1) / (big::THREADS * 8 * trips) > most()) ++trips;
  const long long c = trips * (8 * big::THREADS);
  *blocks = (int)((n + c - 1) / c);
  *chunk = c;
}

size_t topk_scratch_bytes(int n) { return n <= SELECT_MAX ? 0 : ((sizeof(big::State) + 255) & ~size_t(255)); }

// eight consecutive scores of a thread
struct BigTrip {
  float4 a, b;
  bool whole;
  __device__ __forceinline__ void load(const float* score, long long i0, long long end, int vec) {
    whole = vec && i0 + 8 <= end;
    if (whole) {
      a = *(const float4*)(score + i0);
      b = *(const float4*)(score + i0 + 4);
    }
  }
  template <typename F>
  __device__ __forceinline__ void each(const float* score, long long i0, long long end, F f) const {
    if (whole) {
      const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) f(score_key(x[e]));
    } else {
      for (long long i = i0; i < end && i < i0 + 8; ++i) f(score_key(score[i]));
    }
  }
};
// f(key) for this workgroup's chunk; first: the thread's first trip, which the kernel asks for before anything else.  The next trip
// is on its way while one is counted: with one at a time in flight a launch was two round trips to memory longer.
template <typename F>
__device__ __forceinline__ void big_scan(BigTrip t, const float* score, long long beg, long long end, int vec, F f) {
  for (long long i0 = beg + 8 * (long long)threadIdx.x; i0 < end; i0 += 8 * big::THREADS) {
    BigTrip next;
    next.load(score, i0 + 8 * big::THREADS, end, vec);
    t.each(score, i0, end, f);
    t = next;
  }
}
__device__ __forceinline__ void clear_bins(unsigned int (&hist)[big::BINS]) {
#pragma unroll
  for (int q = 0; q < big::BINS / 4 / big::THREADS; ++q) ((uint4*)hist)[threadIdx.x + big::THREADS * q] = make_uint4(0, 0, 0, 0);
}
template <int LEVEL>
__global__ __launch_bounds__(big::THREADS) void topk_hist_kernel(const float* score, long long n, long long k, long long chunk, int vec, big::State* st) {
  __shared__ __attribute__((aligned(16))) unsigned int hist[big::BINS];
  __shared__ unsigned int wt[8], sel[3], flag;
  const int tid = threadIdx.x;
  const long long beg = (long long)blockIdx.x * chunk, end = beg + chunk < n ? beg + chunk : n;
  BigTrip first;
  first.load(score, beg + 8 * tid, end, vec);
  clear_bins(hist);
  const unsigned int prefix = LEVEL ? st->prefix[0] : 0u;
  __syncthreads();
  big_scan(first, score, beg, end, vec, [&](unsigned int key) {
    if (LEVEL == 0) atomicAdd(&hist[key >> 19], 1u);
    else if (key >> 19 == prefix) atomicAdd(&hist[(key >> 6) & 8191u], 1u);
  });
  __syncthreads();
  unsigned int h[16];
#pragma unroll
  for (int b = 0; b < 16; ++b) h[b] = hist[tid + big::THREADS * b];
#pragma unroll
  for (int b = 0; b < 16; ++b)
    if (h[b]) atomicAdd(&st->ghist[LEVEL][tid + big::THREADS * b], h[b]);
  if (!last_block(&st->done[LEVEL], &flag)) return;
  // through LDS: consecutive threads read consecutive counts
#pragma unroll
  for (int b = 0; b < 16; ++b) h[b] = agent_get(&st->ghist[LEVEL][tid + big::THREADS * b]);
#pragma unroll
  for (int b = 0; b < 16; ++b) hist[tid + big::THREADS * b] = h[b];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < 16; ++b) h[b] = hist[16 * tid + b];
  const unsigned int krem = LEVEL ? st->krem[0] : (unsigned int)k;
  pick_bin<16, 8>(h, krem, wt, sel);
  if (tid == 0) {
    st->prefix[LEVEL] = LEVEL ? (prefix << 13) | sel[0] : sel[0];
    st->krem[LEVEL] = krem - sel[1];
  }
}

__global__ __launch_bounds__(big::THREADS) void topk_count_kernel(const float* score, long long n, long long chunk, int vec, float* tau, big::State* st) {
  __shared__ unsigned int low[64], gts, flag, s_low, s_above;
  __shared__ int wtot[8];
  const int tid = threadIdx.x;
  const long long beg = (long long)blockIdx.x * chunk, end = beg + chunk < n ? beg + chunk : n;
  BigTrip first;
  first.load(score, beg + 8 * tid, end, vec);
  if (tid < 64) low[tid] = 0;
  if (tid == 0) gts = 0;
  const unsigned int prefix = st->prefix[1];
  __syncthreads();
  unsigned int above = 0;
  big_scan(first, score, beg, end, vec, [&](unsigned int key) {
    const unsigned int p = key >> 6;
    above += p > prefix ? 1u : 0u;
    if (p == prefix) atomicAdd(&low[key & 63u], 1u);
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) above += __shfl_down(above, o, 64);
  if ((tid & 63) == 0) atomicAdd(&gts, above);
  __syncthreads();
  if (tid < 64) {
    const unsigned int c = low[tid];
    unsigned int suf = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned int v = __shfl_down(suf, o, 64);
      if (tid + o < 64) suf += v;
    }
    agent_put(&st->suf[blockIdx.x][tid], suf);
    if (c) atomicAdd(&st->glow[tid], c);
  }
  if (tid == 64) agent_put(&st->gt[blockIdx.x], gts);
  if (tid == 65) agent_put(&st->suf[blockIdx.x][64], 0u);
  if (!last_block(&st->done[2], &flag)) return;
  const int blocks = (int)gridDim.x;
  // the last six bits of the threshold
  if (tid < 64) {
    const unsigned int krem = st->krem[1];
    const unsigned int c = agent_get(&st->glow[tid]);
    unsigned int suf = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned int v = __shfl_down(suf, o, 64);
      if (tid + o < 64) suf += v;
    }
    const unsigned int over = suf - c;
    if (over < krem && suf >= krem) {
      s_low = (unsigned int)tid;
      s_above = krem - over;             // entries equal to the threshold that are kept
      st->thr = (prefix << 6) | (unsigned int)tid;
      if (tau) *tau = key_score((prefix << 6) | (unsigned int)tid);
    }
  }
  __syncthreads();
  // per workgroup (one thread each): entries above the threshold and equal to it, then their prefixes
  unsigned int g = 0, e = 0;
  if (tid < blocks) {
    const unsigned int over = agent_get(&st->suf[tid][s_low + 1]);
    e = agent_get(&st->suf[tid][s_low]) - over;
    g = agent_get(&st->gt[tid]) + over;
  }
  int tot;
  const unsigned int ebefore = (unsigned int)block_scan((int)e, wtot, &tot);
  const unsigned int ekeep = ebefore >= s_above ? 0u : (e < s_above - ebefore ? e : s_above - ebefore);
  const unsigned int kpre = (unsigned int)block_scan((int)(g + ekeep), wtot, &tot);
  if (tid < blocks) {
    st->kpre[tid] = kpre;
    st->eqkeep[tid] = ekeep;
  }
}

// mask and ascending indices of [beg, end): the keys above thr and the first eqkeep equal to it; run = kept entries before beg
__device__ __forceinline__ void big_write(const BigTrip& first, const float* score, long long beg, long long end, int vec, int group, uint8_t* mask, int32_t* idx,
                                          unsigned int thr, unsigned int eqkeep, unsigned int run, int* wtot) {
  unsigned int eqrun = 0;
  BigTrip t = first;
  for (long long base = beg; base < end; base += 8 * big::THREADS) {
    const long long i0 = base + 8 * (long long)threadIdx.x;
    const bool whole = t.whole;
    unsigned int gt = 0, eq = 0, e8 = 0;
    BigTrip next;
    next.load(score, i0 + 8 * big::THREADS, end, vec);
    t.each(score, i0, end, [&](unsigned int key) {
      gt |= (key > thr ? 1u : 0u) << e8;
      eq |= (key == thr ? 1u : 0u) << e8;
      ++e8;
    });
    t = next;
    // both prefixes in one scan: at most 4096 entries each
    int tot;
    const int pre = block_scan((int)((unsigned)__popc(gt) | ((unsigned)__popc(eq) << 16)), wtot, &tot);
    const unsigned int gpre = (unsigned)pre & 0xffffu, epre = eqrun + ((unsigned)pre >> 16);
    unsigned int ekept_before = epre < eqkeep ? epre : eqkeep, keep = gt;
    unsigned int pos = run + gpre + (ekept_before - (eqrun < eqkeep ? eqrun : eqkeep));
    unsigned int left = eqkeep - ekept_before;
    for (unsigned int q = eq; q && left; q &= q - 1, --left) keep |= q & (0u - q);
    if (whole) {   // eight mask bytes in one store
      unsigned long long m8 = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) m8 |= (unsigned long long)((keep >> e) & 1u) << (8 * e);
      *(unsigned long long*)(mask + i0) = m8;
    } else {
      for (int e = 0; e < 8; ++e)
        if (i0 + e < end) mask[i0 + e] = (uint8_t)((keep >> e) & 1u);
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if ((keep >> e) & 1u) {
        for (int c = 0; c < group; ++c) idx[(long long)pos * group + c] = (int)(i0 + e) * group + c;
        ++pos;
      }
    const unsigned int etot = eqrun + ((unsigned)tot >> 16);
    run += ((unsigned)tot & 0xffffu) + ((etot < eqkeep ? etot : eqkeep) - (eqrun < eqkeep ? eqrun : eqkeep));
    eqrun = etot;
  }
}

__global__ __launch_bounds__(big::THREADS) void topk_write_kernel(const float* score, long long n, long long chunk, int vec, int group, uint8_t* mask,
                                                                  int32_t* idx, const big::State* st) {
  __shared__ int wtot[8];
  const long long beg = (long long)blockIdx.x * chunk, end = beg + chunk < n ? beg + chunk : n;
  BigTrip first;
  first.load(score, beg + 8 * threadIdx.x, end, vec);
  big_write(first, score, beg, end, vec, group, mask, idx, st->thr, st->eqkeep[blockIdx.x], st->kpre[blockIdx.x], wtot);
}

// The same select by one workgroup with its histograms in LDS, for a caller of groups (group > 1) who has set no workspace
// large enough for the four launches.  One CU's loads bound it, so it is taken for nothing else.
__global__ __launch_bounds__(big::THREADS) void topk_lone_kernel(const float* score, long long n, long long k, int vec, int group, uint8_t* mask,
                                                                 int32_t* idx, float* tau) {
  __shared__ __attribute__((aligned(16))) unsigned int hist[big::BINS];
  __shared__ unsigned int wt[8], sel[3];
  __shared__ int wtot[8];
  const int tid = threadIdx.x;
  BigTrip first;
  first.load(score, 8 * tid, n, vec);
  unsigned int prefix = 0, krem = (unsigned int)k;
  for (int level = 0; level < 3; ++level) {      // key bits 31 .. 19, 18 .. 6, 5 .. 0
    const int shift = level == 0 ? 19 : level == 1 ? 6 : 0, bits = level == 2 ? 6 : 13;
    clear_bins(hist);
    __syncthreads();
    big_scan(first, score, 0, n, vec, [&](unsigned int key) {
      if (level == 0 || key >> (shift + bits) == prefix) atomicAdd(&hist[(key >> shift) & ((1u << bits) - 1u)], 1u);
    });
    __syncthreads();
    unsigned int h[16];
#pragma unroll
    for (int b = 0; b < 16; ++b) h[b] = hist[16 * tid + b];
    pick_bin<16, 8>(h, krem, wt, sel);
    prefix = (prefix << bits) | sel[0];
    krem -= sel[1];
    __syncthreads();
  }
  if (tid == 0 && tau) *tau = key_score(prefix);
  big_write(first, score, 0, n, vec, group, mask, idx, prefix, krem, 0, wtot);
}

static void launch_topk_small(strp_ctx* ctx, float* score, int n, int k, int group, uint8_t* mask, int32_t* idx, float* tau, const ScoreSource& in,
                              int32_t* rest) {
  const int vec = (((uintptr_t)score & 15) == 0 && ((uintptr_t)mask & 3) == 0) ? 1 : 0;
  const auto one = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(1), dim3(1024), 0, ctx->stream, score, n, k, group, vec, mask, idx, tau, in, rest); };
  const auto size = [&](auto scored) {
    constexpr bool S = decltype(scored)::value;
    if (n <= 4096) one(topk_small_kernel<1, S, true>);
    else if (n <= 16384) one(topk_small_kernel<4, S, true>);
    else one(topk_small_kernel<4, S, false>);
  };
  if (in.sums) size(std::true_type{});
  else size(std::false_type{});
}

strp_status launch_select(strp_ctx* ctx, const double* sums, const double* n2, int mode, int n, int k, float* score, double* energy_out,
                          uint8_t* mask, int32_t* idx, float* tau, int32_t* rest) {
  if (k >= n) {        // everything is kept, of a vector of any length: in two steps
    STRP_TRY(launch_unit_scores(ctx, sums, n2, n, 1, mode, score, energy_out));
    return launch_topk(ctx, score, n, k, 1, mask, idx, tau, nullptr, 0);
  }
  if (n > SELECT_MAX) return fail(ctx, STRP_EINVAL, "select: %d scores, one block takes %d", n, SELECT_MAX);
  ProfScope ps(ctx, "topk", 0.0, 5.0 * (double)n + 4.0 * (double)k);
  launch_topk_small(ctx, score, n, k, 1, mask, idx, tau, ScoreSource{sums, n2, mode, energy_out}, rest);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

strp_status launch_topk(strp_ctx* ctx, const float* score, int n, int k, int group, uint8_t* mask, int32_t* idx, float* tau,
                        void* scratch, size_t scratch_bytes) {
  ProfScope ps(ctx, "topk", 0.0, 5.0 * (double)n + 4.0 * (double)k * group);
  if (k <= 0 || k >= n) {
    hipLaunchKernelGGL(topk_all_kernel, dim3(1), dim3(1024), 0, ctx->stream, score, n, k >= n ? 1 : 0, group, mask, idx, tau);
  } else if (n <= SELECT_MAX) {
    launch_topk_small(ctx, const_cast<float*>(score), n, k, group, mask, idx, tau, ScoreSource{nullptr, nullptr, 0, nullptr}, nullptr);
  } else {
    const int vec = (((uintptr_t)score & 15) == 0 && ((uintptr_t)mask & 7) == 0) ? 1 : 0;
    if (!scratch || scratch_bytes < topk_scratch_bytes(n)) {
      if (group == 1) return fail(ctx, STRP_ENOMEM, "top-k over %d scores needs %zu bytes of workspace", n, topk_scratch_bytes(n));
      hipLaunchKernelGGL(topk_lone_kernel, dim3(1), dim3(big::THREADS), 0, ctx->stream, score, (long long)n, (long long)k, vec, group, mask, idx, tau);
      STRP_HIP(ctx, hipGetLastError());
      return STRP_OK;
    }
    int blocks;
    long long chunk;
    big_plan(n, &blocks, &chunk);
    big::State* st = (big::State*)scratch;
    STRP_TRY(fill_zero(ctx, st, offsetof(big::State, clear_end)));
    const dim3 b(blocks), th(big::THREADS);
    hipLaunchKernelGGL((topk_hist_kernel<0>), b, th, 0, ctx->stream, score, (long long)n, (long long)k, chunk, vec, st);
    hipLaunchKernelGGL((topk_hist_kernel<1>), b, th, 0, ctx->stream, score, (long long)n, (long long)k, chunk, vec, st);
    hipLaunchKernelGGL(topk_count_kernel, b, th, 0, ctx->stream, score, (long long)n, chunk, vec, tau, st);
    hipLaunchKernelGGL(topk_write_kernel, b, th, 0, ctx->stream, score, (long long)n, chunk, vec, group, mask, idx, (const big::State*)st);
  }
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

}  // namespace strp
