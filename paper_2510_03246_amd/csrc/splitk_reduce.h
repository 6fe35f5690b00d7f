// Sum of a split product's partials, in fp64: the work of one workgroup (gemm_mfma.hip, split_planes.hip).
#pragma once
#include "strp_internal.h"

namespace strp {

// One block reduces a 16 x 64 output tile (thread = column tx, rows ty + 4 i): a wavefront load is 256 contiguous bytes
// of one row of one partial.  Symmetric products: only tiles that reach the lower half are reduced; the strict lower
// part is also written transposed through LDS, so the upper half is a bit-exact mirror and the partials are read once,
// row-contiguously.  Bound by HBM where the output is large (4.7 TB/s); a small output (M = 832: 91 tiles of 64 x 64)
// leaves few workgroups, each with a serial walk over the splits, so tiles are low and four splits are in flight.
__device__ __forceinline__ void splitk_reduce_block(const ReduceP& r, int bx, int by, int nx) {
  constexpr int TN = REDUCE_TILE_N, TM = REDUCE_TILE_M, NI = TM / 4, AHEAD = 4;
  __shared__ double tile[TM][TN + 1];
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const int n0 = bx * TN, m0 = by * TM;
  const int M = r.M, N = r.N;
  if (r.triangle && n0 >= m0 + TM) {
    if (r.dot && threadIdx.x == 0) r.red[by * nx + bx] = 0.0;
    return;
  }
  const long long MN = (long long)M * N;
  const double ridge = r.ridge_dev ? *r.ridge_dev : r.ridge;
  auto put = [&](int m, int n, double s) {
    if (r.outf) {
      float* o = r.outf + (long long)m * r.ldof + n;
      *o = r.accumulate ? (float)((double)*o + s) : (float)s;
    }
    if (r.outd) r.outd[(long long)m * r.ldod + n] = m == n ? s + ridge : r.factored && m < NB && n >= NB ? 0.0 : s;
    if (r.diag && m == n) r.diag[m] = s;
  };
  const int n = n0 + tx;
  double acc[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) acc[i] = 0.0;
  {
    // rows and the column are clamped into range (results of clamped lanes are not stored), and so are the splits of the
    // last group: the loads of a group are then unconditional and all in flight together
    const int nc = n < N ? n : N - 1;
    long long ro[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int m = m0 + ty + 4 * i;
      ro[i] = (long long)(m < M ? m : M - 1) * N + nc;
    }
    for (int sp = 0; sp < r.splits; sp += AHEAD) {
      float v[AHEAD][NI];
#pragma unroll
      for (int q = 0; q < AHEAD; ++q) {
        const float* src = r.part + (long long)(sp + q < r.splits ? sp + q : r.splits - 1) * MN;
#pragma unroll
        for (int i = 0; i < NI; ++i) v[q][i] = src[ro[i]];
      }
#pragma unroll
      for (int q = 0; q < AHEAD; ++q)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[i] += sp + q < r.splits ? (double)v[q][i] : 0.0;
    }
    if (r.dot) {          // <dot, C>: the strict lower part of this tile stands for its mirror image as well
      double s = 0.0;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int m = m0 + ty + 4 * i;
        const double w = (m < M && n < N && n <= m) ? (n < m ? 2.0 : 1.0) : 0.0;
        s = __builtin_fma(w * (double)r.dot[ro[i]], acc[i], s);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
      if (tx == 0) tile[0][ty] = s;
      __syncthreads();
      if (threadIdx.x == 0) r.red[by * nx + bx] = tile[0][0] + tile[0][1] + tile[0][2] + tile[0][3];
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int m = m0 + ty + 4 * i;
    if (m < M && n < N && (!r.triangle || n <= m)) put(m, n, acc[i]);
    tile[ty + 4 * i][tx] = acc[i];
  }
  if (!r.triangle) return;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NI; ++i) {     // element (lo_m, lo_n) of the lower half, mirrored to (lo_n, lo_m)
    const int e = threadIdx.x + 256 * i;
    const int lo_m = m0 + (e & (TM - 1)), lo_n = n0 + e / TM;
    if (lo_n < lo_m && lo_m < M && lo_n < N) put(lo_n, lo_m, tile[e & (TM - 1)][e / TM]);
  }
}

}  // namespace strp
