// MFMA GEMM family for gfx950 on 16-bit operand planes: v_mfma_f32_32x32x16_f16 matrix-core instructions,
// fp32 accumulation; LDS-staged tiles with 2x2 wavefronts per block, and small products straight from memory.
//
// fp32 quantities (ADMM auxiliaries, refitted weights, targets) are kept for the matrix cores as TWO fp16
// planes, x*scale = hi + lo with hi = fp16(x*scale), lo = fp16(x*scale - hi) (fp16 subnormals are honoured by
// the f16 MFMA, so lo is exact to 2^-25 absolute).  A product of two split operands runs the three leading
// passes hi*hi + hi*lo + lo*hi into ONE fp32 accumulator (the dropped lo*lo term is ~2^-22 relative); a bf16
// input is exact in a single fp16 plane.  Planes are written once by the split kernels (split_planes.hip) or by
// a producing epilogue instead of being re-converted by every tile that reads them.
//
// Every operand uses one memory layout, chosen for the matrix cores and for HBM:
//   element (k, r)   k = contraction index, r = output row (P operand) or output column (Q operand)
//   offset(k, r) = (((r / 128) * KG + k / 8) * 128 + r % 128) * 8 + k % 8,   KG = ceil(K / 8), up to a multiple of four
// i.e. panels of 128 rows; inside a panel the 8 k-values a matrix-core lane needs are one 16-byte chunk, the 128
// chunks of a k-group are contiguous (a wavefront load is 1 KB contiguous, an LDS image needs no transpose and
// no padding), and walking k walks memory sequentially (one stream per panel, TLB- and DRAM-page-friendly).
// The kernel computes C[m, n] = sum_k P(k, m) Q(k, n); token-contraction products (Gram matrices, refit
// right-hand sides) use split-K partials, token-parallel products use the fused epilogues.
#include <stdlib.h>

#include "gemm_epilogue.h"
#include "splitk_reduce.h"

namespace strp {

// The 128x128 tile: one panel per operand, K tile 64, two blocks per CU.  (256x256 ones: gemm_dma.hip.)
constexpr int ROWS = 128;               // rows of P and columns of Q per block
constexpr int BK = 64;
constexpr int NCH = ROWS * BK / 8 / 256; // 16-byte chunks per thread per plane per K tile
constexpr int GSTEP = 256 / ROWS;       // k-groups covered by one pass of the block's threads
constexpr int WT = 2;                   // 32x32 MFMA tiles per wavefront per dimension

// Operand tile loader: thread t owns row t % 128 of the panel and k-groups t / 128 + GSTEP * i.
// Loads are unconditional (panel clamped to the last one, k-groups past the end read group 0 and are zeroed
// by select) and pointers advance by one K tile per iteration.
template <int NP>
struct PlaneLoader {
  const unsigned short* bp[NP];     // chunk (group of the next tile + g0, this thread's row)
  const unsigned short* safe[NP];   // same row, group 0
  uint4 r[NP][NCH];
  long long gnext;                  // absolute k-group of bp
  int lds_off;                      // element offset of chunk (g0, row) inside an LDS plane tile

  __device__ __forceinline__ void init(const PlaneOp& op, int row0, long long k0) {
    const int t = threadIdx.x;
    const int rr = t & 127;
    const int g0 = t >> 7;
    int pan = row0 >> 7;
    pan = pan < op.npan ? pan : op.npan - 1;
    gnext = (k0 >> 3) + g0;
    const long long base = ((long long)pan * op.kg * 128 + rr) * 8;
    bp[0] = op.hi + base + gnext * 1024;
    safe[0] = op.hi + base;
    if (NP == 2) {
      bp[NP - 1] = op.lo + base + gnext * 1024;
      safe[NP - 1] = op.lo + base;
    }
    lds_off = (g0 * ROWS + rr) * 8;
  }
  __device__ __forceinline__ void load(long long g_end) {
#pragma unroll
    for (int pl = 0; pl < NP; ++pl) {
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const bool valid = gnext + GSTEP * i < g_end;
        const unsigned short* src = valid ? bp[pl] + (long long)(GSTEP * i) * 1024 : safe[pl];
        const uint4 v = *(const uint4*)src;
        r[pl][i] = valid ? v : make_uint4(0, 0, 0, 0);
      }
      bp[pl] += (BK / 8) * 1024;
    }
    gnext += BK / 8;
  }
  __device__ __forceinline__ void store(unsigned short (*s)[ROWS * BK]) const {
#pragma unroll
    for (int pl = 0; pl < NP; ++pl)
#pragma unroll
      for (int i = 0; i < NCH; ++i) *(uint4*)(&s[pl][lds_off + GSTEP * i * ROWS * 8]) = r[pl][i];
  }
};

__device__ __forceinline__ floatx16 mma(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

template <int NPP, int NPQ>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(const GemmP p) {
  constexpr int KS = BK / 16;
  __shared__ __attribute__((aligned(16))) unsigned short sP[NPP][ROWS * BK];
  __shared__ __attribute__((aligned(16))) unsigned short sQ[NPQ][ROWS * BK];
  __shared__ double sred[4][2];
  __shared__ int srow[ROWS];   // gathered state row of each output row (AUPD / ZUPD)

  // ---- which tile, which K range ---------------------------------------------------------
  int tm, tn, split;
  decode_tile(p, (int)blockIdx.x, (int)gridDim.x, tm, tn, split);
  const int m0 = tm * ROWS, n0 = tn * ROWS;
  const long long k0 = (long long)split * p.kchunk;
  const long long k1 = (k0 + p.kchunk < p.K) ? (k0 + p.kchunk) : p.K;
  const long long g_end = (k1 + 7) >> 3;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < ROWS) srow[tid] = (p.oidx && m0 + tid < p.M) ? p.oidx[m0 + tid] : 0;   // visible after the loop's barriers
  const int wm = wave >> 1, wn = wave & 1;
  constexpr int WROWS = 32 * WT;   // rows (and columns) of the output owned by one wavefront

  PlaneLoader<NPP> lp;
  lp.init(p.P, m0, k0);
  PlaneLoader<NPQ> lq;
  lq.init(p.Q, n0, k0);

  floatx16 acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; ++i)
#pragma unroll
    for (int j = 0; j < WT; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  // fragment addresses of this lane inside an LDS tile [k-group][row][8]: lanes 0-31 take the even group of a
  // 16-deep step, lanes 32-63 the odd one; 32 consecutive rows are 512 contiguous bytes (no bank conflicts)
  const int offP = ((lane >> 5) * ROWS + wm * WROWS + (lane & 31)) * 8;
  const int offQ = ((lane >> 5) * ROWS + wn * WROWS + (lane & 31)) * 8;
  struct Frags { uint4 ph[WT], pl[WT], qh[WT], ql[WT]; };
  auto read_frags = [&](Frags& f, int ks) {
#pragma unroll
    for (int i = 0; i < WT; ++i) {
      const int off = offP + (2 * ks * ROWS + i * 32) * 8;
      f.ph[i] = *(const uint4*)(&sP[0][off]);
      if (NPP == 2) f.pl[i] = *(const uint4*)(&sP[NPP - 1][off]);
    }
#pragma unroll
    for (int j = 0; j < WT; ++j) {
      const int off = offQ + (2 * ks * ROWS + j * 32) * 8;
      f.qh[j] = *(const uint4*)(&sQ[0][off]);
      if (NPQ == 2) f.ql[j] = *(const uint4*)(&sQ[NPQ - 1][off]);
    }
  };
  auto run_mfma = [&](const Frags& f) {
    if (NPQ == 2) {
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = mma(f.ph[i], f.ql[j], acc[i][j]);
    }
    if (NPP == 2) {
#pragma unroll
      for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = mma(f.pl[i], f.qh[j], acc[i][j]);
    }
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
      for (int j = 0; j < WT; ++j) acc[i][j] = mma(f.ph[i], f.qh[j], acc[i][j]);
  };

  if (k0 < k1) {
    lp.load(g_end);
    lq.load(g_end);
  }
  for (long long k = k0; k < k1; k += BK) {
    lp.store(sP);
    lq.store(sQ);
    __syncthreads();
    if (k + BK < k1) {  // next tile's global loads fly during the matrix work
      lp.load(g_end);
      lq.load(g_end);
    }
    // software pipeline over the 16-deep steps: fragments of step ks+1 are read while step ks multiplies
    Frags f[2];
    read_frags(f[0], 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      __builtin_amdgcn_sched_barrier(0);
      if (ks + 1 < KS) read_frags(f[(ks + 1) & 1], ks + 1);
      __builtin_amdgcn_sched_barrier(0);
      run_mfma(f[ks & 1]);
    }
    __syncthreads();
  }

  // ---- epilogue (one specialised, fully unrolled body per epilogue kind) -------------------------
  float unscale = 1.0f;
  if (p.P.maxbits) unscale /= scale_of_max(*p.P.maxbits);
  if (p.Q.maxbits) unscale /= scale_of_max(*p.Q.maxbits);
  double red0 = 0.0, red1 = 0.0;
  const int mbase = m0 + wm * WROWS + 4 * (lane >> 5), nbase = n0 + wn * WROWS + (lane & 31);
  switch (p.epi) {
    case EPI_PARTIAL: epilogue<EPI_PARTIAL, WT, WT>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_STORE: epilogue<EPI_STORE, WT, WT>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_INITZ: epilogue<EPI_INITZ, WT, WT>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_RESID: epilogue<EPI_RESID, WT, WT>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_AUPD: epilogue<EPI_AUPD, WT, WT>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    default: epilogue<EPI_ZUPD, WT, WT>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
  }
  if (p.maxbits) {
    store_maxbits<4>(p, red0, sred);
  } else if (p.red) {
    red0 = wave_sum(red0);
    red1 = wave_sum(red1);
    if (lane == 0) {
      sred[wave][0] = red0;
      sred[wave][1] = red1;
    }
    __syncthreads();
    if (tid == 0) {
      p.red[2 * (long long)blockIdx.x + 0] = sred[0][0] + sred[1][0] + sred[2][0] + sred[3][0];
      p.red[2 * (long long)blockIdx.x + 1] = sred[0][1] + sred[1][1] + sred[2][1] + sred[3][1];
    }
  }
}

// The same products where 128x128 tiles leave the chip idle and a launch is the time of one workgroup: each tile is cut into
// 64x64 blocks (subM x subN of them), one 32x64 tile per wavefront.  The fragments come straight from memory -- the operand
// layout is that of the fragments, 32 consecutive rows are 512 contiguous bytes -- with four contraction steps in flight, no LDS
// image and no barrier; every element is summed in the order of the kernel above.
// A symmetric product in a single split, straight to what a factorisation takes next: fp64 with the ridge on its diagonal, both triangles, and the
// zeros of rows 0 .. 63 (reduce_to_system).
__device__ __forceinline__ void system_epilogue(const GemmP& p, const floatx16 (&acc)[2], float unscale, int mbase, int nbase) {
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = mbase + tile_rowoff<0>(e >> 2) + (e & 3), n = nbase + 32 * j;
      const double v = 0.0 + (double)(acc[j][e] * unscale);
      if (m >= p.M || n > m) continue;
      p.sys[(long long)m * p.ldo + n] = m == n ? v + p.ridge : v;
      if (n < m) p.sys[(long long)n * p.ldo + m] = n < NB && m >= NB ? 0.0 : v;
    }
}
// ASK: an operand may have one plane only (its lo is then read from hi and not multiplied)
template <int NPP, int NPQ, bool ASK>
__device__ __forceinline__ void gemm_small_block(const GemmP& p, int block, int blocks) {
  constexpr int AHEAD = 4;
  __shared__ double sred[2][2];
  __shared__ int srow[64];
  int tm, tn, split;
  const int sub = p.subM * p.subN, b = block / sub, within = block - b * sub;
  decode_tile(p, b, blocks / sub, tm, tn, split);
  const int m0 = tm * 128 + within / p.subN * 64, n0 = tn * 128 + within % p.subN * 64;
  if (m0 >= p.M || n0 >= p.N || (p.triangle && n0 > m0)) {      // nothing to compute
    if (p.red && !p.maxbits && threadIdx.x < 2) p.red[2 * (long long)block + threadIdx.x] = 0.0;
    return;
  }
  const long long k0 = (long long)split * p.kchunk;
  const long long k1 = (k0 + p.kchunk < p.K) ? (k0 + p.kchunk) : p.K;
  const int steps = (int)((k1 - k0 + 15) >> 4);        // k-groups past k1 inside the last step are zero padding
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < 64) srow[tid] = (p.oidx && m0 + tid < p.M) ? p.oidx[m0 + tid] : 0;

  // rows past M and columns past N lie in the operands' padding to whole panels
  const long long g = (k0 >> 3) + (lane >> 5);
  const int mr = m0 + 32 * wave + (lane & 31), nr = n0 + (lane & 31);
  const long long offp = (((long long)(mr >> 7) * p.P.kg + g) * 128 + (mr & 127)) * 8;
  long long offq[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) offq[j] = (((long long)((nr + 32 * j) >> 7) * p.Q.kg + g) * 128 + ((nr + 32 * j) & 127)) * 8;
  struct Frags { uint4 ph, pl, qh[2], ql[2]; } f[AHEAD];
  const bool plo = !ASK || p.P.lo, qlo = !ASK || p.Q.lo;
  const unsigned short* const p_lo = plo ? p.P.lo : p.P.hi;
  const unsigned short* const q_lo = qlo ? p.Q.lo : p.Q.hi;
  auto load = [&](Frags& x, int s) {
    const long long o = (long long)(s < steps ? s : steps - 1) * 2048;
    x.ph = *(const uint4*)(p.P.hi + offp + o);
    if (NPP == 2) x.pl = *(const uint4*)(p_lo + offp + o);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      x.qh[j] = *(const uint4*)(p.Q.hi + offq[j] + o);
      if (NPQ == 2) x.ql[j] = *(const uint4*)(q_lo + offq[j] + o);
    }
  };
  floatx16 acc[1][2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][j][e] = 0.0f;
  auto multiply = [&](const Frags& x) {
    if (NPQ == 2 && qlo) {
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[0][j] = mma(x.ph, x.ql[j], acc[0][j]);
    }
    if (NPP == 2 && plo) {
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[0][j] = mma(x.pl, x.qh[j], acc[0][j]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[0][j] = mma(x.ph, x.qh[j], acc[0][j]);
  };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) load(f[u], u);
  int s = 0;
  for (; s + AHEAD <= steps; s += AHEAD)
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      multiply(f[u]);
      load(f[u], s + AHEAD + u);
    }
#pragma unroll
  for (int u = 0; u < AHEAD - 1; ++u)
    if (s + u < steps) multiply(f[u]);
  __syncthreads();

  float unscale = 1.0f;
  if (p.P.maxbits) unscale /= scale_of_max(*p.P.maxbits);
  if (p.Q.maxbits) unscale /= scale_of_max(*p.Q.maxbits);
  double red0 = 0.0, red1 = 0.0;
  const int mbase = m0 + 32 * wave + 4 * (lane >> 5), nbase = n0 + (lane & 31);
  switch (p.epi) {
    case EPI_PARTIAL: epilogue<EPI_PARTIAL, 1, 2>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_STORE: epilogue<EPI_STORE, 1, 2>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_INITZ: epilogue<EPI_INITZ, 1, 2>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_RESID: epilogue<EPI_RESID, 1, 2>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_AUPD: epilogue<EPI_AUPD, 1, 2>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
    case EPI_SYSTEM: system_epilogue(p, acc[0], unscale, mbase, nbase); break;
    default: epilogue<EPI_ZUPD, 1, 2>(p, acc, unscale, mbase, nbase, split, srow, m0, red0, red1); break;
  }
  if (p.maxbits) {
    store_maxbits<2>(p, red0, sred);
  } else if (p.red) {
    red0 = wave_sum(red0);
    red1 = wave_sum(red1);
    if (lane == 0) {
      sred[wave][0] = red0;
      sred[wave][1] = red1;
    }
    __syncthreads();
    if (tid == 0) {
      p.red[2 * (long long)block + 0] = sred[0][0] + sred[1][0];
      p.red[2 * (long long)block + 1] = sred[0][1] + sred[1][1];
    }
  }
}

template <int NPP, int NPQ>
__global__ __launch_bounds__(128) void gemm_kernel(const GemmP p) { gemm_small_block<NPP, NPQ, false>(p, blockIdx.x, gridDim.x); }

// up to three independent products, one behind the other in the grid: end[i] workgroups up to and with product i.  One kernel
// for all combinations of planes: an operand of one plane is loaded twice, the second time for nothing, which a small product has
// room for (all operands of one plane, us a step with a launch for either product of the fc2 refit / one for both: 64 x 128 over
// 512 tokens 208 / 201, 256 x 512 over 2048 389 / 382, 512 x 1000 over 1024 600 / 597; with two planes 213 / 206, 407 / 399, 629 / 622).
struct GemmGroup {
  GemmP p[3];
  int end[3];
};
__global__ __launch_bounds__(128) void gemm_group_kernel(const GemmGroup g) {
  const int b = (int)blockIdx.x, i = b >= g.end[1] ? 2 : b >= g.end[0] ? 1 : 0, start = i ? g.end[i - 1] : 0;
  gemm_small_block<2, 2, true>(g.p[i], b - start, g.end[i] - start);
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
// Fewer 128x128 workgroups than the chip runs at a time (512) are cut into 64x64 ones, up to half of that.  us of the product
// alone, 128x128 / 64x64 (4 us of either are the timing): Gram matrices 128 x 512 12.4 / 7.9, 256 x 4000 13.2 / 8.7, 400 x 4000
// (150 workgroups) 15.8 / 11.8; 1536 x 768 over 768 (72) 31 / 21.6, 768 x 768 (36) 27.6 / 14.6, 2048 x 2048 over 2048 (256)
// 67 / 67.
constexpr int SMALL_BLOCKS = 256;
void gemm_small_tiles(GemmP& p) {
  if (p.wt != 2 || p.ntiles * p.splits > SMALL_BLOCKS) return;
  p.wt = 1;
  p.subM = p.M > 64 ? 2 : 1;
  p.subN = p.N > 64 ? 2 : 1;
}

// Products of the state's kept rows in 128x256 tiles, two workgroups on a CU (gemm_half_kernel).  us, the tile before / this one (E, A_S, Z1):
// 768 over 1536 units and 65536 tokens 373 / 371, 446 / 434, 361 / 337;  2048, 3277, 65536 1904 / 1855, 2107 / 2104, 1558 / 1454;  1000, 1013,
// 30011, fp32 X 183 / 180, 208 / 200, 207 / 198.  More where 256-row tiles pad (264, 270, 66000, fp32 X 119 / 79, 142 / 93, 144 / 100) or
// fill their last round badly (1600, 2500, 8000: A_S 222 / 179, Z1 172 / 142) and where fewer than 192 of them left the product
// to 128x128 ones (1536, 2304, 4096: A_S 139 / 112, Z1 107 / 77).  Not where 256x256 tiles fill one round and both operands
// have two planes, since half a round of each is then the same work with a longer start (768, 1536, 16384: E 119 / 127; 2048, 3277, 4096: A_S 144 / 150;
// with one plane of X 63 / 55 and 109 / 106 for Z1), nor for fewer workgroups than CUs (512, 700, 8192: A_S 192 of them 35 / 34, E 33 / 42), nor
// where 128 rows or six pairs of stages are all there is (130 kept of 128 over 70000: 37 / 41, 43 / 43, 46 / 48).  The initialisation's products,
// which write three tensors or run over all units, are no faster (2048 x 6824 x 16384: 657 / 746, 622 / 664).
// Nor for E and A_S of two planes each from sixteen rounds of 256x256 tiles and contractions of 4096 on, where those pad by no more than a
// thirty-second.  Power bounds either tile there, but the 64 workgroups of an XCD drift apart over a long contraction and fetch their panels again: A_S of
// 4096 x 4915 x 262144 79 GB where the 32 of the larger tiles fetch 39 to 42, at 1.66 and 1.76 GHz.  ms of a step, 128x256 / 256x256 tiles for both:  7168, 8602, 65536
// 157.4 / 155.5 (A_S 18.11 / 17.64, E 26.23 / 25.46);  5120, 4608, 131072 91.7 / 91.4;  no more than two runs differ  4096, 4915, 262144 148.2 / 148.1, 131072 79.96 /
// 80.01, 65536 46.74 / 46.63;  below both lines  4096, 4100, 24000 20.06 / 20.20;  2048, 3277, 262144 52.30 / 52.38;  2560, 3072, 200000 46.56 / 46.59.  Z1 keeps
// this tile: 87.09 / 87.38 with it changed as well (4096, 4915, 131072, fp32 X), and 15.7 / 16.7 of its own with one plane of X (4096, 4915, 262144).
static bool half_tiles_pay(const GemmP& p, long long n4) {
  if (p.epi != EPI_RESID && p.epi != EPI_AUPD && p.epi != EPI_ZUPD) return false;
  if (p.M <= 128 || p.K < 192 || (long long)((p.M + 127) / 128) * ((p.N + 255) / 256) < 256) return false;
  if (!p.P.lo || !p.Q.lo) return true;
  const int rows3 = (p.M + 127) / 128, rows4 = (p.M + 255) / 256 * 2;      // of 128, padded
  if (p.epi != EPI_ZUPD && gemm_tile256_ok(p) && p.K >= 4096 && n4 >= 4096 && 32 * rows4 <= 33 * rows3) return false;
  return n4 < 192 || n4 > 256;
}

// Products that 256x256 and 128x256 tiles leave to 128x128 ones and to 64x64 blocks, in 64x256 tiles (gemm_half_kernel too, four pairs of stages in
// flight where the 128x128 kernel has one).  us, 128x128 (or 64x64, marked *) / this tile:  448 over 400 units and 9000 tokens A_S 30.4 / 21.5, Z1 27.9 / 21.3;  896,
// 400, 9000 49 / 30, 41 / 28;  1024, 1536, 4096 57 / 49, 45 / 36, E* 97 / 72;  72, 40, 150000 (fp32, GAIN) 50 / 36, 55 / 46, E 43 / 44;  1536,
// 2000, 2048 59 / 44, 47 / 37, E* 107 / 79, Y* 178 / 120;  440, 1440 units, 9000 Y 53 / 44.  The blocks of 64x64 read their operands again for every 64
// rows and columns, which costs nothing while a launch is the time of one of them: the line is at 160 thousand tiles of 128x128 times steps (768, 1200,
// 4096, 230 thousand, E 47 / 36;  600, 800, 5000, 160, 47 / 34;  896, 400, 4096, 115, A_S 23 / 26;  512, 640, 4000, 82, 20.6 / 21.2).  E and Y, whose
// epilogues write planes, gain from long contractions only, and not where 128x128 tiles fill their two places a CU (256, 512, 30000 E 40 / 48, Y 52 / 66;  96, 150,
// 40000 E 22.7 / 25.0).
static bool quarter_tiles_pay(const GemmP& p) {
  if (p.N < 256 || (p.epi != EPI_AUPD && p.epi != EPI_ZUPD && p.epi != EPI_RESID && p.epi != EPI_STORE)) return false;
  const long long n2 = (long long)((p.M + 127) / 128) * ((p.N + 127) / 128);
  if (n2 <= SMALL_BLOCKS) return (double)n2 * (double)p.K >= 1.6e5;
  return p.epi == EPI_AUPD || p.epi == EPI_ZUPD || p.K >= 1000 || (n2 <= 384 && p.K >= 500);
}

void gemm_plan_tiles(GemmP& p, int want_splits, int wt) {
  p.subM = p.subN = 1;
  if (wt) {
    p.wt = wt;
  } else {
    // 256x256 tiles with the LDS-DMA pipeline when they still give most CUs a block
    const long long n4 = (long long)((p.M + 255) / 256) * ((p.N + 255) / 256);
    p.wt = gemm_tile256_ok(p) && n4 >= 192 ? 4 : 2;
    if (half_tiles_pay(p, n4)) p.wt = 3;
    else if (p.wt == 2 && quarter_tiles_pay(p)) p.wt = 5;
  }
  const int RM = p.wt == 3 ? 128 : p.wt == 5 ? 64 : 64 * p.wt, RN = p.wt == 3 || p.wt == 5 ? 256 : 64 * p.wt, BK = p.wt == 2 ? 64 : 32;
  p.tilesM = (p.M + RM - 1) / RM;
  p.tilesN = (p.N + RN - 1) / RN;
  p.ntiles = p.triangle ? p.tilesM * (p.tilesM + 1) / 2 : p.tilesM * p.tilesN;
  if (p.triangle) {
    p.gridM = (p.tilesM + 1) / 2;
    p.gridN = 2 * (p.tilesM / 2) + 1;
  } else {
    p.gridM = p.tilesM;
    p.gridN = p.tilesN;
  }
  {
    // tile group: 32 tiles, shaped to the grid
    int gm = p.wt == 3 || p.wt == 5 ? 8 : 4;
    while (gm > 1 && gm > p.gridM) gm >>= 1;
    int gn = (p.wt == 3 || p.wt == 5 ? 64 : 32) / gm;
    while (gn > 1 && gn / 2 >= p.gridN) { gn >>= 1; if (gm * 2 <= p.gridM) gm <<= 1; }
    p.gm = gm;
    p.gn = gn;
  }
  if (want_splits <= 1) {
    p.splits = 1;
    p.kchunk = ((p.K + BK - 1) / BK) * BK;
  } else {
    long long chunk = (p.K + want_splits - 1) / want_splits;
    chunk = ((chunk + BK - 1) / BK) * BK;
    p.kchunk = chunk;
    p.splits = (int)((p.K + chunk - 1) / chunk);
  }
  if (!wt) gemm_small_tiles(p);
}

int gemm_grid_blocks(const GemmP& p) { return p.gridM * p.gridN * p.splits * (p.wt == 1 ? p.subM * p.subN : 1); }

void launch_gemm_dma(strp_ctx* ctx, const GemmP& p, int npp, int npq);   // gemm_dma.hip

template <int NPP, int NPQ>
static void launch_one(strp_ctx* ctx, const GemmP& p) {
  if (p.wt >= 3)
    launch_gemm_dma(ctx, p, NPP, NPQ);
  else if (p.wt == 1)
    hipLaunchKernelGGL((gemm_kernel<NPP, NPQ>), dim3(gemm_grid_blocks(p)), dim3(128), 0, ctx->stream, p);
  else
    hipLaunchKernelGGL((gemm_tile_kernel<NPP, NPQ>), dim3(gemm_grid_blocks(p)), dim3(256), 0, ctx->stream, p);
}

static strp_status check_gemm(strp_ctx* ctx, const GemmP& p) {
  if (p.M <= 0 || p.N <= 0 || p.K <= 0) return fail(ctx, STRP_EINVAL, "gemm: empty shape");
  if (p.ntiles <= 0 || p.splits <= 0 || p.wt < 1 || p.wt > 5) return fail(ctx, STRP_EINVAL, "gemm: tiles not planned");
  if (!p.P.hi || !p.Q.hi) return fail(ctx, STRP_EINVAL, "gemm: null operand plane");
  if (p.P.kg * 8 < p.K || p.Q.kg * 8 < p.K || (p.P.kg & 3) || (p.Q.kg & 3))
    return fail(ctx, STRP_EINVAL, "gemm: operand planes shorter than K or a group count that is not a multiple of four");
  if ((long long)p.P.npan * 128 < p.M || (long long)p.Q.npan * 128 < p.N) return fail(ctx, STRP_EINVAL, "gemm: operand planes narrower than the output");
  if (p.k8_hi && p.k8_kg != plane_kg(p.M)) return fail(ctx, STRP_EINVAL, "gemm: planes of another height than the output");
  if (p.epi == EPI_SYSTEM && (p.wt != 1 || !p.triangle)) return fail(ctx, STRP_EINVAL, "gemm: a system comes of a small symmetric product");
  if (p.epi != EPI_PARTIAL && p.splits != 1) return fail(ctx, STRP_EINVAL, "gemm: fused epilogues do not split K");
  return STRP_OK;
}

// algorithmic operations and bytes of a product: operand planes once, outputs (and what an epilogue reads beside them) once
struct GemmWork { double flops, bytes; };
static GemmWork gemm_work(const GemmP& p) {
  const int npp = p.P.lo ? 2 : 1, npq = p.Q.lo ? 2 : 1;
  const double mn = p.triangle ? 0.5 * (double)p.M * ((double)p.M + 1.0) : (double)p.M * (double)p.N;
  static const double out_words[] = {1.0, 1.0, 3.0, 2.0, 2.0, 2.0, 4.0};
  double obytes = 4.0 * out_words[p.epi] * (double)p.M * (double)p.N * (p.epi == EPI_PARTIAL ? (double)p.splits : 1.0);
  if (p.epi == EPI_RESID) obytes *= 0.5;
  if (p.k8_hi) obytes += (p.k8_lo ? 4.0 : 2.0) * (double)p.M * (double)p.N;
  const double ibytes = p.triangle ? 2.0 * npp * (double)p.M * (double)p.K
                                   : 2.0 * npp * (double)p.M * (double)p.K + 2.0 * npq * (double)p.N * (double)p.K;
  return {2.0 * mn * (double)p.K, ibytes + obytes};
}

strp_status launch_gemm(strp_ctx* ctx, GemmP& p) {
  STRP_TRY(check_gemm(ctx, p));
  const int npp = p.P.lo ? 2 : 1, npq = p.Q.lo ? 2 : 1;
  static const char* const epi_names[] = {"partial", "store", "initz", "resid", "aupd", "zupd", "system"};
  static char names[3][3][7][40];
  char* name = names[npp][npq][p.epi];
  if (!name[0]) snprintf(name, 40, "gemm_h%dx%d_%s", npp, npq, epi_names[p.epi]);
  const GemmWork work = gemm_work(p);
  ProfScope ps(ctx, name, work.flops, work.bytes);
  switch (npp * 10 + npq) {
    case 11: launch_one<1, 1>(ctx, p); break;
    case 12: launch_one<1, 2>(ctx, p); break;
    case 21: launch_one<2, 1>(ctx, p); break;
    default: launch_one<2, 2>(ctx, p); break;
  }
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// Up to three products of which none reads what another writes: in one launch where all are small ones, which saves launches
// (4 us each) and fills the chip better; otherwise one after the other.
bool gemm_is_small(const GemmP& p) { return p.wt == 1; }
strp_status launch_gemm_group(strp_ctx* ctx, GemmP* p, int n) {
  bool one = true;
  for (int i = 0; i < n; ++i) one = one && gemm_is_small(p[i]);
  if (!one) {
    for (int i = 0; i < n; ++i) STRP_TRY(launch_gemm(ctx, p[i]));
    return STRP_OK;
  }
  GemmGroup g;
  int blocks = 0;
  GemmWork work{0.0, 0.0};
  for (int i = 0; i < 3; ++i) {
    g.p[i] = p[i < n ? i : 0];
    if (i < n) {
      STRP_TRY(check_gemm(ctx, p[i]));
      blocks += gemm_grid_blocks(p[i]);
      const GemmWork w = gemm_work(p[i]);
      work.flops += w.flops;
      work.bytes += w.bytes;
    }
    g.end[i] = blocks;
  }
  ProfScope ps(ctx, "gemm_group", work.flops, work.bytes);
  hipLaunchKernelGGL(gemm_group_kernel, dim3(blocks), dim3(128), 0, ctx->stream, g);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---- split-K reduction -----------------------------------------------------------------------
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const ReduceP r) { splitk_reduce_block(r, blockIdx.x, blockIdx.y, gridDim.x); }
// up to three of them, end[i] workgroups up to and with reduction i
struct ReduceGroup {
  ReduceP r[3];
  int end[3];
};
__global__ __launch_bounds__(256) void splitk_reduce_group_kernel(const ReduceGroup g) {
  const int i = (int)blockIdx.x >= g.end[1] ? 2 : (int)blockIdx.x >= g.end[0] ? 1 : 0;
  const ReduceP r = g.r[i];
  const int b = (int)blockIdx.x - (i ? g.end[i - 1] : 0), nx = (r.N + REDUCE_TILE_N - 1) / REDUCE_TILE_N;
  splitk_reduce_block(r, b % nx, b / nx, nx);
}

// algorithmic bytes: the partials (of a symmetric product half of them) once, the results once
static double reduce_bytes(const ReduceP& r) {
  return (double)r.M * r.N * (4.0 * (double)r.splits * (r.triangle ? 0.5 : 1.0) + (r.outf ? 4.0 : 0.0) + (r.outd ? 8.0 : 0.0));
}
strp_status launch_splitk_reduce(strp_ctx* ctx, const ReduceP& r) {
  if (r.triangle && r.M != r.N) return fail(ctx, STRP_EINVAL, "split-K reduce: a symmetric product must be square");
  if (r.dot && !r.triangle) return fail(ctx, STRP_EINVAL, "split-K reduce: the inner product is for symmetric products");
  ProfScope ps(ctx, "splitk_reduce", 0.0, reduce_bytes(r));
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3((r.N + REDUCE_TILE_N - 1) / REDUCE_TILE_N, (r.M + REDUCE_TILE_M - 1) / REDUCE_TILE_M), dim3(256), 0, ctx->stream, r);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

strp_status launch_splitk_reduce_group(strp_ctx* ctx, const ReduceP* r, int n) {
  ReduceGroup g;
  int blocks = 0;
  double bytes = 0.0;
  for (int i = 0; i < 3; ++i) {
    g.r[i] = r[i < n ? i : 0];
    if (i < n) {
      blocks += reduce_blocks(r[i].M, r[i].N);
      bytes += reduce_bytes(r[i]);
    }
    g.end[i] = blocks;
  }
  ProfScope ps(ctx, "splitk_reduce", 0.0, bytes);
  hipLaunchKernelGGL(splitk_reduce_group_kernel, dim3(blocks), dim3(256), 0, ctx->stream, g);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

}  // namespace strp
