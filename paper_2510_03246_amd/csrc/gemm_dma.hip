// Pipelined MFMA GEMM for large problems: 256x256 block tile, eight wavefronts of 128x64, operand tiles
// brought from HBM/L2 straight into LDS by the global-load-to-LDS path (no staging registers), LDS stages of
// 16 contraction steps each, the stages behind the one being multiplied in flight.
//
// Why: with staging registers only one K tile can be in flight per CU (the accumulator registers of a
// 128x64 wavefront tile leave little room for more), and one tile in flight (64 KB per CU) at ~2 us of loaded
// memory latency caps the chip at ~9 TB/s of operand traffic.  LDS has room for two to four pairs of stages.
//
// The operand layout (see gemm_mfma.hip) makes every load one contiguous KB: a wavefront instruction
// moves the 64 chunks (16 B each) of 64 consecutive rows of one k-group, and the hardware writes lane l's
// chunk at LDS base + 16 l, which is exactly the [k-group][row][8] image the matrix-core fragments read.
//
// The loads are issued from inline assembly, so the compiler does not track them: completion is enforced
// here with explicit vmcnt waits (loads retire in order) followed by a workgroup barrier.
#include <stdlib.h>

#include "gemm_epilogue.h"

namespace strp {

namespace dma {
constexpr int ROWS = 256;          // rows of P / columns of Q per block
constexpr int PLANE_STAGE_BYTES = 2 * ROWS * 16;   // one plane of one operand in one stage (16 contraction steps = two k-groups): 8 KB
}  // namespace dma

// m0 is written here, so it is named as clobbered; the compiler treats m0 as a reserved register (it never keeps a
// value in it across statements) and warns about the listing, which is silenced for this one statement.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma_16(const void* gptr, unsigned lds_addr) {
  // m0 = LDS byte address of lane 0's chunk; lane l lands at m0 + 16 l
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_addr), "v"(gptr) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt_lgkm0() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(N) : "memory");
}

// ---------------------------------------------------------------------------------------------------------------------
// The matrix-core instruction is v_mfma_f32_16x16x32_f16: each wavefront's 128 x 64 outputs are 8 x 4 tiles of
// 16 x 16, one instruction contracts 32 steps.  Measured on this chip with random fp16 operands fed from LDS in exactly
// this wavefront shape, the 16x16x32 instruction sustains 11 % more than the 32x32x16 one (the chip is power-limited
// while the matrix cores run; the smaller accumulator tile costs less energy per flop).
// Two consecutive 16-step stages form the 32 steps of one instruction (lanes 0-31 read their operand chunks from the
// first stage of the pair, lanes 32-63 from the second), so the pipeline advances by pairs: while pair p is multiplied,
// the next one to three pairs are in flight (LDS holds two pairs of four planes, three of three, four of two), and the
// slots of pair p are refilled as soon as every wavefront has its last fragment of the pair in registers.  The Q fragments of a pair stay in registers (double
// buffered across pairs), the P fragments stream through two register sets.
// TOKENS: the accumulators are transposed (the instruction's operands exchanged), for the epilogues that move four consecutive
// columns per lane (PARTIAL, AUPD, ZUPD); the others write operand planes, whose chunks are consecutive rows.
// It is also the cheaper order for the matrix cores, which are bound by power on real data: the operand that stays the same over
// four instructions is the second one.  Chains of 8192 tokens, M x N = 2048 x 3277: right-hand sides 7780 -> 7590 us (three
// passes), 5310 -> 5200 (two); z-update of 3277 x 262144 over 2048 6230 -> 6035, a-update 8390 -> 8300.  At d = 768 the two
// are even.
template <int NPP, int NPQ, bool TOKENS>
__global__ __launch_bounds__(512, 1) void gemm_dma_kernel(const GemmP p) {
  using namespace dma;
  constexpr int NW = 8;
  constexpr int NPL = NPP + NPQ;
  constexpr int STAGE_BYTES = NPL * PLANE_STAGE_BYTES;
  constexpr int LPW = 8 * NPL / NW;
  // pairs of stages LDS holds: two with four planes (128 KB), three with three (144 KB), four with two (128 KB)
  constexpr int NP = NPL == 4 ? 2 : (NPL == 3 ? 3 : 4);
  __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * NP * STAGE_BYTES];
  __shared__ double sred[NW][2];
  __shared__ int srow[dma::ROWS];

  int tm, tn, split;
  decode_tile(p, (int)blockIdx.x, (int)gridDim.x, tm, tn, split);
  const int m0 = tm * ROWS, n0 = tn * ROWS;
  const long long k0 = (long long)split * p.kchunk;                 // a multiple of 32
  const long long k1 = (k0 + p.kchunk < p.K) ? (k0 + p.kchunk) : p.K;
  const int npairs = (int)((k1 - k0 + 31) / 32);                    // k-groups past k1 inside the last pair are zero padding
  const long long g0 = k0 >> 3;
  const long long g_last = ((k1 + 7) >> 3) - 1;

  const int tid = threadIdx.x, lane = tid & 63;
  int my_row = 0;
  if (p.oidx && tid < ROWS && m0 + tid < p.M) my_row = p.oidx[m0 + tid];
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;

  const unsigned short* gp[LPW];
  unsigned lds_off[LPW];
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int q = wave + NW * i;
    const int plane = q >> 3, g = (q >> 2) & 1, seg = q & 3;
    const bool isP = plane < NPP;
    const PlaneOp& op = isP ? p.P : p.Q;
    const int pl = isP ? plane : plane - NPP;
    const unsigned short* base = pl == 0 ? op.hi : op.lo;
    const int row0 = isP ? m0 : n0;
    int pan = (row0 >> 7) + (seg >> 1);
    pan = pan < op.npan ? pan : op.npan - 1;
    const int rr = (seg & 1) * 64 + lane;
    gp[i] = base + (((long long)pan * op.kg + g0 + g) * 128 + rr) * 8;
    lds_off[i] = (unsigned)(plane * PLANE_STAGE_BYTES + (g * ROWS + seg * 64) * 16);
  }
  // stage s = k-groups g0 + 2 s, g0 + 2 s + 1; the planes are padded to a multiple of four k-groups, so both stages of
  // the last pair exist in memory; stages past them re-read the last one (never multiplied)
  const long long last_stage = 2 * (long long)npairs - 1;
  auto issue_stage = [&](int s) {
    const long long sp = s < last_stage ? s : last_stage;
    const unsigned slot = lds_base + (unsigned)(s % (2 * NP)) * STAGE_BYTES;
#pragma unroll
    for (int i = 0; i < LPW; ++i) lds_dma_16(gp[i] + sp * 2048, slot + lds_off[i]);
  };
  (void)g_last;

  floatx4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

  // lane l reads the chunk of k-group l / 16 of the 32-deep step: groups 0, 1 in the pair's first stage, 2, 3 in its second
  const int kgl = lane >> 4;
  const int offP = (kgl >> 1) * STAGE_BYTES + ((kgl & 1) * ROWS + wm * 128 + (lane & 15)) * 16;
  const int offQ = (kgl >> 1) * STAGE_BYTES + NPP * PLANE_STAGE_BYTES + ((kgl & 1) * ROWS + wn * 64 + (lane & 15)) * 16;
  struct QF { uint4 h[4], l[4]; };
  struct PF { uint4 h, l; };
  auto read_q = [&](QF& f, int pr) {
    const unsigned char* st = smem + (pr % NP) * 2 * STAGE_BYTES;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f.h[j] = *(const uint4*)(st + offQ + j * 256);
      if (NPQ == 2) f.l[j] = *(const uint4*)(st + PLANE_STAGE_BYTES + offQ + j * 256);
    }
  };
  auto read_p = [&](PF& f, int pr, int i) {
    const unsigned char* st = smem + (pr % NP) * 2 * STAGE_BYTES;
    f.h = *(const uint4*)(st + offP + i * 256);
    if (NPP == 2) f.l = *(const uint4*)(st + PLANE_STAGE_BYTES + offP + i * 256);
  };
  auto mma = [&](uint4 a, uint4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, TOKENS ? b : a), __builtin_bit_cast(half8, TOKENS ? a : b), c, 0, 0, 0);
  };
  auto pass_hl = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
    if (NPQ == 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = mma(a.h, b.l[j], c[j]);
    }
  };
  auto pass_lh = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
    if (NPP == 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = mma(a.l, b.h[j], c[j]);
    }
  };
  auto pass_hh = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = mma(a.h, b.h[j], c[j]);
  };
  auto run_row = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
    pass_hl(c, a, b);
    pass_lh(c, a, b);
    pass_hh(c, a, b);
  };
  // One pair: bc holds the pair's Q fragments, pa its first P fragment; on return bn / pa hold those of the next pair.
  PF pa, pb;
  // Instruction order: the fragment reads of row i + 1 are issued ahead of the matrix-core instructions of row i (a
  // scheduling barrier after each pair of reads keeps the compiler from sinking them to where they are needed).
  auto pair_step = [&](int pr, const QF& bc, QF& bn) {
#define STRP_ROW(i, cur, nxt)                \
    read_p(nxt, pr, (i) + 1);                \
    __builtin_amdgcn_sched_barrier(0);       \
    run_row(acc[i], cur, bc);                \
    __builtin_amdgcn_sched_barrier(0);
    STRP_ROW(0, pa, pb)
    STRP_ROW(1, pb, pa)
    STRP_ROW(2, pa, pb)
    STRP_ROW(3, pb, pa)
    STRP_ROW(4, pa, pb)
    STRP_ROW(5, pb, pa)
    STRP_ROW(6, pa, pb)
#undef STRP_ROW
    wait_vmcnt_lgkm0<(NP - 2) * 2 * LPW>();   // the next pair has landed; this wavefront's fragment reads of this pair are complete
    __syncthreads();               // ... and so for every wavefront: the pair's slots may be overwritten
    // the last row needs nothing from LDS: its matrix-core instructions go out first and run while the refill is
    // requested and the next pair's first fragments are read
    pass_hh(acc[7], pb, bc);
    __builtin_amdgcn_sched_barrier(0);
    issue_stage(2 * (pr + NP));
    issue_stage(2 * (pr + NP) + 1);
    __builtin_amdgcn_sched_barrier(0);
    pass_hl(acc[7], pb, bc);
    __builtin_amdgcn_sched_barrier(0);
    read_q(bn, pr + 1);            // past the last pair this reads slots that are never multiplied
    read_p(pa, pr + 1, 0);
    __builtin_amdgcn_sched_barrier(0);
    pass_lh(acc[7], pb, bc);
    __builtin_amdgcn_sched_barrier(0);
  };

#pragma unroll
  for (int q = 0; q < 2 * NP; ++q) issue_stage(q);
  QF q0, q1;
  wait_vmcnt<(NP - 1) * 2 * LPW>();   // the first pair has landed
  __syncthreads();
  read_q(q0, 0);
  read_p(pa, 0, 0);
  int pr = 0;
#pragma unroll 1
  for (; pr + 1 < npairs; pr += 2) {
    pair_step(pr, q0, q1);
    pair_step(pr + 1, q1, q0);
  }
  if (pr < npairs) pair_step(pr, q0, q1);
  wait_vmcnt<0>();
  if (tid < ROWS) srow[tid] = my_row;
  __syncthreads();

  float unscale = 1.0f;
  if (p.P.maxbits) unscale /= scale_of_max(*p.P.maxbits);
  if (p.Q.maxbits) unscale /= scale_of_max(*p.Q.maxbits);
  double red0 = 0.0, red1 = 0.0;
  if constexpr (TOKENS) {
    const int m0w = m0 + wm * 128, n0w = n0 + wn * 64;
    if (p.epi == EPI_PARTIAL) token_epilogue<EPI_PARTIAL, true, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (p.epi == EPI_AUPD && p.rs_z0) token_epilogue<EPI_AUPD, true, true>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (p.epi == EPI_AUPD) token_epilogue<EPI_AUPD, true, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (!p.write_out) token_epilogue<EPI_ZUPD, false, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (p.rs_z0) token_epilogue<EPI_ZUPD, true, true>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else token_epilogue<EPI_ZUPD, true, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
  } else {
    const int mbase = m0 + wm * 128 + 8 * (lane >> 5), nbase = n0 + wn * 64 + (lane & 31);
    switch (p.epi) {
      case EPI_STORE: epilogue16<EPI_STORE>(p, acc, unscale, mbase, nbase, m0, red0, red1); break;
      case EPI_INITZ: epilogue16<EPI_INITZ>(p, acc, unscale, mbase, nbase, m0, red0, red1); break;
      default: epilogue16<EPI_RESID>(p, acc, unscale, mbase, nbase, m0, red0, red1); break;
    }
  }
  if (p.maxbits) {
    store_maxbits<NW>(p, red0, sred);
  } else if (p.red) {
    red0 = wave_sum(red0);
    red1 = wave_sum(red1);
    if (lane == 0) {
      sred[wave][0] = red0;
      sred[wave][1] = red1;
    }
    __syncthreads();
    if (tid == 0) {
      double r0 = 0.0, r1 = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        r0 += sred[w][0];
        r1 += sred[w][1];
      }
      p.red[2 * (long long)blockIdx.x + 0] = r0;
      p.red[2 * (long long)blockIdx.x + 1] = r1;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------------
// The same products in tiles of 128 x 256 by four wavefronts, two workgroups on a CU: one has matrix instructions to issue while the
// other fills its pipeline or moves the state tensors of its epilogue.  The wavefronts lie side by side, so a wavefront's 64 columns
// of Q are its own: their fragments come straight from memory into registers (the operand layout is the fragments': four runs of
// 256 bytes an instruction), a pair of stages ahead, and only P, which all four read, passes through LDS: 16 KB of fragment reads a
// wavefront and 32 steps instead of 24.  What bounds it is power, as the kernel above, on large products (A_S of 768 x 1536 x 65536 434 us,
// 1.07 PFLOP/s executed, whatever the wavefronts' priorities or a staggered start), and on smaller ones the start and epilogue of the last
// round, which are half as long.  The sums are those of the kernel above, bit for bit.
// NI: 16-row tiles of P a workgroup has, 8 (128 x 256) or, for products with few tiles, 4 (64 x 256).
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma_16s(const void* base, unsigned lane_off, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_addr), "v"(lane_off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
template <int NPP, int NPQ, bool TOKENS, int NI>
__global__ __launch_bounds__(256, 2) void gemm_half_kernel(const GemmP p) {
  constexpr int NW = 4, PM = 16 * NI, PN = 256;
  constexpr int PAIR = 8192;                       // bytes of one plane of a panel of 128 rows over 32 contraction steps, contiguous in memory
  constexpr int PLANE = 64 * PM;                   // the tile's rows of them, in LDS
  // pairs of stages in flight or in use: with 64 rows a pair is multiplied in half the time, and there are registers for twice as many
  constexpr int DEPTH = NI == 8 ? 2 : 4;
  constexpr int LP = NPP * NI / 4, LQ = 4 * NPQ;   // a wavefront's requests for a pair
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DEPTH][NPP * PLANE];
  __shared__ double sred[NW][2];
  __shared__ int srow[PM];

  int tm, tn, split;
  decode_tile(p, (int)blockIdx.x, (int)gridDim.x, tm, tn, split);
  const int m0 = tm * PM, n0 = tn * PN;
  const long long k0 = (long long)split * p.kchunk;                 // a multiple of 32
  const long long k1 = (k0 + p.kchunk < p.K) ? (k0 + p.kchunk) : p.K;
  const int npairs = (int)((k1 - k0 + 31) / 32);                    // k-groups past k1 inside the last pair are zero padding
  const long long g0 = k0 >> 3;

  const int tid = threadIdx.x, lane = tid & 63;
  int my_row = 0;
  if (p.oidx && tid < PM && m0 + tid < p.M) my_row = p.oidx[m0 + tid];
  const int wn = __builtin_amdgcn_readfirstlane(tid >> 6);

  // P: this wavefront moves its share of each plane of a pair, a KB at a time: 64 rows of a k-group
  const char* pp[NPP];
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)&smem[0][0];
#pragma unroll
  for (int pl = 0; pl < NPP; ++pl)
    pp[pl] = (const char*)((pl ? p.P.lo : p.P.hi) + ((long long)(m0 >> 7) * p.P.kg + g0) * 1024) + wn * 2048 + (m0 & 127) * 16;
  auto issue_p = [&](int pr) {
    const long long o = (long long)(pr < npairs ? pr : npairs - 1) * PAIR;
#pragma unroll
    for (int pl = 0; pl < NPP; ++pl)
#pragma unroll
      for (int i = 0; i < NI / 4; ++i)
        lds_dma_16s(pp[pl] + o + i * 1024, lane * 16, lds_base + (unsigned)((pr & (DEPTH - 1)) * NPP + pl) * PLANE + wn * (16 * PM) + i * 1024);
  };
  // lane l has the chunk of k-group l / 16 and row l % 16 of a fragment
  const unsigned frag = (unsigned)((lane >> 4) * 128 + (lane & 15)) * 16, frag_p = (unsigned)((lane >> 4) * PM + (lane & 15)) * 16;
  const char* qp[NPQ];
  {
    const int n = n0 + wn * 64;
    int pan = n >> 7;
    pan = pan < p.Q.npan ? pan : p.Q.npan - 1;
#pragma unroll
    for (int pl = 0; pl < NPQ; ++pl) qp[pl] = (const char*)((pl ? p.Q.lo : p.Q.hi) + ((long long)pan * p.Q.kg + g0) * 1024) + (n & 127) * 16;
  }
  typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));
  struct QF { uintx4 h[4], l[4]; };
  struct PF { uintx4 h, l; };
  auto load_q = [&](QF& f, int pr) {
    const long long o = (long long)(pr < npairs ? pr : npairs - 1) * PAIR;
    const char* const h = qp[0] + o;
    const char* const l = qp[NPQ - 1] + o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f.h[j] = *(const uintx4*)(h + frag + j * 256);
      if (NPQ == 2) f.l[j] = *(const uintx4*)(l + frag + j * 256);
    }
  };
  auto read_p = [&](PF& f, int pr, int i) {
    const unsigned char* st = smem[pr & (DEPTH - 1)];
    f.h = *(const uintx4*)(st + frag_p + i * 256);
    if (NPP == 2) f.l = *(const uintx4*)(st + PLANE + frag_p + i * 256);
  };

  floatx4 acc[NI][4];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  auto mma = [&](uintx4 a, uintx4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, TOKENS ? b : a), __builtin_bit_cast(half8, TOKENS ? a : b), c, 0, 0, 0);
  };
  auto pass_hl = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
    if (NPQ == 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = mma(a.h, b.l[j], c[j]);
    }
  };
  auto pass_lh = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
    if (NPP == 2) {
#pragma unroll
      for (int j = 0; j < 4; ++j) c[j] = mma(a.l, b.h[j], c[j]);
    }
  };
  auto pass_hh = [&](floatx4 (&c)[4], const PF& a, const QF& b) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = mma(a.h, b.h[j], c[j]);
  };
  PF pa, pb;
  // One pair: b holds its Q fragments, pa its first P fragment; on return pa holds that of the next pair, and b's registers are being
  // filled for the one behind it.
  // The compiler does not see that P's loads are in flight: it is made to wait for the next pair's Q fragments where everything
  // that has been asked for is waited for, since behind that it would count too few loads after them.
  auto arrived = [&](QF& f) {
    asm volatile("" : "+v"(f.h[0]), "+v"(f.h[1]), "+v"(f.h[2]), "+v"(f.h[3]));
    if (NPQ == 2) asm volatile("" : "+v"(f.l[0]), "+v"(f.l[1]), "+v"(f.l[2]), "+v"(f.l[3]));
  };
  auto pair_step = [&](int pr, QF& b, QF& bn) {
    // the fragments of a row of tiles are read ahead of the matrix-core instructions of the row before it
#pragma unroll
    for (int i = 0; i < NI - 1; ++i) {
      PF& cur = i & 1 ? pb : pa;
      read_p(i & 1 ? pa : pb, pr, i + 1);
      __builtin_amdgcn_sched_barrier(0);
      pass_hl(acc[i], cur, b);
      pass_lh(acc[i], cur, b);
      pass_hh(acc[i], cur, b);
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_vmcnt_lgkm0<(DEPTH - 2) * (LP + LQ)>();         // the next pair has landed; this wavefront's fragment reads of this pair are complete
    arrived(bn);
    __syncthreads();               // ... and so for every wavefront: the pair's slot may be overwritten
    pass_hh(acc[NI - 1], pb, b);
    __builtin_amdgcn_sched_barrier(0);
    issue_p(pr + DEPTH);
    read_p(pa, pr + 1, 0);         // past the last pair this reads a slot that is never multiplied
    __builtin_amdgcn_sched_barrier(0);
    pass_hl(acc[NI - 1], pb, b);
    pass_lh(acc[NI - 1], pb, b);
    __builtin_amdgcn_sched_barrier(0);
    load_q(b, pr + DEPTH);
    __builtin_amdgcn_sched_barrier(0);
  };

  QF q[DEPTH];
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    issue_p(d);
    load_q(q[d], d);
  }
  wait_vmcnt<(DEPTH - 1) * (LP + LQ)>();
  arrived(q[0]);
  __syncthreads();
  read_p(pa, 0, 0);
  int pr = 0;
#pragma unroll 1
  for (; pr + DEPTH <= npairs; pr += DEPTH)
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) pair_step(pr + d, q[d], q[(d + 1) % DEPTH]);
#pragma unroll
  for (int d = 0; d < DEPTH - 1; ++d)
    if (pr + d < npairs) pair_step(pr + d, q[d], q[d + 1]);
  wait_vmcnt<0>();
  if (tid < PM) srow[tid] = my_row;
  __syncthreads();

  float unscale = 1.0f;
  if (p.P.maxbits) unscale /= scale_of_max(*p.P.maxbits);
  if (p.Q.maxbits) unscale /= scale_of_max(*p.Q.maxbits);
  double red0 = 0.0, red1 = 0.0;
  if constexpr (TOKENS) {
    const int m0w = m0, n0w = n0 + wn * 64;
    if (p.epi == EPI_PARTIAL) token_epilogue<EPI_PARTIAL, true, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (p.epi == EPI_AUPD && p.rs_z0) token_epilogue<EPI_AUPD, true, true>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (p.epi == EPI_AUPD) token_epilogue<EPI_AUPD, true, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (!p.write_out) token_epilogue<EPI_ZUPD, false, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else if (p.rs_z0) token_epilogue<EPI_ZUPD, true, true>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
    else token_epilogue<EPI_ZUPD, true, false>(p, acc, unscale, m0w, n0w, split, srow, m0, red0, red1);
  } else {
    const int mbase = m0 + 8 * (lane >> 5), nbase = n0 + wn * 64 + (lane & 31);
    switch (p.epi) {
      case EPI_STORE: epilogue16<EPI_STORE>(p, acc, unscale, mbase, nbase, m0, red0, red1); break;
      case EPI_INITZ: epilogue16<EPI_INITZ>(p, acc, unscale, mbase, nbase, m0, red0, red1); break;
      default: epilogue16<EPI_RESID>(p, acc, unscale, mbase, nbase, m0, red0, red1); break;
    }
  }
  if (p.maxbits) {
    store_maxbits<NW>(p, red0, sred);
  } else if (p.red) {
    red0 = wave_sum(red0);
    red1 = wave_sum(red1);
    if (lane == 0) {
      sred[wn][0] = red0;
      sred[wn][1] = red1;
    }
    __syncthreads();
    if (tid == 0) {
      double r0 = 0.0, r1 = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        r0 += sred[w][0];
        r1 += sred[w][1];
      }
      p.red[2 * (long long)blockIdx.x + 0] = r0;
      p.red[2 * (long long)blockIdx.x + 1] = r1;
    }
  }
}

template <int NPP, int NPQ>
static void launch_dma(strp_ctx* ctx, const GemmP& p) {
  if (p.wt == 3 || p.wt == 5) {
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(gemm_grid_blocks(p)), dim3(256), 0, ctx->stream, p); };
    const bool tokens = p.epi == EPI_PARTIAL || p.epi == EPI_AUPD || p.epi == EPI_ZUPD;
    if (p.wt == 3) tokens ? go(gemm_half_kernel<NPP, NPQ, true, 8>) : go(gemm_half_kernel<NPP, NPQ, false, 8>);
    else tokens ? go(gemm_half_kernel<NPP, NPQ, true, 4>) : go(gemm_half_kernel<NPP, NPQ, false, 4>);
    return;
  }
  const dim3 grid(gemm_grid_blocks(p)), block(512);
  if (p.epi == EPI_PARTIAL || p.epi == EPI_AUPD || p.epi == EPI_ZUPD) hipLaunchKernelGGL((gemm_dma_kernel<NPP, NPQ, true>), grid, block, 0, ctx->stream, p);
  else hipLaunchKernelGGL((gemm_dma_kernel<NPP, NPQ, false>), grid, block, 0, ctx->stream, p);
}
void launch_gemm_dma(strp_ctx* ctx, const GemmP& p, int npp, int npq) {
  switch (npp * 10 + npq) {
    case 11: launch_dma<1, 1>(ctx, p); break;
    case 12: launch_dma<1, 2>(ctx, p); break;
    case 21: launch_dma<2, 1>(ctx, p); break;
    default: launch_dma<2, 2>(ctx, p); break;
  }
}

}  // namespace strp
