// fp64 tiles on the matrix cores: lane layout, LDS images, and the 64 x 64 tiles that the factorisation is made of.
#pragma once
#include "strp_internal.h"

namespace strp {

typedef double doublex4 __attribute__((ext_vector_type(4)));
typedef double doublex2 __attribute__((ext_vector_type(2)));
typedef double doublex2u __attribute__((ext_vector_type(2), aligned(8)));      // two doubles anywhere: a caller's matrix may have odd rows

// MFMA lane layout: A operand lane l = A[i = l % 16][k = l / 16], B operand lane l = B[k = l / 16][j = l % 16],
// result register r of lane l = D[i = 4 r + l / 16][j = l % 16].
__device__ __forceinline__ doublex4 mma_f64(double a, double b, doublex4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Barrier of a workgroup whose wavefronts exchange data through LDS only: unlike __syncthreads it does not wait for the
// global loads and stores in flight (a store acknowledgement costs a step of the factorisation chain about 1 us).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// LDS images of an operand tile of R rows and K contraction steps:
//   KC (the source is contiguous in k):   [k / 2][R + 1][2]: a lane takes two k at once (16 bytes)
//   RC (the source is contiguous in rows): [k][R + 4]
// Eight contraction steps are two matrix-core instructions: instruction s multiplies k = 8 c + 2 (l / 16) + s, the same
// order for both operands, so a 16-byte KC read feeds both.  The odd pitches keep writes and reads free of bank conflicts.
template <int R>
__device__ __forceinline__ int kc_off(int k, int r) { return ((k >> 1) * (R + 1) + r) * 2 + (k & 1); }
template <int R>
__device__ __forceinline__ int rc_off(int k, int r) { return k * (R + 4) + r; }

// ---------------------------------------------------------------------------------------------
// 64 x 64 tiles of the factorisation chain
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ double rsqrt_f64(double d) {
  double y = __builtin_amdgcn_rsq(d);
  y = y * (1.5 - 0.5 * d * y * y);
  y = y * (1.5 - 0.5 * d * y * y);
  return y;
}

constexpr int F64_IMG = NB * (NB + 4);    // doubles of the larger image of a 64 x 64 tile
constexpr int SL = NB + 1;                // pitch of the square working tiles of the diagonal block
struct StepShared {
  double a[F64_IMG];
  double b[F64_IMG];
  double y[NB];
};

// Diagonal block: A = Lu D Lu^T (Lu unit lower) by 16-column panels, and W = Lu^-1.
//   in : S = sh.b, pitch SL, its first 16 columns (rows past a ragged edge are the identity); block(q, i, k): the other 16 x 16
//        blocks of the lower triangle in the accumulator layout, asked for when they are needed
//   out: rows of L^-1 = D^-1/2 W, as they are finished.  A pivot that is not positive counts as 1 and raises ENOTPD:
//        everything stays finite.
// The chain of 64 dependent pivots is what bounds it, so one wavefront runs it out of registers: every 16-lane row of
// the wavefront holds a copy of the panel's 16 x 16 diagonal block (d: lane = row, register = column), so pivots and
// multiplier rows are broadcast by row_newbcast operands of the updates themselves (no LDS, no barrier, no move); beside it
// lanes 16 .. 63 hold the rows below (a) and lanes 0 .. 15 the columns of an identity, which the same operation turns into the
// inverse of the diagonal block.  A wavefront alone issues a 64-bit operation every 5.5 cycles, a reciprocal every 20 and a
// store to LDS every 19 (two doubles: 27), so what it leaves to the others is what it would have to store or scale: it stores
// the unscaled columns, two at a time, and 16 reciprocals per panel: a launch of the chain (n = 1536) 14.0 -> 13.0 us.
// The three other wavefronts meanwhile form what the finished panels allow of W on the matrix cores, scale it and store it,
// so that only the last 16 rows are left when the chain ends.  16 x 16 blocks of S while it runs (i > p):
//   S(i, p): Lu(i, p) D(p)      S(p, p): W(p, p) transposed      S(p, i), i < 3: W(i, p)      y: -1 / D
constexpr int EYE = NB * SL + 16;         // behind S: 31 doubles with a 1 in the middle (rows of an identity)
__device__ __forceinline__ void put_eye(StepShared& sh, int tid) {
  if (tid < 31) sh.b[EYE + tid] = tid == 15 ? 1.0 : 0.0;
}
struct PanelRegs {
  double d[16], a[16];
  double dj, y, e;      // pivot, minus its reciprocal (in the making)
  double yt[4];         // of pivot 4 b + q: lanes 4 b .. of every 16, register q
  bool ok, all;         // the pivot is positive; all were
};
// v_rcp_f64 is good to 2^-23; y (1 + e + e^2), e = 1 - d y, leaves e^3
constexpr int PIVOT_STAGES = 4;
template <int STAGE>
__device__ __forceinline__ void pivot_stage(PanelRegs& g) {
  if constexpr (STAGE == 0) g.y = __builtin_amdgcn_rcp(g.dj);
  if constexpr (STAGE == 1) g.e = __builtin_fma(-g.dj, g.y, 1.0);
  if constexpr (STAGE == 2) {
    g.e = __builtin_fma(g.e, g.e, g.e);
    g.ok = g.dj > 0.0;
    g.all &= g.ok;
  }
  if constexpr (STAGE == 3) {
    const double y = __builtin_fma(g.e, -g.y, -g.y);
    g.y = g.ok ? y : -1.0;
  }
  __builtin_amdgcn_sched_barrier(0);
}
template <int STAGE>
__device__ __forceinline__ void pivot_rest(PanelRegs& g) {
  if constexpr (STAGE < PIVOT_STAGES) {
    pivot_stage<STAGE>(g);
    pivot_rest<STAGE + 1>(g);
  }
}
// A DPP operand must not be read within two VALU instructions of its being written, and the compiler does not see into these
// statements: the first column's begins with the two multiplications that its operand needs anyway and ends with the broadcast
// of the next pivot, two instructions behind it; no later one reads what was written since.
template <int J>
__device__ __forceinline__ void panel_first_col(PanelRegs& g, double& md, double& ma) {
  asm("v_mul_f64 %0, %6, %8\n\t"
      "v_mul_f64 %1, %7, %8\n\t"
      "v_fmac_f64_dpp %2, %6, %0 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_fmac_f64_dpp %3, %6, %1 row_newbcast:%9 row_mask:0xf bank_mask:0xf\n\t"
      "v_mov_b64_dpp %4, %8 row_newbcast:0 row_mask:0xf bank_mask:%10\n\t"
      "v_mov_b64_dpp %5, %2 row_newbcast:%9 row_mask:0xf bank_mask:0xf"
      : "=&v"(md), "=&v"(ma), "+v"(g.d[J + 1]), "+v"(g.a[J + 1]), "+v"(g.yt[J & 3]), "=&v"(g.dj)
      : "v"(g.d[J]), "v"(g.a[J]), "v"(g.y), "n"(J + 1), "n"(1 << (J >> 2)));
  __builtin_amdgcn_sched_barrier(0);
}
template <int J, int K>
__device__ __forceinline__ void panel_cols(PanelRegs& g, double md, double ma) {
  if constexpr (K < 16) {
    asm("v_fmac_f64_dpp %0, %2, %3 row_newbcast:%5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f64_dpp %1, %2, %4 row_newbcast:%5 row_mask:0xf bank_mask:0xf"
        : "+v"(g.d[K]), "+v"(g.a[K]) : "v"(g.d[J]), "v"(md), "v"(ma), "n"(K));
    if constexpr (K - J - 1 < PIVOT_STAGES) pivot_stage<K - J - 1>(g);
    panel_cols<J, K + 1>(g, md, ma);
  } else {
    pivot_rest<(15 - J < PIVOT_STAGES ? 15 - J : PIVOT_STAGES)>(g);
  }
}
// out: where this lane's columns go
template <int J>
__device__ __forceinline__ void panel_steps(PanelRegs& g, double* out) {
  if constexpr (J < 15) {
    double md, ma;
    panel_first_col<J>(g, md, ma);
    pivot_stage<0>(g);
    if constexpr (J & 1) {
      out[J - 1] = g.a[J - 1];
      out[J] = g.a[J];
    }
    panel_cols<J, J + 2>(g, md, ma);
    panel_steps<J + 1>(g, out);
  } else {
    out[14] = g.a[14];
    out[15] = g.a[15];
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:0 row_mask:0xf bank_mask:0x8" : "+v"(g.yt[3]) : "v"(g.y));
  }
}
// the wavefront that runs the chain
__device__ __forceinline__ bool diag_chain(StepShared& sh, int lane) {
  double* S = sh.b;
  const int l16 = lane & 15;
  PanelRegs g;
  g.all = true;
#pragma unroll
  for (int q = 0; q < 4; ++q) asm("" : "=v"(g.yt[q]));
  int d0 = l16 * SL, a0 = lane < 16 ? EYE + 15 - lane : lane * SL, out = lane * SL;
#pragma unroll 1
  for (int p = 0; p < 4; ++p) {
#pragma unroll
    for (int c = 0; c < 16; ++c) g.d[c] = S[d0 + c];
#pragma unroll
    for (int c = 0; c < 16; ++c) g.a[c] = S[a0 + c];
    asm("s_nop 1\n\tv_mov_b64_dpp %0, %1 row_newbcast:0 row_mask:0xf bank_mask:0xf" : "=v"(g.dj) : "v"(g.d[0]));
    pivot_rest<0>(g);
    panel_steps<0>(g, S + out);
    double* y = sh.y + 16 * p + 4 * (l16 >> 2);
#pragma unroll
    for (int q = 0; q < 4; ++q) y[q] = g.yt[q];
    // rows below panel q sit in lanes 16 .. 63 - 16 q; lanes without one write to the blocks S(., 3)
    // above the diagonal, which hold nothing
    const int q = p + 1, row = (lane + 16 * q) & 63;
    d0 += 16 * SL + 16;
    if (lane >= 16) a0 = row * SL + 16 * q;
    out = lane < 64 - 16 * q ? row * SL + 16 * q : (16 * (3 - (lane >> 4)) + l16) * SL + 48;
    lds_barrier();
    if (p < 3) lds_barrier();
  }
  return g.all;
}
// out: the tile's place in L^-1 (leading dimension ldo), of which rows and columns below jb exist; or, IMG, a KC image in LDS, of
// which the 16 x 16 blocks above the diagonal are left as they are.  beside: what the wavefronts still have to store.
template <bool IMG, typename Block, typename Beside>
__device__ __forceinline__ void diag_block(StepShared& sh, int tid, double* out, long long ldo, int jb, int32_t* status, Block block, Beside beside) {
  double* S = sh.b;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  // rows 16 i .. of columns 16 c .. of L^-1: this lane's elements (4 r + lq, l16) of a block of W
  auto put = [&](int i, int c, const doublex4& w) {
    double rs[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double v = -sh.y[16 * i + 4 * r + lq], q = rsqrt_f64(v), s = v * q;
      rs[r] = __builtin_fma(__builtin_fma(-s, s, v), 0.5 * q, s);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * i + 4 * r + lq, k = 16 * c + l16;
      const double v = k <= m ? w[r] * rs[r] : 0.0;
      if (IMG) out[kc_off<NB>(k, m)] = v;
      else if (m < jb && k < jb) out[(long long)m * ldo + k] = v;
    }
  };
  auto put_diag = [&](int i) {
    doublex4 w;
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = S[(16 * i + l16) * SL + 16 * i + 4 * r + lq];
    put(i, i, w);
  };
  if (wave == 3) {
    const bool all = diag_chain(sh, lane);
    put_diag(3);
    if (!IMG) beside();
    if (!all && lane == 0) atomicCAS(status, 0, (int)STRP_ENOTPD);
    return;
  }
  // -Lu(i, k) as an A operand: columns 4 s + lq of row l16
  auto lu = [&](int i, int k, int s) { return S[(16 * i + l16) * SL + 16 * k + 4 * s + lq] * sh.y[16 * k + 4 * s + lq]; };
  // t += -Lu(i, k) W(k, c); one wavefront, 16 x 16 blocks.  A result register is the next product's B operand.
  auto w_add = [&](doublex4& t, int i, int k, int c) {
    doublex4 u = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double x = lu(i, k, s), y = k == c ? S[(16 * c + l16) * SL + 16 * c + 4 * s + lq] : S[(16 * c + 4 * s + lq) * SL + 16 * k + l16];
      if (s & 1) u = mma_f64(x, y, u);
      else t = mma_f64(x, y, t);
    }
    t += u;
  };
  // W(i, c) = W(i, i) t, t = -sum_{k = c}^{i - 1} Lu(i, k) W(k, c), into the image (unless it is the last row) and out
  auto w_finish = [&](const doublex4& t, int i, int c) {
    doublex4 u[2];
    u[0] = u[1] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      u[s & 1] = mma_f64(S[(16 * i + 4 * s + lq) * SL + 16 * i + l16], t[s], u[s & 1]);
    const doublex4 w = u[0] + u[1];
    if (i < 3) {
#pragma unroll
      for (int r = 0; r < 4; ++r) S[(16 * c + 4 * r + lq) * SL + 16 * i + l16] = w[r];
    }
    put(i, c, w);
  };
  // c = block (i, k) -= Lu(i, p) D Lu(k, p)^T
  auto s_update = [&](doublex4& c, int i, int k, int p) {
    doublex4 u = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double x = lu(i, p, s), y = S[(16 * k + l16) * SL + 16 * p + 4 * s + lq];
      if (s & 1) u = mma_f64(x, y, u);
      else c = mma_f64(x, y, c);
    }
    c += u;
  };
  auto s_put = [&](const doublex4& c, int i, int k) {
#pragma unroll
    for (int r = 0; r < 4; ++r) S[(16 * i + 4 * r + lq) * SL + 16 * k + l16] = c[r];
  };
  doublex4 t2, t3;                     // sums of wavefront c < 3 for W(2, c) and W(3, c)
  t2 = t3 = doublex4{0.0, 0.0, 0.0, 0.0};
  const int i2 = wave == 0 ? 2 : 3, k2 = wave == 2 ? 3 : 2;      // the wavefront's block of the last two block columns
  // beside panel 0
  if (IMG) beside();
  doublex4 c1 = block(1, 1 + wave, 1);
  if (!IMG) beside();
  lds_barrier();
  s_update(c1, 1 + wave, 1, 0);        // the next panel's columns
  s_put(c1, 1 + wave, 1);
  lds_barrier();
  // beside panel 1
  doublex4 c2 = block(2, i2, k2);
  s_update(c2, i2, k2, 0);
  if (wave == 0) put_diag(0);
  lds_barrier();
  if (wave < 2) {
    s_update(c2, i2, k2, 1);
    s_put(c2, i2, k2);
  }
  lds_barrier();
  // beside panel 2
  if (wave == 0) {
    doublex4 t1 = doublex4{0.0, 0.0, 0.0, 0.0};
    w_add(t1, 1, 0, 0);
    w_finish(t1, 1, 0);
    w_add(t2, 2, 0, 0);
    w_add(t2, 2, 1, 0);
  } else if (wave == 1) {
    w_add(t2, 2, 1, 1);
    w_add(t3, 3, 1, 1);
    put_diag(1);
  } else {
    s_update(c2, 3, 3, 1);
  }
  lds_barrier();
  if (wave == 2) {
    s_update(c2, 3, 3, 2);
    s_put(c2, 3, 3);
  }
  lds_barrier();
  // beside panel 3
  if (wave == 0) {
    w_add(t3, 3, 0, 0);
    w_add(t3, 3, 1, 0);
  }
  if (wave < 2) w_finish(t2, 2, wave);
  else put_diag(2);
  w_add(t3, 3, 2, wave);
  // blocks of L^-1 above the diagonal
#pragma unroll
  for (int c = 1; c < 4; ++c)
    if (!IMG && wave < c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * wave + 4 * r + lq, k = 16 * c + l16;
        if (m < jb && k < jb) out[(long long)m * ldo + k] = 0.0;
      }
  lds_barrier();
  w_finish(t3, 3, wave);
}

// 64 x 64 global tile (row-major) -> registers; rows [0, rv) and columns [0, cv) are valid.  src is the same for the whole
// wavefront: one 32-bit offset per lane, the rows' distances are scalar.
struct TileRegs {
  doublex2 r[8];
  __device__ __forceinline__ void load(const double* src, long long ld, int rv, int cv) {
    const int ch = threadIdx.x & 31, row0 = threadIdx.x >> 5;
    const unsigned int off = ((unsigned int)row0 * (unsigned int)ld + 2u * ch) * 8u;
    if (rv >= NB && cv >= NB) {
#pragma unroll
      for (int q = 0; q < 8; ++q) r[q] = *(const doublex2*)((const char*)(src + 8 * q * ld) + off);
    } else {
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int row = row0 + 8 * q;
        const double* p = (const double*)((const char*)(src + 8 * q * ld) + off);
        r[q] = doublex2{(row < rv && 2 * ch < cv) ? p[0] : 0.0, (row < rv && 2 * ch + 1 < cv) ? p[1] : 0.0};
      }
    }
  }
  __device__ __forceinline__ void store_kc(double* img) const {
    const int ch = threadIdx.x & 31, row0 = threadIdx.x >> 5;
#pragma unroll
    for (int q = 0; q < 8; ++q) *(doublex2*)(img + kc_off<NB>(2 * ch, row0 + 8 * q)) = r[q];
  }
  __device__ __forceinline__ void store_rc(double* img) const {
    const int ch = threadIdx.x & 31, row0 = threadIdx.x >> 5;
#pragma unroll
    for (int q = 0; q < 8; ++q) *(doublex2*)(img + rc_off<NB>(row0 + 8 * q, 2 * ch)) = r[q];
  }
};

// acc += tile product of two LDS images (A always KC)
template <bool BKC, int NI>
__device__ __forceinline__ void tile_mma(const double* ia, const double* ib, int wm, int wn, int lane, doublex4 (&acc)[NI][2]) {
  const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll 2
  for (int c = 0; c < 8; ++c) {
    const int k = 8 * c + 2 * lq;
    doublex2 af[NI], bf[2];
#pragma unroll
    for (int i = 0; i < NI; ++i) af[i] = *(const doublex2*)(ia + kc_off<NB>(k, wm + 16 * i + l16));
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (BKC) bf[j] = *(const doublex2*)(ib + kc_off<NB>(k, wn + 16 * j + l16));
      else bf[j] = doublex2{ib[rc_off<NB>(k, wn + 16 * j + l16)], ib[rc_off<NB>(k + 1, wn + 16 * j + l16)]};
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mma_f64(af[i].x, bf[j].x, acc[i][j]);
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = mma_f64(af[i].y, bf[j].y, acc[i][j]);
  }
}

// Products with a triangular operand: the wavefront pair that shares it takes 16-wide tiles {0, 3} and {1, 2} of the
// triangular side, 10 eight-step chunks each, instead of 6 against 14.
__device__ __forceinline__ int tri_tile(int half, int j) { return half ? 1 + j : 3 * j; }
// acc[i][j] = T (rows wm + 16 i) times M^T (columns 16 tri_tile(half, j)), M lower triangular; both KC images.  Even and odd
// contraction steps are summed apart: a chain on one accumulator runs at the instruction's latency, four keep it busy.  The fragments of
// a step are read one step ahead, across the two columns too.
template <int NI, int T0, int T1>
__device__ __forceinline__ void mma_lower_t_cols(const double* it, const double* im, int wm, int lane, doublex4 (&acc)[NI][2]) {
  constexpr int N0 = 2 * (T0 + 1), N = N0 + (T1 >= 0 ? 2 * (T1 + 1) : 0);
  const int l16 = lane & 15, lq = lane >> 4;
  doublex4 s[NI][2];
  doublex2 b[2], a[2][NI];
  const double* const am = im + kc_off<NB>(2 * lq, l16);
  const double* const at = it + kc_off<NB>(2 * lq, wm + l16);
  auto read = [&](int e) {
    const int k = 8 * (e < N0 ? e : e - N0);
    b[e & 1] = *(const doublex2*)(am + kc_off<NB>(k, 16 * (e < N0 ? T0 : T1)));
#pragma unroll
    for (int i = 0; i < NI; ++i) a[e & 1][i] = *(const doublex2*)(at + kc_off<NB>(k, 16 * i));
  };
  read(0);
#pragma unroll
  for (int e = 0; e < N; ++e) {
    if (e == 0 || e == N0) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if (e) acc[i][0] = s[i][0] + s[i][1];
        s[i][0] = s[i][1] = doublex4{0.0, 0.0, 0.0, 0.0};
      }
    }
    if (e + 1 < N) read(e + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NI; ++i) s[i][0] = mma_f64(a[e & 1][i].x, b[e & 1].x, s[i][0]);
#pragma unroll
    for (int i = 0; i < NI; ++i) s[i][1] = mma_f64(a[e & 1][i].y, b[e & 1].y, s[i][1]);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) acc[i][T1 >= 0 ? 1 : 0] = s[i][0] + s[i][1];
}
template <int NI>
__device__ __forceinline__ void mma_lower_t(const double* it, const double* im, int wm, int half, int lane, doublex4 (&acc)[NI][2]) {
  if (half) mma_lower_t_cols<NI, 1, 2>(it, im, wm, lane, acc);
  else mma_lower_t_cols<NI, 0, 3>(it, im, wm, lane, acc);
}
// acc[i][j] = M (rows 16 tri_tile(half, i), lower triangular, KC image) times T (columns wn + 16 j, RC image)
__device__ __forceinline__ void mma_lower(const double* im, const double* it, int half, int wn, int lane, doublex4 (&acc)[2][2]) {
  const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int mt = tri_tile(half, i);
    doublex4 s[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) s[j][0] = s[j][1] = doublex4{0.0, 0.0, 0.0, 0.0};
    for (int c2 = 0; c2 <= mt; ++c2)
#pragma unroll
    for (int c = 2 * c2; c < 2 * c2 + 2; ++c) {
      const int k = 8 * c + 2 * lq;
      const doublex2 a = *(const doublex2*)(im + kc_off<NB>(k, 16 * mt + l16));
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        s[j][0] = mma_f64(a.x, it[rc_off<NB>(k, wn + 16 * j + l16)], s[j][0]);
        s[j][1] = mma_f64(a.y, it[rc_off<NB>(k + 1, wn + 16 * j + l16)], s[j][1]);
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = s[j][0] + s[j][1];
  }
}

// the 64 x 64 tile at `src` in the accumulator layout (this lane's 16 elements; past a ragged edge the edge's)
template <int NI>
__device__ __forceinline__ void load_acc(const double* src, long long ld, int rv, int cv, int wm, int wn, int lane, doublex4 (&c)[NI][2]) {
  const int l16 = lane & 15, lq = lane >> 4;
  const bool full = rv >= NB && cv >= NB;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = wm + 16 * i + 4 * r, k = wn + 16 * j;
        if (full) {
          c[i][j][r] = *(const double*)((const char*)(src + m * ld + k) + ((unsigned int)lq * (unsigned int)ld + l16) * 8u);
        } else {                // a clamped address keeps the ragged case free of branches
          const unsigned int mc = m + lq < rv ? m + lq : rv - 1, kc = k + l16 < cv ? k + l16 : cv - 1;
          c[i][j][r] = *(const double*)((const char*)src + (mc * (unsigned int)ld + kc) * 8u);
        }
      }
}
template <int NI>
__device__ __forceinline__ void store_acc(double* dst, long long ld, int rv, int cv, int wm, int wn, int lane, const doublex4 (&c)[NI][2]) {
  const int l16 = lane & 15, lq = lane >> 4;
  const bool full = rv >= NB && cv >= NB;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = wm + 16 * i + 4 * r, k = wn + 16 * j;
        if (full || (m + lq < rv && k + l16 < cv))
          *(double*)((char*)(dst + m * ld + k) + ((unsigned int)lq * (unsigned int)ld + l16) * 8u) = c[i][j][r];
      }
}
template <int NI>
__device__ __forceinline__ void zero_acc(doublex4 (&c)[NI][2]) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) c[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};
}

// this lane's elements of a result whose columns are 16 tri_tile(half, j), into a KC image (row = m, k = n)
template <int NI, int T0, int T1>
__device__ __forceinline__ void put_kc_cols(double* img, const doublex4 (&acc)[NI][2]) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) img[kc_off<NB>(16 * (j ? T1 : T0), 16 * i + 4 * r)] = acc[i][j][r];
}
template <int NI>
__device__ __forceinline__ void put_kc_tri(double* img, int wm, int half, int lane, const doublex4 (&acc)[NI][2]) {
  double* const at = img + kc_off<NB>(lane & 15, wm + (lane >> 4));
  if (half) put_kc_cols<NI, 1, 2>(at, acc);
  else put_kc_cols<NI, 0, 3>(at, acc);
}

}  // namespace strp
