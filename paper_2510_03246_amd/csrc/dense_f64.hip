// fp64 dense kernels for the ridge systems: one launch chain that factors an SPD matrix and inverts its triangular
// factor at the same time, right-side solves as two triangular-aware GEMMs, and small cast / scatter helpers.
// The Gram systems reach condition numbers ~1e4, so factor and solve stay in fp64.  Everything runs on the fp64
// matrix cores: v_mfma_f64_16x16x4_f64 sustains 73-77 TFLOP/s here with four or more independent accumulators per
// SIMD (plain v_fma_f64 67; the two share their units, a mix of both is no faster), far above what LDS or L2 can feed
// to a naive tiling -- so the kernels below are about operand traffic, loads in flight and launches, not arithmetic.
#include "cojob.h"
#include "f64_tiles.h"
#include "strp_internal.h"

namespace strp {

// ---------------------------------------------------------------------------------------------
// dgemm: C[m, n] = sum_k A(m, k) B(k, n), C row-major.
//   block = 4 wavefronts (2 x 2) or two such shares of K, TM x TN output tile, K staged DK at a time through double-buffered LDS; the next
//   stage's 16-byte loads are in flight while a stage is multiplied.
//   A: AKC ? A[m * lda + k] : A[k * lda + m];   B: BKC ? B[n * ldb + k] : B[k * ldb + n].
//   tri restricts the K range of a tile to where a triangular operand is non-zero:
//     1: k < n0 + TN (B upper in (k, n)),  2: k >= n0 (B lower),  3: k >= m0 (A upper in (m, k), with lower).
//   lower != 0 skips output tiles entirely above the diagonal.
// ---------------------------------------------------------------------------------------------
struct DgemmP {
  int M, N, K;
  const double* A; long long lda;
  const double* B; long long ldb;
  double* C; long long ldc;
  int lower, tri;
  unsigned int* maxbits;    // optional: atomic maximum of the bits of |C|
  WeightsOut w;             // w.W: the result as refitted weights instead of C (one fp64 matrix less to write and read)
};

template <int R, int DK, bool KC, int NT>
struct F64Loader {
  static constexpr int NCH = R * DK / 2 / NT;   // 16-byte pieces per thread and stage
  doublex2 r[NCH];
  // A whole stage with 16-byte loads: the same instructions for every tile and stage, so that the wait for one stage leaves the
  // next one's loads in flight (behind a branch the compiler has to wait for all of them).  Rows past the edge repeat the
  // last one: what comes of them is not stored.
  static __device__ __forceinline__ void offsets(unsigned int (&off)[NCH], long long ld, int rv) {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int e = (int)threadIdx.x + NT * q;
      if (KC) {
        const int row = e / (DK / 2);
        off[q] = ((unsigned int)(row < rv ? row : rv - 1) * (unsigned int)ld + 2u * (e % (DK / 2))) * 8u;
      } else {
        const int row = 2 * (e % (R / 2)), last = (rv - 1) & ~1;        // a row pair, which ends inside an even leading dimension
        off[q] = ((unsigned int)(e / (R / 2)) * (unsigned int)ld + (unsigned int)(row < rv ? row : last)) * 8u;
      }
    }
  }
  // src: row 0 at the stage's first k
  __device__ __forceinline__ void load_whole(const double* src, const unsigned int (&off)[NCH]) {
#pragma unroll
    for (int q = 0; q < NCH; ++q) r[q] = *(const doublex2u*)((const char*)src + off[q]);
  }
  // rows [0, rv) and k in [k0, kend) are valid; src points at row 0
  __device__ __forceinline__ void load(const double* src, long long ld, int rv, int k0, int kend) {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int e = (int)threadIdx.x + NT * q;
      if (KC) {
        const int ch = e % (DK / 2), row = e / (DK / 2);
        const int k = k0 + 2 * ch;
        const double* p = src + (long long)row * ld + k;
        r[q] = doublex2{(row < rv && k < kend) ? p[0] : 0.0, (row < rv && k + 1 < kend) ? p[1] : 0.0};
      } else {
        const int pr = e % (R / 2), kk = k0 + e / (R / 2);
        const int row = 2 * pr;
        const double* p = src + (long long)kk * ld + row;
        r[q] = doublex2{(row < rv && kk < kend) ? p[0] : 0.0, (row + 1 < rv && kk < kend) ? p[1] : 0.0};
      }
    }
  }
  __device__ __forceinline__ void store(double* img) const {
#pragma unroll
    for (int q = 0; q < NCH; ++q) {
      const int e = (int)threadIdx.x + NT * q;
      if (KC) *(doublex2*)(img + kc_off<R>(2 * (e % (DK / 2)), e / (DK / 2))) = r[q];
      else *(doublex2*)(img + rc_off<R>(e / (R / 2), 2 * (e % (R / 2)))) = r[q];
    }
  }
};
template <int R, int DK, bool KC>
constexpr int f64_img_elems() { return KC ? DK / 2 * (R + 1) * 2 : DK * (R + 4); }

constexpr int CUS = 256;
// The two small tiles have eight wavefronts: two shares of every stage's K, whose sums are added at the end.  With four, a long tile that
// is left alone on its CU has one wavefront and two to four chains of products per SIMD, and nothing to issue while that one reads LDS or
// waits at a barrier.  Both products of a solve, us, four / eight wavefronts: 256 x 512 28.7 / 25.2, 1000 x 1013 59.5 / 51.3, 768 x 1536
// 89.4 / 78.7, 2048 x 3277 700 / 681, 4096 x 4915 (64 x 64) 3190 / 3032 (65 TFLOP/s).  The 128 x 128 tile has 16 chains a wavefront.
constexpr int k_shares(int TM, int TN) { return TM * TN >= 128 * 128 ? 1 : 2; }
template <int TM, int TN, int DK, bool AKC, bool BKC>
__device__ __forceinline__ void dgemm_block(const DgemmP& p, int block) {
  constexpr int WM = TM / 32, WN = TN / 32;     // 16 x 16 tiles per wavefront
  constexpr int KS = k_shares(TM, TN);
  __shared__ __attribute__((aligned(16))) double As[2][f64_img_elems<TM, DK, AKC>()];
  __shared__ __attribute__((aligned(16))) double Bs[2][f64_img_elems<TN, DK, BKC>()];
  const int tilesM = (p.M + TM - 1) / TM, tilesN = (p.N + TN - 1) / TN;
  // the rows of C walk fastest; column tiles go in order of decreasing K range
  int tn_ = block / tilesM, tm_ = block - tn_ * tilesM;
  // Of a solve with up to three workgroups per CU all run from the start, and a CU has those that are 256 apart: every other 256
  // go in order of increasing K range, so that a CU with a long tile has short ones beside it.  With more of them the longest
  // first end the soonest, since a CU takes the next when it has done with one.  In order / turned, us of both products: 576 x 928
  // (261 tiles) 50.1 / 50.8, 1000 x 1013 (512) 65.4 / 59.5, 768 x 1536 (576) 96.8 / 89.4,
  // 640 x 2000 (630) 133.2 / 125.5, 200 x 4000 (500) 213.1 / 188.3, 1024 x 1536 (768) 109.9 / 102.7.
  if (TN == 32 && p.tri != 3 && tilesM <= CUS && tilesM * tilesN > CUS && tilesM * tilesN <= 3 * CUS) {
    const int turn = CUS / tilesM, beg = tn_ / turn * turn, end = beg + turn < tilesN ? beg + turn : tilesN;
    if (tn_ / turn & 1) tn_ = beg + end - 1 - tn_;
  }
  const int m0 = tm_ * TM, n0 = (p.tri == 1 ? tilesN - 1 - tn_ : tn_) * TN;
  if (p.lower && n0 >= m0 + TM) return;
  int kbeg = 0, kend = p.K;
  if (p.tri == 1) kend = n0 + TN < p.K ? n0 + TN : p.K;
  if (p.tri == 2) kbeg = n0;
  if (p.tri == 3) kbeg = m0;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave >> 1 & 1) * (TM / 2), wn = (wave & 1) * (TN / 2), share = wave >> 2;
  const int l16 = lane & 15, lq = lane >> 4;
  doublex4 acc[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = doublex4{0.0, 0.0, 0.0, 0.0};

  const double* A = AKC ? p.A + (long long)m0 * p.lda : p.A + m0;
  const double* B = BKC ? p.B + (long long)n0 * p.ldb : p.B + n0;
  const int rvm = p.M - m0, rvn = p.N - n0;
  // Stages in flight in registers besides the one in LDS that is multiplied: two, since with few workgroups per CU a stage of a
  // small tile is multiplied in less time than a load takes; one for the 128 x 128 tile, whose stage takes far longer than that and
  // whose accumulators leave no room for a second (two spilled 52 registers: 6000 x 6000 6642 us instead of 6479, 8602 x 7168 13497
  // instead of 13089).
  constexpr int SETS = TM * TN >= 128 * 128 ? 1 : 2;
  F64Loader<TM, DK, AKC, 256 * KS> la[SETS];
  F64Loader<TN, DK, BKC, 256 * KS> lb[SETS];
  auto multiply = [&](int buf) {
    const double* as = As[buf];
    const double* bs = Bs[buf];
#pragma unroll
    for (int c = 0; c < DK / 8 / KS; ++c) {
      doublex2 af[WM], bf[WN];
      const int k = DK / KS * share + 8 * c + 2 * lq;
#pragma unroll
      for (int i = 0; i < WM; ++i) {
        if (AKC) af[i] = *(const doublex2*)(as + kc_off<TM>(k, wm + 16 * i + l16));
        else af[i] = doublex2{as[rc_off<TM>(k, wm + 16 * i + l16)], as[rc_off<TM>(k + 1, wm + 16 * i + l16)]};
      }
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        if (BKC) bf[j] = *(const doublex2*)(bs + kc_off<TN>(k, wn + 16 * j + l16));
        else bf[j] = doublex2{bs[rc_off<TN>(k, wn + 16 * j + l16)], bs[rc_off<TN>(k + 1, wn + 16 * j + l16)]};
      }
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = mma_f64(af[i].x, bf[j].x, acc[i][j]);
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = mma_f64(af[i].y, bf[j].y, acc[i][j]);
    }
  };
  const bool pairs = (AKC || rvm >= TM || p.lda % 2 == 0) && (BKC || rvn >= TN || p.ldb % 2 == 0);
  const int whole = pairs && kend > kbeg ? (kend - kbeg) / DK : 0;
  if (whole) {
    unsigned int offa[F64Loader<TM, DK, AKC, 256 * KS>::NCH], offb[F64Loader<TN, DK, BKC, 256 * KS>::NCH];
    F64Loader<TM, DK, AKC, 256 * KS>::offsets(offa, p.lda, rvm);
    F64Loader<TN, DK, BKC, 256 * KS>::offsets(offb, p.ldb, rvn);
    auto gload = [&](int set, int s) {      // past the end: the last one again, never multiplied
      const long long k = kbeg + (long long)(s < whole ? s : whole - 1) * DK;
      la[set].load_whole(AKC ? A + k : A + k * p.lda, offa);
      lb[set].load_whole(BKC ? B + k : B + k * p.ldb, offb);
    };
    auto put = [&](int set, int buf) {      // the buffer's readers finished before the previous barrier
      la[set].store(As[buf]);
      lb[set].store(Bs[buf]);
    };
    auto stage = [&](int buf, int s) {      // multiply stage s, held in As[buf]; the next one is in set buf ^ 1, or in the only one
      if constexpr (SETS == 2) {
        gload(buf, s + 2);
        multiply(buf);
        put(buf ^ 1, buf ^ 1);
      } else {
        put(0, buf ^ 1);
        gload(0, s + 2);
        multiply(buf);
      }
      lds_barrier();
    };
    gload(0, 0);
    if constexpr (SETS == 2) gload(1, 1);
    put(0, 0);
    if constexpr (SETS == 1) gload(0, 1);
    lds_barrier();
    int s = 0;
    for (; s + 2 <= whole; s += 2) {
      stage(0, s);
      stage(1, s + 1);
    }
    if (s < whole) stage(0, s);
  }
  // what is left of K, and row pairs that would end past an odd matrix
  for (int k0 = kbeg + whole * DK; k0 < kend; k0 += DK) {
    la[0].load(A, p.lda, rvm, k0, kend);
    lb[0].load(B, p.ldb, rvn, k0, kend);
    la[0].store(As[0]);
    lb[0].store(Bs[0]);
    lds_barrier();
    multiply(0);
    lds_barrier();
  }
  if constexpr (KS == 2) {         // the second share's sums to the first, through LDS that nobody reads any more
    static_assert(TM * TN <= 2 * f64_img_elems<TM, DK, AKC>(), "");
    double* x = As[0] + (wave & 3) * (WM * WN * 4 * 64) + lane;
    if (share) {
#pragma unroll
      for (int e = 0; e < WM * WN * 4; ++e) x[64 * e] = acc[e / 4 / WN][e / 4 % WN][e % 4];
    }
    lds_barrier();
    if (!share) {
#pragma unroll
      for (int e = 0; e < WM * WN * 4; ++e) acc[e / 4 / WN][e / 4 % WN][e % 4] += x[64 * e];
    }
  }
  double big = 0.0, sq = 0.0;
  if (share) {
  } else if (p.w.W) {
    const bool fc2 = p.w.side == STRP_SIDE_FC2;
    // where rows and columns go, all indices asked for at once and clamped (under the condition of the store each one was waited for: 64 rows of 128
    // 8.2 / 7.5 us, 200 of 400 14.1 / 13.3)
    int wrow[WM][4], wcol[WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + 4 * r + lq;
        wrow[i][r] = m < p.M ? m : p.M - 1;
      }
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int n = n0 + wn + 16 * j + l16;
      wcol[j] = n < p.N ? n : p.N - 1;
    }
    if (fc2) {
#pragma unroll
      for (int j = 0; j < WN; ++j) wcol[j] = p.w.idx[wcol[j]];
    } else {
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) wrow[i][r] = p.w.idx[wrow[i][r]];
    }
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int n = n0 + wn + 16 * j + l16;
#pragma unroll
      for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + wm + 16 * i + 4 * r + lq;
          if (m < p.M && n < p.N) {
            const float v = (float)acc[i][j][r];
            p.w.W[(long long)wrow[i][r] * p.w.ldw + wcol[j]] = v;
            if (p.w.Wc) p.w.Wc[(long long)m * p.w.ldc + n] = v;
            big = fmax(big, fabs((double)v));
            sq = __builtin_fma((double)v, (double)v, sq);
          }
        }
    }
  } else {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int n = n0 + wn + 16 * j + l16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + wm + 16 * i + 4 * r + lq;
          if (m < p.M && n < p.N) {
            p.C[(long long)m * p.ldc + n] = acc[i][j][r];
            big = fmax(big, fabs(acc[i][j][r]));
          }
        }
      }
  }
  unsigned int* maxbits = p.w.W ? p.w.maxbits : p.maxbits;
  if (maxbits || p.w.sumsq) {
    double* red = As[0];                    // every wavefront is past the last barrier
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      big = fmax(big, __shfl_down(big, o, 64));
      sq += __shfl_down(sq, o, 64);
    }
    if constexpr (KS == 2) lds_barrier();
    if (lane == 0 && !share) {
      red[2 * wave] = big;
      red[2 * wave + 1] = sq;
    }
    lds_barrier();
    if (tid == 0) {
      if (maxbits) atomicMax(maxbits, __builtin_bit_cast(unsigned int, (float)fmax(fmax(red[0], red[2]), fmax(red[4], red[6]))));
      if (p.w.sumsq) p.w.sumsq[tn_ * tilesM + tm_] = red[1] + red[3] + red[5] + red[7];
    }
  }
}

template <int TM, int TN, int DK, bool AKC, bool BKC>
__global__ __launch_bounds__(256 * k_shares(TM, TN), 2) void dgemm_kernel(const DgemmP p) { dgemm_block<TM, TN, DK, AKC, BKC>(p, blockIdx.x); }

// two independent products, one behind the other in the grid: `first` workgroups are the first's
struct DgemmPair {
  DgemmP p[2];
  int first;
};
template <int TM, int TN, int DK, bool AKC, bool BKC>
__global__ __launch_bounds__(256 * k_shares(TM, TN), 2) void dgemm_pair_kernel(const DgemmPair g) {
  const int second = (int)blockIdx.x >= g.first;
  dgemm_block<TM, TN, DK, AKC, BKC>(g.p[second], (int)blockIdx.x - second * g.first);
}

// Tile of a product by its grid: 128 x 128 tiles read the fewest operand bytes per flop but need enough of them to fill
// the chip; below that the longest tile (whole K) sets the run time and a smaller one ends sooner.  Solves X (L L^T)^-1 of
// m x n (two products, rows of whole cache lines), us with 64 x 64 / 128 x 128 tiles (in brackets the tiles of 128):  4096 x 4915 (1248) 3053 / 3231,
// 64 TFLOP/s;  4915 x 4096 2515 / 2677;  5100 x 5100 (1600) 4065 / 4171;  6000 x 5990 (2209) 6588 / 6628;  6400 x 6300 (2500) 7757 / 7784;
// 8000 x 5000 (2520) 6090 / 6286;  7000 x 7000 (3025) 11049 / 10630;  8602 x 7168 (3808) 13723 / 13082.
// Between the two small ones the number of tile rows decides: workgroups go to the 8 XCDs in turn, so that with an even number an
// XCD meets only some rows of A, again and again, and with an odd one all of them, which costs the tile that reads A for fewer
// columns.  64 x 32 / 64 x 64 (tiles of 64), even:  768 x 1536 (288) 80 / 122;  2048 x 2458 (1248) 394 / 407;  1784 x 3611 (1596) 746 / 764;  2048 x 3277
// (1664) 694 / 699;  1912 x 3637 (1710) 833 / 815;  2424 x 2869 (1710) 645 / 633;  3320 x 2101 (1716) 469 / 473;  2680 x 2869 (1890) 723 / 700.  Of
// 17 such numbers of rows 11 have 64 x 64 ahead at about 1700 tiles, 3 at 1500.  Odd:  1344 x 1653 (546) 156 / 169;  1088 x 2229 (595) 217 / 226;
// 1984 x 1205 (589) 134 / 133;  1344 x 1909 (630) 199 / 201;  1728 x 1525 (648) 170 / 166;  960 x 2741 (645) 298 / 283;  576 x 4853 (684) 544 / 505.
// Linv^T Linv (half the tiles), order, 64 x 32 / 64 x 64:  1536 (288) 41 / 68;  2200 (612) 102 / 120;  2600 (840) 159 / 145;  2800 (968) 152 / 158;
// 2904 (1058) 208 / 175;  3104 (1200) 251 / 209;  4096 (2048) 514 / 440;  64 x 64 / 128 x 128 (tiles of 128):  7168 (1568) 2180 / 2313;
// 8192 (2048) 3384 / 3507;  8704 (2312) 3822 / 3812;  9216 (2592) 4554 / 4439;  10240 (3200) 6720 / 6056.
constexpr int DGEMM_T128 = 2600, DGEMM_T128_LOWER = 2500, DGEMM_T64 = 1700, DGEMM_T64_ODD = 630, DGEMM_T64_LOWER = 1000;

static inline bool aligned_vec(const void* p, long long ld) { return ((uintptr_t)p & 15u) == 0 && (ld & 1) == 0; }

struct DgemmTile { int tm, tn; };
static DgemmTile dgemm_tile(int M, int N, int lower) {
  auto tiles = [&](int tm, int tn) { return (long long)((M + tm - 1) / tm) * ((N + tn - 1) / tn) / (lower ? 2 : 1); };
  if (tiles(128, 128) >= (lower ? DGEMM_T128_LOWER : DGEMM_T128)) return {128, 128};
  const int t64 = lower ? DGEMM_T64_LOWER : (M + 63) / 64 % 2 ? DGEMM_T64_ODD : DGEMM_T64;
  return tiles(64, 64) >= t64 ? DgemmTile{64, 64} : DgemmTile{64, 32};
}
static int dgemm_blocks(int M, int N, DgemmTile t) { return ((M + t.tm - 1) / t.tm) * ((N + t.tn - 1) / t.tn); }
int weights_out_blocks(int m, int n) { return dgemm_blocks(m, n, dgemm_tile(m, n, 0)); }

template <bool AKC, bool BKC>
static strp_status dgemm_launch(strp_ctx* ctx, const DgemmP& p) {
  if (p.M <= 0 || p.N <= 0) return STRP_OK;
  const DgemmTile t = dgemm_tile(p.M, p.N, p.lower);
  const dim3 grid(dgemm_blocks(p.M, p.N, t));
  if (t.tm == 128) hipLaunchKernelGGL((dgemm_kernel<128, 128, 16, AKC, BKC>), grid, dim3(256), 0, ctx->stream, p);
  else if (t.tn == 64) hipLaunchKernelGGL((dgemm_kernel<64, 64, 32, AKC, BKC>), grid, dim3(512), 0, ctx->stream, p);
  else hipLaunchKernelGGL((dgemm_kernel<64, 32, 32, AKC, BKC>), grid, dim3(512), 0, ctx->stream, p);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// Lower triangle (128-row tiles on or below the diagonal) of S = Linv^T Linv, Linv lower triangular.
strp_status gram_of_inverse(strp_ctx* ctx, const double* Linv, int n, long long ldl, double* S, long long lds, unsigned int* maxbits) {
  DgemmP p;
  memset(&p, 0, sizeof(p));
  p.M = n; p.N = n; p.K = n; p.A = Linv; p.lda = ldl; p.B = Linv; p.ldb = ldl; p.C = S; p.ldc = lds; p.lower = 1; p.tri = 3; p.maxbits = maxbits;
  return dgemm_launch<false, false>(ctx, p);
}

// The chain, for what chol_flow_ok leaves to it: orders 65 .. 71, and 63 .. 68 and 84 .. 90 tiles without a long pass; a single tile is
// its first launch alone.
// One launch of it: everything that step t can do once the steps before it are complete.  Panels are 64 columns
// (tile index = row or column / 64); A is factored in place below its diagonal tiles, Linv is built beside it by
// carrying the identity through the same elimination (its row i holds partial sums V until step i).  Panel t - 1 is
// applied to the tiles behind it by launch t ("pending"):
//   P(t + 1):  L(t+1, t) = A(t+1, t) L(t, t)^-T,  A(t+1, t+1) -= L(t+1, t) L(t+1, t)^T, and the factor of that diagonal
//              tile, inverted: Linv(t+1, t+1)
//   P(i):      L(i, t) = (A(i, t) - L(i, t-1) L(t, t-1)^T) L(t, t)^-T,  A(i, i) -= L(i, t) L(i, t)^T
//   ahead(h):  rows 32 h .. of what the next launch's first task would otherwise have to begin with: both panels' part of
//              A(t+2, t+1), for which it forms those rows of L(t+2, t) and L(t+1, t) a second time
//   R(c):      Linv(t, c) = L(t, t)^-1 (V(t, c) - L(t, t-1) Linv(t-1, c)),  c < t
//   TA(i, k):  A(i, k) -= L(i, t-1) L(k, t-1)^T,  i > k > t, (i, k) != (t + 2, t + 1)
//   TV(i, c):  V(i, c) -= L(i, t-1) Linv(t-1, c),  i > t, c < t
// No workgroup of a launch reads what another one of it writes: L(t+1, t) and L(t+2, t) go to a buffer of their own (near_l)
// because ahead reads what they would replace; the next launch is the last to read them.  A launch costs what P(t + 1) does
// while the others fit beside it: 5 us for two 64^3 products at the 0.3 TFLOP/s of one CU and their operands, of which the
// second needs only its first 16 columns before the diagonal tile's chain of 64 pivots can begin, and 6 us for that chain.
// us a launch of few tiles: 17.5 with one workgroup for P(t + 2) and ahead, which took longer than P(t + 1), 14.0 with these
// apart, 13.0 with fewer stores in the chain, 12.2 with the second product beside the chain.  Larger orders are bound by the trailing
// tiles' traffic: 29 us a launch on average at n = 4096 (1.85 ms), 44 at 5376 (3.69).
struct StepP {
  double* A; long long ld;
  double* V; long long ldv;     // Linv
  double* sub;                  // up to four tiles [NB * NB]: L(t+1, t) and L(t+2, t) of this launch and the last (near_l)
  int n, N;                     // order, tiles
  int t;
  int each;                     // tiles of TA and TV per workgroup
  int32_t* status;
};

// where L(t + 1 + far, t) is, t the launch that forms it
__device__ __forceinline__ double* near_l(const StepP& p, int t, int far) { return p.sub + (2 * far + (t & 1)) * NB * NB; }
// P(i) of launch t.  FIRST: i = t + 1 (nothing pending, factors the diagonal tile).
template <bool FIRST>
__device__ __forceinline__ void step_panel(const StepP& p, StepShared& sh, int i) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32, half = wave & 1;
  const int l16 = lane & 15, lq = lane >> 4;
  const int t = p.t;
  const int rows = p.n - i * NB, jb = rows < NB ? rows : NB;
  auto At = [&](int r, int c) { return p.A + (long long)r * NB * p.ld + (long long)c * NB; };
  const double* inv_t = p.V + (long long)t * NB * (p.ldv + 1);     // L(t, t)^-1
  TileRegs ra, rb;
  doublex4 acc[2][2];
  if (FIRST || t == 0) {                  // nothing is pending: the tile goes to LDS as it is
    ra.load(At(i, t), p.ld, rows, NB);
    rb.load(inv_t, p.ldv, NB, NB);
    ra.store_kc(sh.a);
    rb.store_kc(sh.b);
  } else {
    doublex4 c[2][2];
    ra.load(At(i, t - 1), p.ld, rows, NB);
    rb.load(near_l(p, t - 1, 0), NB, NB, NB);
    load_acc(At(i, t), p.ld, rows, NB, wm, wn, lane, c);
    ra.store_kc(sh.a);
    rb.store_kc(sh.b);
    lds_barrier();
    rb.load(inv_t, p.ldv, NB, NB);
    zero_acc(acc);
    tile_mma<true>(sh.a, sh.b, wm, wn, lane, acc);
    lds_barrier();
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sh.a[kc_off<NB>(wn + 16 * j + l16, wm + 16 * ii + 4 * r + lq)] = c[ii][j][r] - acc[ii][j][r];
    rb.store_kc(sh.b);
  }
  // 16 x 16 blocks of the diagonal tile A(i, i), lower triangle.  FIRST: block (wave, 0), which the chain begins with, and for
  // wavefronts 0 .. 2 those that diag_block asks for.  Otherwise three for wavefronts 0 and 1, two (and one of them again) for 2 and 3
  const int dn = wave < 2 ? 3 : 2;
  const auto drow = [&](int q) {
    if (FIRST) return q == 0 ? wave : q == 1 ? (wave < 3 ? 1 + wave : 3) : wave == 0 ? 2 : 3;
    return wave == 0 ? int(q > 0) : wave == 1 ? 2 : 3;
  };
  const auto dcol = [&](int q) {
    if (FIRST) return q == 0 ? 0 : q == 1 ? 1 : wave < 2 ? 2 : 3;
    return wave == 0 ? int(q > 1) : wave == 1 ? q : wave == 2 ? q : 2 + (q & 1);
  };
  doublex4 dc[3];
#pragma unroll
  for (int q = 0; q < 3; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int m = 16 * drow(q) + 4 * r + lq, k = 16 * dcol(q) + l16;
      m = m < jb ? m : jb - 1;
      k = k < jb ? k : jb - 1;
      dc[q][r] = At(i, i)[(long long)m * p.ld + k];
    }
  lds_barrier();
  mma_lower_t(sh.a, sh.b, wm, half, lane, acc);
  lds_barrier();
  put_kc_tri(sh.a, wm, half, lane, acc);
  auto store_l = [&] {
    const bool aside = i <= t + 2;
    double* out = aside ? near_l(p, t, i - t - 1) : At(i, t);
    const long long ldo = aside ? NB : p.ld;
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = wm + 16 * ii + 4 * r + lq;
          if (aside || m < jb) out[(long long)m * ldo + 16 * tri_tile(half, j) + l16] = acc[ii][j][r];
        }
  };
  if (!FIRST) store_l();
  lds_barrier();
  if constexpr (FIRST) {
    // rows of L past the edge are zero: what is put there stays
    auto block = [&](int q) {
      doublex4 u[2];
      u[0] = u[1] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) {
        const int k = 8 * cc + 2 * lq;
        const doublex2 x = *(const doublex2*)(sh.a + kc_off<NB>(k, 16 * drow(q) + l16)), y = *(const doublex2*)(sh.a + kc_off<NB>(k, 16 * dcol(q) + l16));
        u[0] = mma_f64(x.x, y.x, u[0]);
        u[1] = mma_f64(x.y, y.y, u[1]);
      }
      doublex4 v = dc[q];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * drow(q) + 4 * r + lq, k = 16 * dcol(q) + l16;
        if (jb < NB) v[r] = m < jb && k < jb ? v[r] : (m == k ? 1.0 : 0.0);
      }
      return v - (u[0] + u[1]);
    };
    put_eye(sh, tid);                     // sh.b: its readers are past the barrier before last
    const doublex4 c0 = block(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) sh.b[(16 * wave + 4 * r + lq) * SL + l16] = c0[r];
    lds_barrier();
    diag_block<false>(sh, tid, p.V + (long long)i * NB * (p.ldv + 1), p.ldv, jb, p.status, [&](int q, int, int) { return block(q); }, store_l);
    return;
  }
  {
    doublex4 s[3][2];
#pragma unroll
    for (int q = 0; q < 3; ++q) s[q][0] = s[q][1] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int cc = 0; cc < 8; ++cc) {
      const int k = 8 * cc + 2 * lq;
      doublex2 x[3], y[3];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        x[q] = *(const doublex2*)(sh.a + kc_off<NB>(k, 16 * drow(q) + l16));
        y[q] = *(const doublex2*)(sh.a + kc_off<NB>(k, 16 * dcol(q) + l16));
      }
#pragma unroll
      for (int q = 0; q < 3; ++q) s[q][0] = mma_f64(x[q].x, y[q].x, s[q][0]);
#pragma unroll
      for (int q = 0; q < 3; ++q) s[q][1] = mma_f64(x[q].y, y[q].y, s[q][1]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) dc[q] -= s[q][0] + s[q][1];
  }
#pragma unroll
  for (int q = 0; q < 3; ++q)
    if (q < dn)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * drow(q) + 4 * r + lq, k = 16 * dcol(q) + l16;
        if (m < jb && k < jb) At(i, i)[(long long)m * p.ld + k] = dc[q][r];
      }
}

// What the next launch's first task would otherwise have to begin with, rows 32 h .. of the tile: both panels' part of
// A(t+2, t+1), for which L(t+2, t) is formed once more (these rows), and L(t+1, t).
__device__ __forceinline__ void step_ahead(const StepP& p, StepShared& sh, int h) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = 32 * h + (wave >> 1) * 16, wn = (wave & 1) * 32, half = wave & 1;
  const int l16 = lane & 15, lq = lane >> 4;
  const int t = p.t, i = t + 2, rows = p.n - i * NB;
  auto At = [&](int r, int c) { return p.A + (long long)r * NB * p.ld + (long long)c * NB; };
  const double* inv_t = p.V + (long long)t * NB * (p.ldv + 1);
  TileRegs ra, rb;
  doublex4 acc[1][2], acc2[1][2], c[1][2], lx[2][2];
  zero_acc(acc2);
  if (t == 0) {
    ra.load(At(i, t), p.ld, rows, NB);
    rb.load(inv_t, p.ldv, NB, NB);
    ra.store_kc(sh.a);
    rb.store_kc(sh.b);
  } else {
    ra.load(At(i, t - 1), p.ld, rows, NB);
    rb.load(near_l(p, t - 1, 0), NB, NB, NB);
    load_acc(At(i, t), p.ld, rows, NB, wm, wn, lane, c);
    ra.store_kc(sh.a);
    rb.store_kc(sh.b);
    lds_barrier();
    ra.load(near_l(p, t - 1, 1), NB, NB, NB);
    rb.load(inv_t, p.ldv, NB, NB);
    zero_acc(acc);
    tile_mma<true>(sh.a, sh.b, wm, wn, lane, acc);
    lds_barrier();
    ra.store_kc(sh.b);
    lds_barrier();
    tile_mma<true>(sh.a, sh.b, wm, wn, lane, acc2);
    lds_barrier();
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) sh.a[kc_off<NB>(wn + 16 * j + l16, wm + 4 * r + lq)] = c[0][j][r] - acc[0][j][r];
    rb.store_kc(sh.b);
  }
  ra.load(At(t + 1, t), p.ld, NB, NB);
  load_acc(At(i, t + 1), p.ld, rows, NB, wm, wn, lane, c);
  lds_barrier();
  mma_lower_t(sh.a, sh.b, wm, half, lane, acc);
  lds_barrier();
  ra.store_kc(sh.a);
  lds_barrier();
  mma_lower_t(sh.a, sh.b, (wave >> 1) * 32, half, lane, lx);
  lds_barrier();
  put_kc_tri(sh.a, wm, half, lane, acc);
  put_kc_tri(sh.b, (wave >> 1) * 32, half, lane, lx);
  lds_barrier();
  tile_mma<true>(sh.a, sh.b, wm, wn, lane, acc2);
#pragma unroll
  for (int j = 0; j < 2; ++j) c[0][j] -= acc2[0][j];
  store_acc(At(i, t + 1), p.ld, rows, NB, wm, wn, lane, c);
}

// tiles of TA, and of TA and TV, in launch t of a chain of N tiles
__host__ __device__ static inline int step_ta_tiles(int N, int t) {
  const int m = N - 1 - t;                       // tile rows (and columns of A) behind column t
  return t > 0 && m > 1 ? m * (m - 1) / 2 - 1 : 0;      // without (t + 2, t + 1), the first of the enumeration
}
__host__ __device__ static inline int step_tiles(int N, int t) { return step_ta_tiles(N, t) + (N - 1 - t) * t; }
__global__ __launch_bounds__(256, 2) void chol_step_kernel(const StepP p) {
  __shared__ __attribute__((aligned(16))) StepShared sh;
  int b = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const int n = p.n, N = p.N, t = p.t;
  auto rows_of = [&](int i) { return n - i * NB; };
  auto At = [&](int i, int k) { return p.A + (long long)i * NB * p.ld + (long long)k * NB; };
  auto Vt = [&](int i, int k) { return p.V + (long long)i * NB * p.ldv + (long long)k * NB; };
  const int nP = N - 1 - t;
  if (b < nP) {
    if (b == 0) step_panel<true>(p, sh, t + 1);
    else step_panel<false>(p, sh, t + 1 + b);
    return;
  }
  b -= nP;
  if (nP > 1) {
    if (b < 2) {
      step_ahead(p, sh, b);
      return;
    }
    b -= 2;
  }
  doublex4 acc[2][2], c[2][2];
  zero_acc(acc);
  zero_acc(c);
  TileRegs ra, rb;
  if (b < t) {                                                        // ---- R(c)
    const int cc = b;
    ra.load(near_l(p, t - 1, 0), NB, NB, NB);
    rb.load(Vt(t - 1, cc), p.ldv, NB, NB);
    if (cc < t - 1) load_acc(Vt(t, cc), p.ldv, rows_of(t), NB, wm, wn, lane, c);
    ra.store_kc(sh.a);
    rb.store_rc(sh.b);
    lds_barrier();
    ra.load(Vt(t, t), p.ldv, rows_of(t), rows_of(t));
    tile_mma<false>(sh.a, sh.b, wm, wn, lane, acc);
    lds_barrier();
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          sh.b[rc_off<NB>(wm + 16 * ii + 4 * r + (lane >> 4), wn + 16 * j + (lane & 15))] = c[ii][j][r] - acc[ii][j][r];
    ra.store_kc(sh.a);
    lds_barrier();
    mma_lower(sh.a, sh.b, wave >> 1, wn, lane, acc);
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = 16 * tri_tile(wave >> 1, ii) + 4 * r + (lane >> 4);
          if (m < rows_of(t)) Vt(t, cc)[(long long)m * p.ldv + wn + 16 * j + (lane & 15)] = acc[ii][j][r];
        }
    return;
  }
  b -= t;
  // what is left goes to each workgroup `each` tiles at a time
  const int nTA = step_ta_tiles(N, t), total = step_tiles(N, t);
  for (int e = b * p.each, e1 = e + p.each < total ? e + p.each : total; e < e1; ++e) {
    if (e > b * p.each) {
      lds_barrier();
      zero_acc(acc);
      zero_acc(c);
    }
    if (e < nTA) {                                                    // ---- TA(i, k)
      int i = (int)((__builtin_sqrtf(8.0f * (float)(e + 1) + 1.0f) - 1.0f) * 0.5f);
      while (i * (i + 1) / 2 > e + 1) --i;
      while ((i + 1) * (i + 2) / 2 <= e + 1) ++i;
      i = __builtin_amdgcn_readfirstlane(i);
      const int k = e + 1 - i * (i + 1) / 2 + t + 1;
      i += t + 2;
      ra.load(At(i, t - 1), p.ld, rows_of(i), NB);
      if (k == t + 1) rb.load(near_l(p, t - 1, 1), NB, NB, NB);
      else rb.load(At(k, t - 1), p.ld, NB, NB);
      load_acc(At(i, k), p.ld, rows_of(i), NB, wm, wn, lane, c);
      ra.store_kc(sh.a);
      rb.store_kc(sh.b);
      lds_barrier();
      tile_mma<true>(sh.a, sh.b, wm, wn, lane, acc);
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int j = 0; j < 2; ++j) c[ii][j] -= acc[ii][j];
      store_acc(At(i, k), p.ld, rows_of(i), NB, wm, wn, lane, c);
    } else {                                                          // ---- TV(i, c)
      const int i = t + 1 + (e - nTA) / t, cc = (e - nTA) % t;
      if (i == t + 1) ra.load(near_l(p, t - 1, 1), NB, NB, NB);
      else ra.load(At(i, t - 1), p.ld, rows_of(i), NB);
      rb.load(Vt(t - 1, cc), p.ldv, NB, NB);
      if (cc < t - 1) load_acc(Vt(i, cc), p.ldv, rows_of(i), NB, wm, wn, lane, c);
      ra.store_kc(sh.a);
      rb.store_rc(sh.b);
      lds_barrier();
      tile_mma<false>(sh.a, sh.b, wm, wn, lane, acc);
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int j = 0; j < 2; ++j) c[ii][j] -= acc[ii][j];
      store_acc(Vt(i, cc), p.ldv, rows_of(i), NB, wm, wn, lane, c);
    }
  }
}

// First launch of the chain: block 0 factors diagonal tile 0, the next `clear` ones clear the tiles of Linv above the
// diagonal, and what is left of the chip streams the ride-along job.
__global__ __launch_bounds__(256, 2) void chol_begin_kernel(const StepP p, int clear, const CoJob job) {
  __shared__ __attribute__((aligned(16))) StepShared sh;
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    const int jb = p.n < NB ? p.n : NB;
    const int k = tid & 63;
    put_eye(sh, tid);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int i = (tid >> 6) + 4 * q;
      const bool in = i < jb && k <= i;
      const double v = p.A[in ? (long long)i * p.ld + k : 0];
      sh.b[i * SL + k] = in ? v : (i == k ? 1.0 : 0.0);
    }
    lds_barrier();
    diag_block<false>(sh, tid, p.V, p.ldv, jb, p.status,
               [&](int, int i, int c) {
                 doublex4 v;
#pragma unroll
                 for (int r = 0; r < 4; ++r) v[r] = sh.b[(16 * i + 4 * r + (tid >> 4 & 3)) * SL + 16 * c + (tid & 15)];
                 return v;
               },
               [] {});
    return;
  }
  if ((int)blockIdx.x > clear) {
    cojob_run(job, blockIdx.x - 1 - clear, gridDim.x - 1 - clear);
    return;
  }
  const int nt = p.N * (p.N - 1) / 2;
  for (int e = (int)blockIdx.x - 1; e < nt; e += clear) {
    int c = (int)((__builtin_sqrtf(8.0f * (float)e + 1.0f) - 1.0f) * 0.5f);      // tile (r, c + 1), r <= c
    while (c * (c + 1) / 2 > e) --c;
    while ((c + 1) * (c + 2) / 2 <= e) ++c;
    const int r0 = (e - c * (c + 1) / 2) * NB, col = (c + 1) * NB + (tid & 63);
    if (col < p.n)
      for (int r = r0 + (tid >> 6); r < r0 + NB; r += 4) p.V[(long long)r * p.ldv + col] = 0.0;
  }
}

// Linv [n x n, ldv] = L^-1 of A = L L^T (lower part of A [n x n, ld], destroyed); upper part of Linv zero.
// sub: chol_scratch_elems(n) doubles of scratch.  ld and ldv even, A and Linv 16-byte aligned.
strp_status chol_inverse(strp_ctx* ctx, double* A, int n, long long ld, double* sub, double* Linv, long long ldv, int32_t* status) {
  if (!aligned_vec(A, ld) || !aligned_vec(Linv, ldv)) return fail(ctx, STRP_EINVAL, "chol_inverse: operands not 16-byte aligned or odd leading dimension");
  CoJob job;
  memset(&job, 0, sizeof(job));
  if (ctx->cojob) job = *ctx->cojob;
  ctx->cojob = nullptr;
  const double pass_bytes = (job.Z0 ? 16.0 : 12.0) * (double)job.nrows * (double)job.T;
  ProfScope ps(ctx, "chol_factor_f64", 2.0 * (double)n * n * n / 3.0, 16.0 * (double)n * n + pass_bytes);
  if (chol_flow_ok(n, pass_bytes)) return chol_flow(ctx, A, n, ld, Linv, ldv, status, job);
  StepP p;
  memset(&p, 0, sizeof(p));
  p.A = A; p.ld = ld; p.V = Linv; p.ldv = ldv; p.sub = sub; p.n = n; p.N = (n + NB - 1) / NB; p.status = status;
  const int nt = p.N * (p.N - 1) / 2;
  const int clear = nt < 1024 ? nt : 1024;
  const unsigned int ride = job.units < 510u ? job.units : 510u;      // two workgroups of this kernel per CU, one place left to block 0
  hipLaunchKernelGGL(chol_begin_kernel, dim3(1 + clear + ride), dim3(256), 0, ctx->stream, p, clear, job);
  for (int t = 0; t < p.N; ++t) {
    p.t = t;
    const int m = p.N - 1 - t;
    // up to three tiles each, so that a launch of few tiles leaves the critical workgroup a CU of its own; beyond 576
    // tiles the launch is theirs and a workgroup that takes several only ends later.  One tile each / up to three below 577 / up to
    // three below 1025, us for the whole chain of 4096: 1851 / 1835 / 1876
    const int total = step_tiles(p.N, t);
    p.each = (total + 191) / 192;
    if (p.each > 3 || p.each < 1) p.each = 1;
    const int blocks = m + (m > 1 ? 2 : 0) + t + (total + p.each - 1) / p.each;
    if (blocks > 0) hipLaunchKernelGGL(chol_step_kernel, dim3(blocks), dim3(256), 0, ctx->stream, p);      // none: a single tile, the first launch was all
  }
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// tmp[m, j] = sum_{k <= j} X[m, k] Linv[j, k], then result[m, j] = sum_{k >= j} tmp[m, k] Linv[k, j]
static void solve_products(const SolveIn& in, DgemmP (&p)[2]) {
  memset(p, 0, sizeof(p));
  for (int i = 0; i < 2; ++i) {
    p[i].M = in.m; p[i].N = in.n; p[i].K = in.n;
    p[i].A = i ? in.tmp : in.X; p[i].lda = in.ldx; p[i].B = in.Linv; p[i].ldb = in.ldl; p[i].tri = 1 + i;
  }
  p[0].C = in.tmp; p[0].ldc = in.ldx;
  p[1].w = in.out;
}

// algorithmic bytes of a solve: L^-1 once, X and the result of either product written and read once
static double solve_bytes(int m, int n) { return 8.0 * ((double)n * n + 4.0 * (double)m * n); }

strp_status apply_inverse_right(strp_ctx* ctx, const double* Linv, int n, long long ldl, const double* X, int m, long long ldx, double* tmp,
                                const WeightsOut& out) {
  ProfScope ps(ctx, "chol_solve_f64", 2.0 * (double)m * n * n, solve_bytes(m, n));
  DgemmP p[2];
  solve_products(SolveIn{Linv, n, ldl, X, m, ldx, tmp, out}, p);
  STRP_TRY((dgemm_launch<true, true>(ctx, p[0])));
  return dgemm_launch<true, false>(ctx, p[1]);
}

// Two solves side by side pay where each has no more than a workgroup a compute unit: one takes as long as the longest tile then
// (64 x 128 beside 128 x 64: 15.8 + 13.5 us one after the other, 17.4 together).  A whole step, the solves apart / together,
// d x kept units (tiles of either): 64 x 128 182 / 174 us;  256 x 512 (64) 364 / 345;  384 x 768 (144) 478 / 456;  512 x 512 (128) 445 / 416;
// 64 x 1000 (32) 434 / 423;  512 x 1000 (256) 607 / 583.  The line is where this argument ends and not
// the gain: 720 x 720 (276) 615 / 592, 768 x 1000 (384) 696 / 661, 1000 x 1000 (512) 800 / 773 if it were further up.
bool solve_is_small(int m, int n) {
  return dgemm_tile(m, n, 0).tn == 32 && dgemm_blocks(m, n, {64, 32}) <= 256;
}
strp_status apply_inverse_right_pair(strp_ctx* ctx, const SolveIn& a, const SolveIn& b) {
  if (!solve_is_small(a.m, a.n) || !solve_is_small(b.m, b.n)) return fail(ctx, STRP_EINVAL, "two solves in one launch: not small");
  ProfScope ps(ctx, "chol_solve_f64", 2.0 * ((double)a.m * a.n * a.n + (double)b.m * b.n * b.n), solve_bytes(a.m, a.n) + solve_bytes(b.m, b.n));
  DgemmP p[2], q[2];
  solve_products(a, p);
  solve_products(b, q);
  const int first = dgemm_blocks(a.m, a.n, {64, 32}), blocks = first + dgemm_blocks(b.m, b.n, {64, 32});
  const DgemmPair g0{{p[0], q[0]}, first}, g1{{p[1], q[1]}, first};
  hipLaunchKernelGGL((dgemm_pair_kernel<64, 32, 32, true, true>), dim3(blocks), dim3(512), 0, ctx->stream, g0);
  hipLaunchKernelGGL((dgemm_pair_kernel<64, 32, 32, true, false>), dim3(blocks), dim3(512), 0, ctx->stream, g1);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---------------------------------------------------------------------------------------------
// casts, scatter, fill
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void f32_to_f64_ridge_kernel(const float* Af, long long ldf, double* Ad, long long ld, int n,
                                                               double lam, const double* lam_dev) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)n * n) return;
  const int i = (int)(e / n), j = (int)(e % n);
  double v = (double)Af[(long long)i * ldf + j];
  if (i == j) v += lam_dev ? *lam_dev : lam;
  if (i < NB && j >= NB) v = 0.0;      // as chol_inverse wants it
  Ad[(long long)i * ld + j] = v;
}

strp_status f32_to_f64_ridge(strp_ctx* ctx, const float* Af, long long ldf, double* Ad, long long ld, int n, double lam,
                             const double* lam_dev) {
  const long long tot = (long long)n * n;
  hipLaunchKernelGGL(f32_to_f64_ridge_kernel, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, ctx->stream, Af, ldf,
                     Ad, ld, n, lam, lam_dev);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

__global__ __launch_bounds__(256) void copy_f64_kernel(const double* src, long long lds, double* dst, long long ldd, int n) {
  const long long e = (long long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long long)n * n) return;
  const int i = (int)(e / n), j = (int)(e % n);
  dst[(long long)i * ldd + j] = src[(long long)i * lds + j];
}

strp_status copy_f64(strp_ctx* ctx, const double* src, long long lds, double* dst, long long ldd, int n) {
  hipLaunchKernelGGL(copy_f64_kernel, dim3((unsigned)(((long long)n * n + 255) / 256)), dim3(256), 0, ctx->stream, src, lds, dst, ldd, n);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// The compact weights of an earlier refit, with what apply_inverse_right would have left beside them.
__global__ __launch_bounds__(256) void gather_weights_kernel(const WeightsOut w, int m, int n) {
  double big = 0.0, sq = 0.0;
  for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < (long long)m * n; e += (long long)gridDim.x * 256) {
    const int i = (int)(e / n), j = (int)(e % n);
    const float v = w.side == STRP_SIDE_FC2 ? w.W[(long long)i * w.ldw + w.idx[j]] : w.W[(long long)w.idx[i] * w.ldw + j];
    w.Wc[(long long)i * w.ldc + j] = v;
    big = fmax(big, fabs((double)v));
    sq = __builtin_fma((double)v, (double)v, sq);
  }
  __shared__ double red[4][2];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    big = fmax(big, __shfl_down(big, o, 64));
    sq += __shfl_down(sq, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6][0] = big;
    red[threadIdx.x >> 6][1] = sq;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (w.maxbits) atomicMax(w.maxbits, __builtin_bit_cast(unsigned int, (float)fmax(fmax(red[0][0], red[1][0]), fmax(red[2][0], red[3][0]))));
    if (w.sumsq) w.sumsq[blockIdx.x] = red[0][1] + red[1][1] + red[2][1] + red[3][1];
  }
}
int gather_blocks(int m, int n) {
  const long long b = ((long long)m * n + 1023) / 1024;
  return b > 1024 ? 1024 : (int)b;
}
strp_status gather_weights(strp_ctx* ctx, const WeightsOut& io, int m, int n) {
  hipLaunchKernelGGL(gather_weights_kernel, dim3(gather_blocks(m, n)), dim3(256), 0, ctx->stream, io, m, n);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

__global__ __launch_bounds__(256) void fill_zero_kernel(const FillRanges f) { fill_block(f, blockIdx.x, gridDim.x); }

strp_status fill_ranges(strp_ctx* ctx, const FillRange* ranges, int n, FillRanges* f, long long* most) {
  memset(f, 0, sizeof(*f));
  *most = 0;
  for (int i = 0; i < n; ++i) {
    if (ranges[i].bytes % 4 != 0) return fail(ctx, STRP_EINVAL, "fill_zero: size not a multiple of 4");
    f->p[i] = (uint32_t*)ranges[i].ptr;
    f->words[i] = (long long)(ranges[i].bytes / 4);
    *most = f->words[i] > *most ? f->words[i] : *most;
  }
  return STRP_OK;
}
strp_status fill_zero(strp_ctx* ctx, const FillRange* ranges, int n) {
  FillRanges f;
  long long most;
  STRP_TRY(fill_ranges(ctx, ranges, n, &f, &most));
  if (most == 0) return STRP_OK;
  long long blocks = (most + 1023) / 1024;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, ctx->stream, f);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}
strp_status fill_zero(strp_ctx* ctx, void* ptr, size_t bytes) {
  const FillRange r{ptr, bytes};
  return fill_zero(ctx, &r, 1);
}

}  // namespace strp
