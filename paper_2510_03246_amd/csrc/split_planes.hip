// Split kernels: fp32 / bf16 / fp64 sources -> fp16 operand planes in the panel-major chunk layout
//   offset(k, r) = (((r / 128) * KG + k / 8) * 128 + r % 128) * 8 + k % 8
// (see gemm_mfma.hip).  All padding (rows up to a full panel, k up to a full group) is written as zero.
#include "splitk_reduce.h"
#include "strp_internal.h"

namespace strp {

__device__ __forceinline__ unsigned short sp_half_bits(float x) {
  _Float16 h = (_Float16)x;
  return __builtin_bit_cast(unsigned short, h);
}
__device__ __forceinline__ void sp_split_half(float x, unsigned short& hi, unsigned short& lo) {
  x = __builtin_fminf(__builtin_fmaxf(x, -65504.0f), 65504.0f);
  _Float16 h = (_Float16)x;
  hi = __builtin_bit_cast(unsigned short, h);
  lo = sp_half_bits(x - (float)h);
}
__device__ __forceinline__ unsigned int sp_pack2(unsigned short a, unsigned short b) {
  return (unsigned int)a | ((unsigned int)b << 16);
}

// Activations [rows x T] (optionally gathered by idx) -> planes.  Both kernels read the source row-contiguously
// and write whole contiguous kilobytes per wavefront store (a 16-byte chunk per lane, consecutive lanes =
// consecutive chunks): partial-line stores cost twice the HBM write traffic.
//   T-planes (contraction over tokens,   k = token,   r = channel row): [ceil(rows/128)][KG(T)][128][8]
//   C-planes (contraction over channels, k = channel, r = token):       [ceil(T/128)][KG(rows)][128][8]
// sixteen bytes of a row: four fp32 or eight bf16 tokens
template <bool SRC_BF16>
__device__ __forceinline__ void load16(const void* src, long long off, float (&v)[SRC_BF16 ? 8 : 4]) {
  if constexpr (SRC_BF16) {
    const uint4 w = *(const uint4*)((const unsigned short*)src + off);
    const unsigned int u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[2 * q] = __builtin_bit_cast(float, u[q] << 16);
      v[2 * q + 1] = __builtin_bit_cast(float, u[q] & 0xffff0000u);
    }
  } else {
    const float4 a = *(const float4*)((const float*)src + off);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  }
}

// T-planes: one block = one 128-row panel x 64 tokens (8 k-groups).  Phase 1 reads 16 bytes per lane (fp32: 16 lanes cover
// the 64 tokens of a row, a wavefront 4 rows; bf16: 8 lanes, 8 rows, a lane's eight tokens are a chunk) and drops the fp16 halves
// into an LDS image of the output ([k-group][row][8], k-groups padded by one chunk against bank conflicts); phase 2 copies the
// image out linearly: the block's output is one contiguous 16 KB run per plane.  A bf16 source has one plane and so one
// image, and twice the blocks per CU: 832 gathered rows of 65536 tokens 81 -> 44 us (4.9 TB/s).
// WITH_C: the same pass also writes the C-planes of the block's 128 rows x 64 tokens from the LDS image (a chunk = one
// token's 8 consecutive rows, gathered as 2-byte reads; a wavefront stores 64 consecutive tokens of one row group =
// 1 KB contiguous).  relu_c on top of an image without relu: relu(x) has the planes of x where hi is not negative
// and zero planes elsewhere (hi carries the sign of x, also when it rounds to zero).
constexpr int SPLIT_GP = 128 * 16 + 16;   // bytes per k-group in LDS
template <bool SRC_BF16, bool WITH_C>
__device__ __forceinline__ void split_t_block(unsigned char* sh, unsigned char* sl, const void* src, long long lds, const int* idx, int rows, long long T,
                                              int relu, unsigned short* t_hi, unsigned short* t_lo, long long TGa,
                                              int relu_c, unsigned short* c_hi, unsigned short* c_lo, int KGc, int32_t* status) {
  constexpr int GP = SPLIT_GP;
  constexpr int NT = SRC_BF16 ? 8 : 4, NR = 128 * 64 / 256 / NT;      // tokens of a row per lane and rows per lane
  bool bad = false;                   // a value the fp16 planes cannot hold: NaN, Inf or |x| > 65504
  const int t = threadIdx.x, piece = t & (64 / NT - 1), rsub = t / (64 / NT);
  const int pan = blockIdx.y;
  const long long tg0 = (long long)blockIdx.x * 8;
  const long long tok = tg0 * 8 + piece * NT;
  // clamped addresses (the source's pitch is a multiple of eight): a load under a condition waits for its row's index before the next one is
  // asked for (both refits' planes of 128 rows over 512 tokens 8.0 / 6.4 us)
  float v[NR][NT];
  int srow[NR];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int row = pan * 128 + rsub + 128 / NR * i;
    srow[i] = row < rows ? row : rows - 1;
  }
  if (idx)
#pragma unroll
    for (int i = 0; i < NR; ++i) srow[i] = idx[srow[i]];
#pragma unroll
  for (int i = 0; i < NR; ++i) load16<SRC_BF16>(src, (long long)srow[i] * lds + (tok < T ? tok : 0), v[i]);
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int rr = rsub + 128 / NR * i;
    const long long end = pan * 128 + rr < rows ? T : 0;
    unsigned short h[NT], l[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) {
      float x = tok + c < end ? v[i][c] : 0.0f;
      bad |= !(__builtin_fabsf(x) <= 65504.0f);
      if (relu) x = __builtin_fmaxf(x, 0.0f);
      sp_split_half(x, h[c], l[c]);
    }
    if constexpr (SRC_BF16) {
      *(uint4*)(sh + piece * GP + rr * 16) = make_uint4(sp_pack2(h[0], h[1]), sp_pack2(h[2], h[3]), sp_pack2(h[4], h[5]), sp_pack2(h[6], h[7]));
    } else {
      const int o = (piece >> 1) * GP + rr * 16 + (piece & 1) * 8;
      *(uint2*)(sh + o) = make_uint2(sp_pack2(h[0], h[1]), sp_pack2(h[2], h[3]));
      if (t_lo) *(uint2*)(sl + o) = make_uint2(sp_pack2(l[0], l[1]), sp_pack2(l[2], l[3]));
    }
  }
  if (bad) atomicCAS(status, 0, (int32_t)STRP_ENONFINITE);
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int c = t + 256 * j, g = c >> 7, rr = c & 127;
    if (tg0 + g >= TGa) continue;
    const long long o = (((long long)pan * TGa + tg0 + g) * 128 + rr) * 8;
    *(uint4*)(t_hi + o) = *(const uint4*)(sh + g * GP + rr * 16);
    if (!SRC_BF16 && t_lo) *(uint4*)(t_lo + o) = *(const uint4*)(sl + g * GP + rr * 16);
  }
  if (WITH_C) {
    const long long tok_c = tg0 * 8 + (t & 63);                  // this thread's token
    if (tok_c < (((T + 127) >> 7) << 7)) {                        // inside the last token panel
      const int tl = t & 63;
      const unsigned char* bh = sh + (tl >> 3) * GP + (tl & 7) * 2;
      const unsigned char* bl = sl + (tl >> 3) * GP + (tl & 7) * 2;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int g = (t >> 6) + 4 * j;                           // row group of the panel (8 rows)
        const int rg = pan * 16 + g;
        if (rg >= KGc) continue;
        unsigned short h[8], l[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          h[r] = *(const unsigned short*)(bh + (g * 8 + r) * 16);
          l[r] = !SRC_BF16 && c_lo ? *(const unsigned short*)(bl + (g * 8 + r) * 16) : (unsigned short)0;
          if (relu_c && (h[r] & 0x8000u)) h[r] = l[r] = 0;
        }
        const long long o = (((tok_c >> 7) * KGc + rg) * 128 + (tok_c & 127)) * 8;
        *(uint4*)(c_hi + o) = make_uint4(sp_pack2(h[0], h[1]), sp_pack2(h[2], h[3]), sp_pack2(h[4], h[5]), sp_pack2(h[6], h[7]));
        if (!SRC_BF16 && c_lo) *(uint4*)(c_lo + o) = make_uint4(sp_pack2(l[0], l[1]), sp_pack2(l[2], l[3]), sp_pack2(l[4], l[5]), sp_pack2(l[6], l[7]));
      }
    }
  }
}

template <bool SRC_BF16, bool WITH_C>
__global__ __launch_bounds__(256) void split_t_kernel(const void* src, long long lds, const int* idx, int rows, long long T,
                                                      int relu, unsigned short* t_hi, unsigned short* t_lo, long long TGa,
                                                      int relu_c, unsigned short* c_hi, unsigned short* c_lo, int KGc,
                                                      int32_t* status) {
  __shared__ __attribute__((aligned(16))) unsigned char sh[8 * SPLIT_GP];
  __shared__ __attribute__((aligned(16))) unsigned char sl[SRC_BF16 ? 16 : 8 * SPLIT_GP];
  split_t_block<SRC_BF16, WITH_C>(sh, sl, src, lds, idx, rows, T, relu, t_hi, t_lo, TGa, relu_c, c_hi, c_lo, KGc, status);
}
// The same rows of two fp32 matrices, as the refits of a small module need them: blockIdx.z = 0 the T-planes of a, 1 the T-planes
// of z and the C-planes of relu(z); from 2 on, the step's clearing.
__global__ __launch_bounds__(256) void split_t_pair_kernel(const float* a, const float* z, long long lds, const int* idx, int rows, long long T,
                                                           unsigned short* a_hi, unsigned short* a_lo, unsigned short* z_hi, unsigned short* z_lo,
                                                           long long TGa, unsigned short* c_hi, unsigned short* c_lo, int KGc, int32_t* status,
                                                           const FillRanges clear) {
  __shared__ __attribute__((aligned(16))) unsigned char sh[8 * SPLIT_GP];
  __shared__ __attribute__((aligned(16))) unsigned char sl[8 * SPLIT_GP];
  if (blockIdx.z >= 2) fill_block(clear, ((blockIdx.z - 2) * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, (gridDim.z - 2) * gridDim.y * gridDim.x);
  else if (blockIdx.z == 0) split_t_block<false, false>(sh, sl, a, lds, idx, rows, T, 0, a_hi, a_lo, TGa, 0, nullptr, nullptr, 0, status);
  else split_t_block<false, true>(sh, sl, z, lds, idx, rows, T, 0, z_hi, z_lo, TGa, 1, c_hi, c_lo, KGc, status);
}

// C-planes: thread = token, a chunk is that token's 8 consecutive channels; one block covers 256 tokens x 32
// channels (4 k-groups).  Every load of a row is 1 KB contiguous per wavefront, every store 1 KB contiguous.
template <bool SRC_BF16>
__global__ __launch_bounds__(256) void split_c_kernel(const void* src, long long lds, const int* idx, int rows, long long T,
                                                      int relu, unsigned short* c_hi, unsigned short* c_lo, int KGa,
                                                      int32_t* status) {
  const long long tok = (long long)blockIdx.x * 256 + threadIdx.x;
  const int rg0 = blockIdx.y * 4;
  if (tok >= (((T + 127) >> 7) << 7)) return;   // past the last token panel
  bool bad = false;
  float v[4][8];
#pragma unroll
  for (int g = 0; g < 4; ++g)
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int row = (rg0 + g) * 8 + r;
      float x = 0.0f;
      if (row < rows && tok < T) {
        const long long srow = idx ? (long long)idx[row] : (long long)row;
        if (SRC_BF16) x = __builtin_bit_cast(float, (unsigned int)((const unsigned short*)src)[srow * lds + tok] << 16);
        else x = ((const float*)src)[srow * lds + tok];
      }
      bad |= !(__builtin_fabsf(x) <= 65504.0f);
      v[g][r] = relu ? __builtin_fmaxf(x, 0.0f) : x;
    }
  if (bad) atomicCAS(status, 0, (int32_t)STRP_ENONFINITE);
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    if (rg0 + g >= KGa) continue;
    unsigned short h[8], l[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) sp_split_half(v[g][r], h[r], l[r]);
    const long long o = (((tok >> 7) * KGa + rg0 + g) * 128 + (tok & 127)) * 8;
    *(uint4*)(c_hi + o) = make_uint4(sp_pack2(h[0], h[1]), sp_pack2(h[2], h[3]), sp_pack2(h[4], h[5]), sp_pack2(h[6], h[7]));
    if (c_lo) *(uint4*)(c_lo + o) = make_uint4(sp_pack2(l[0], l[1]), sp_pack2(l[2], l[3]), sp_pack2(l[4], l[5]), sp_pack2(l[6], l[7]));
  }
}

// Two passes that each leave most of the chip idle, in one launch: a model of two d = 64 layers 12.90 -> 12.50 ms, a step 197 -> 194 us.  With the
// clearing of the step's buffers in it as well: steps of 64 x 128 kept units over 512 tokens 150.8 -> 148.8 us, 200 x 400, 4000 302.7 -> 299.2, 768 x 600 of
// 3400, 768 (21 MB to clear) 474.7 -> 471.9.
strp_status split_act_pair(strp_ctx* ctx, const float* a, const float* z, long long lds, const int* idx, int rows, long long T, const PlaneOp& At,
                           const PlaneOp& Zt, const PlaneOp& Zc, const FillRange* clear) {
  if (rows <= 0 || T <= 0) return fail(ctx, STRP_EINVAL, "split_act: empty");
  if (!ctx->status_dev) return fail(ctx, STRP_ENOMEM, "split_act: no workspace set");
  if (lds % 8 || lds < T) return fail(ctx, STRP_EINVAL, "split_act: source pitch must be a multiple of 8 and at least T");
  ProfScope ps(ctx, "split_act", 0.0, (2.0 * 4.0 + 3.0 * (At.lo ? 4.0 : 2.0)) * (double)rows * (double)T);
  FillRanges f;
  long long most;
  STRP_TRY(fill_ranges(ctx, clear, 3, &f, &most));
  // both reach the end of the last 128-token panel (the C-planes' padding), which the T-planes end in
  const dim3 grid((unsigned)(2 * ((T + 127) / 128)), (unsigned)((rows + 127) / 128), 2);
  const long long layer = (long long)grid.x * grid.y, layers = ((most + 1023) / 1024 + layer - 1) / layer;      // a kilobyte of words a workgroup, as far as sixteen layers go
  hipLaunchKernelGGL(split_t_pair_kernel, dim3(grid.x, grid.y, 2 + (unsigned)(layers < 16 ? layers : 16)), dim3(256), 0, ctx->stream, a, z, lds, idx,
                     rows, T, (unsigned short*)At.hi, (unsigned short*)At.lo, (unsigned short*)Zt.hi, (unsigned short*)Zt.lo, plane_kg(T),
                     (unsigned short*)Zc.hi, (unsigned short*)Zc.lo, (int)plane_kg(rows), ctx->status_dev, f);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

strp_status split_act(strp_ctx* ctx, const void* src, int src_dtype, long long lds, const int* idx, int rows, long long T,
                      int relu_t, int relu_c, unsigned short* t_hi, unsigned short* t_lo, unsigned short* c_hi,
                      unsigned short* c_lo) {
  if (rows <= 0 || T <= 0) return fail(ctx, STRP_EINVAL, "split_act: empty");
  if (!ctx->status_dev) return fail(ctx, STRP_ENOMEM, "split_act: no workspace set");
  if (src_dtype == STRP_BF16 && (t_lo || c_lo)) return fail(ctx, STRP_EINVAL, "split_act: a bf16 source has one plane");
  if (lds % 8 || lds < T) return fail(ctx, STRP_EINVAL, "split_act: source pitch must be a multiple of 8 and at least T");
  const double es = src_dtype == STRP_BF16 ? 2.0 : 4.0;
  const double wb = (t_hi ? 2.0 : 0.0) + (t_lo ? 2.0 : 0.0) + (c_hi ? 2.0 : 0.0) + (c_lo ? 2.0 : 0.0);
  const bool one_read = t_hi && c_hi && (relu_t == relu_c || !relu_t) && (t_lo != nullptr) == (c_lo != nullptr);
  ProfScope ps(ctx, "split_act", 0.0, (es * (one_read ? 1.0 : (t_hi ? 1.0 : 0.0) + (c_hi ? 1.0 : 0.0)) + wb) * (double)rows * (double)T);
  // both layouts of the same rows in one pass over the source when the C-planes can be derived from the T image
  const bool fused = t_hi && c_hi && (relu_t == relu_c || !relu_t) && (t_lo != nullptr) == (c_lo != nullptr);
  if (t_hi) {
    const long long TGa = plane_kg(T);
    const int KGc = (int)plane_kg(rows);
    const int rc = fused ? (relu_c && !relu_t) : 0;
    // fused: the blocks reach the end of the last 128-token panel, whose padding the C-planes hold as zeros
    const long long gx = fused ? 2 * ((T + 127) / 128) : (TGa + 7) / 8;
    dim3 grid((unsigned)gx, (unsigned)((rows + 127) / 128));
    if (fused && src_dtype == STRP_BF16)
      hipLaunchKernelGGL((split_t_kernel<true, true>), grid, dim3(256), 0, ctx->stream, src, lds, idx, rows, T, relu_t, t_hi, t_lo, TGa, rc, c_hi, c_lo, KGc, ctx->status_dev);
    else if (fused)
      hipLaunchKernelGGL((split_t_kernel<false, true>), grid, dim3(256), 0, ctx->stream, src, lds, idx, rows, T, relu_t, t_hi, t_lo, TGa, rc, c_hi, c_lo, KGc, ctx->status_dev);
    else if (src_dtype == STRP_BF16)
      hipLaunchKernelGGL((split_t_kernel<true, false>), grid, dim3(256), 0, ctx->stream, src, lds, idx, rows, T, relu_t, t_hi, t_lo, TGa, 0,
                         (unsigned short*)nullptr, (unsigned short*)nullptr, 0, ctx->status_dev);
    else
      hipLaunchKernelGGL((split_t_kernel<false, false>), grid, dim3(256), 0, ctx->stream, src, lds, idx, rows, T, relu_t, t_hi, t_lo, TGa, 0,
                         (unsigned short*)nullptr, (unsigned short*)nullptr, 0, ctx->status_dev);
    STRP_HIP(ctx, hipGetLastError());
  }
  if (c_hi && !fused) {
    const int KGa = (int)plane_kg(rows);
    dim3 grid((unsigned)(((T + 127) / 128 * 128 + 255) / 256), (unsigned)((KGa + 3) / 4));
    if (src_dtype == STRP_BF16)
      hipLaunchKernelGGL((split_c_kernel<true>), grid, dim3(256), 0, ctx->stream, src, lds, idx, rows, T, relu_c, c_hi, c_lo, KGa, ctx->status_dev);
    else
      hipLaunchKernelGGL((split_c_kernel<false>), grid, dim3(256), 0, ctx->stream, src, lds, idx, rows, T, relu_c, c_hi, c_lo, KGa, ctx->status_dev);
    STRP_HIP(ctx, hipGetLastError());
  }
  return STRP_OK;
}

__device__ __forceinline__ double small_src(const double* s, long long i) { return s[i]; }
__device__ __forceinline__ double small_src(const float* s, long long i) { return (double)s[i]; }
__device__ __forceinline__ double small_src(const unsigned short* s, long long i) {
  return (double)__builtin_bit_cast(float, (unsigned int)s[i] << 16);
}


// Small matrices (weights): planes of src * scale, [ceil(rows/128)][plane_kg(cols)][128][8], zero padded.  A thread makes one
// 16-byte chunk (eight k of one row) of each plane, so stores are whole kilobytes per wavefront; sources that are
// stored along k are read 16 bytes at a time, the others (and a row's last entries) along consecutive rows.  Few bytes and one chunk a thread: what it takes beyond a launch is the chain from the arguments to the loads, so
// what a wavefront has in common stays in scalar registers (an entry of the job list picked per lane came from memory per lane).
// us: 1536 x 768 fp32 10.2 -> 7.8, both dense matrices of 768 x 3072 in bf16 18.4 -> 11.6, 768 x 1536 both ways 14.4 -> 11.3,
// 128 x 64 5.2 -> 4.4; fp64 768 x 768, of which the lower half is valid, 8.0 -> 8.1.
struct SplitJobs {
  SplitJob j[3];
  long long chunk0[4];      // first chunk of each job
};
template <typename TS>
__device__ __forceinline__ void split_chunk(const SplitJob& b, long long e, unsigned int pg) {
  const TS* src = (const TS*)b.src;
  const unsigned int KG = (unsigned int)plane_kg(b.cols);
  const int g = (int)(pg % KG), r = (int)(pg / KG) * 128 + (int)(e & 127);
  const double scale = b.maxbits ? (double)scale_of_max(*b.maxbits) : 1.0;
  double x[8];
  constexpr int PER = 16 / (int)sizeof(TS);
  // whole chunks of a row (an address of any alignment would do, but rows begin at multiples of 16 bytes: the entry points see to that)
  if (!b.transpose && g * 8 + 8 <= b.cols) {
    const TS* row = src + (long long)(r < b.rows ? r : b.rows - 1) * b.lds + g * 8;
    uint4 v[8 / PER];
#pragma unroll
    for (int q = 0; q < 8 / PER; ++q) v[q] = ((const uint4*)row)[q];
    TS w[8];
    __builtin_memcpy(w, v, sizeof(w));
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = small_src(w, j);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      // clamped addresses: the eight loads are unconditional and in flight together
      const int rc = r < b.rows ? r : b.rows - 1, c = g * 8 + j < b.cols ? g * 8 + j : b.cols - 1;
      const bool swap = b.transpose == 2 ? rc < c : b.transpose != 0;
      x[j] = small_src(src, swap ? (long long)c * b.lds + rc : (long long)rc * b.lds + c);
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (r >= b.rows || g * 8 + j >= b.cols) x[j] = 0.0;
  unsigned short h[8], l[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const double y = fmin(fmax(x[j] * scale, -65504.0), 65504.0);
    const _Float16 hh = (_Float16)y;
    h[j] = __builtin_bit_cast(unsigned short, hh);
    l[j] = __builtin_bit_cast(unsigned short, (_Float16)(y - (double)hh));
  }
  *(uint4*)(b.hi + e * 8) = make_uint4(sp_pack2(h[0], h[1]), sp_pack2(h[2], h[3]), sp_pack2(h[4], h[5]), sp_pack2(h[6], h[7]));
  if (b.lo) *(uint4*)(b.lo + e * 8) = make_uint4(sp_pack2(l[0], l[1]), sp_pack2(l[2], l[3]), sp_pack2(l[4], l[5]), sp_pack2(l[6], l[7]));
}
__device__ __forceinline__ void split_small_block(const SplitJobs& jobs) {
  // chunk counts are multiples of 128: a wavefront's chunks are of one job and one k-group
  const unsigned int half = 2 * blockIdx.x + __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
  const long long e0 = 128ll * half;
  if (e0 >= jobs.chunk0[3]) return;
  const int q = (e0 >= jobs.chunk0[1]) + (e0 >= jobs.chunk0[2]);
  const SplitJob& b = jobs.j[q];
  const unsigned int pg = half - (unsigned int)(jobs.chunk0[q] >> 7);
  const long long c = 128ll * pg + (threadIdx.x & 127);
  if (b.kind == SRC_F64) split_chunk<double>(b, c, pg);
  else if (b.kind == SRC_F32) split_chunk<float>(b, c, pg);
  else split_chunk<unsigned short>(b, c, pg);
}
__global__ __launch_bounds__(256) void split_small_kernel(const SplitJobs jobs) { split_small_block(jobs); }

static SplitJobs split_jobs(const SplitJob* jobs, int n) {
  SplitJobs s;
  memset(&s, 0, sizeof(s));
  for (int i = 0; i < 3; ++i) {
    if (i < n) s.j[i] = jobs[i];
    s.chunk0[i + 1] = s.chunk0[i] + (i < n ? (long long)plane_elems(jobs[i].rows, jobs[i].cols) / 8 : 0);
  }
  return s;
}
strp_status split_small(strp_ctx* ctx, const SplitJob* jobs, int n) {
  const SplitJobs s = split_jobs(jobs, n);
  hipLaunchKernelGGL(split_small_kernel, dim3((unsigned)((s.chunk0[3] + 255) / 256)), dim3(256), 0, ctx->stream, s);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// grid-wide max of |x| through an integer atomic on the float bits (order-preserving for x >= 0)
template <typename TS>
__device__ __forceinline__ float row_max(const TS* row, int cols) {
  float m = 0.0f;
  // eight independent loads per trip keep enough requests in flight for a latency-bound reduction
  int c = threadIdx.x;
  for (; c + 7 * 256 < cols; c += 8 * 256) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = (float)small_src(row, c + 256 * q);
#pragma unroll
    for (int q = 0; q < 8; ++q) m = __builtin_fmaxf(m, __builtin_fabsf(v[q]));
  }
  for (; c < cols; c += 256) m = __builtin_fmaxf(m, __builtin_fabsf((float)small_src(row, c)));
  return m;
}
struct MaxJobs {
  MaxJob j[2];
};
__global__ __launch_bounds__(256) void absmax_kernel(const MaxJobs jobs) {
  const MaxJob& b = jobs.j[blockIdx.y];
  float m = 0.0f;
  for (int r = blockIdx.x; r < b.rows; r += gridDim.x)       // a block walks whole rows: no division per element
    m = __builtin_fmaxf(m, b.kind == SRC_F32 ? row_max((const float*)b.src + (long long)r * b.lds, b.cols)
                                             : row_max((const unsigned short*)b.src + (long long)r * b.lds, b.cols));
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = __builtin_fmaxf(m, __shfl_down(m, o, 64));
  // one atomic per block: thousands of atomics on one address serialise in L2 and were the whole run time
  __shared__ float wm[4];
  if ((threadIdx.x & 63) == 0) wm[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = __builtin_fmaxf(__builtin_fmaxf(wm[0], wm[1]), __builtin_fmaxf(wm[2], wm[3]));
    if (m > 0.0f) atomicMax(b.maxbits, __builtin_bit_cast(unsigned int, m));
  }
}

strp_status abs_max(strp_ctx* ctx, const MaxJob* jobs, int n) {
  MaxJobs m;
  memset(&m, 0, sizeof(m));
  int rows = 1;
  for (int i = 0; i < n; ++i) {
    m.j[i] = jobs[i];
    rows = jobs[i].rows > rows ? jobs[i].rows : rows;
  }
  hipLaunchKernelGGL(absmax_kernel, dim3(rows < 512 ? rows : 512, n), dim3(256), 0, ctx->stream, m);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// ---------------------------------------------------------------------------------------------
// One fp16 plane with k = channel, r = token  ->  the same values as a plane with k = token, r = channel.
// A block moves 128 tokens x 128 channels: both its source (16 k-groups of one token panel) and its destination
// (16 k-groups of one channel panel) are contiguous 32 KB runs; the 2-byte transposition happens in LDS.
// Tokens >= T are written as zero (they are contraction padding on the output side).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void plane_c_to_t_block(const unsigned short* src, unsigned short* dst, long long T, long long kg_src, long long kg_dst, long long pt,
                                                   int pc) {
  constexpr int GS = 1024 + 8;                    // elements per source k-group in LDS (+16 B against bank conflicts)
  __shared__ __attribute__((aligned(16))) unsigned short sm[16 * GS];
  const int tid = threadIdx.x;
  // load: source k-groups 16 pc .. 16 pc + 15 (those below kg_src) of token panel pt
  for (int q = tid; q < 2048; q += 256) {
    const int g = q >> 7, piece = q & 127;        // 128 16-byte pieces (one token each) per k-group
    const long long cg = (long long)pc * 16 + g;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (cg < kg_src) v = *(const uint4*)(src + ((pt * kg_src + cg) * 128 + piece) * 8);
    *(uint4*)(sm + g * GS + piece * 8) = v;
  }
  __syncthreads();
  // store: destination k-groups 16 pt .. 16 pt + 15 (those below kg_dst) of channel panel pc
  for (int q = tid; q < 2048; q += 256) {
    const int tg = q >> 7, cl = q & 127;          // piece = channel cl, token group tg
    const long long tgg = pt * 16 + tg;
    if (tgg >= kg_dst) continue;
    const unsigned short* col = sm + (cl >> 3) * GS + (cl & 7);
    unsigned short e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const long long t = tgg * 8 + j;
      e[j] = t < T ? col[(tg * 8 + j) * 8] : (unsigned short)0;
    }
    uint4 v;
    v.x = e[0] | ((unsigned)e[1] << 16);
    v.y = e[2] | ((unsigned)e[3] << 16);
    v.z = e[4] | ((unsigned)e[5] << 16);
    v.w = e[6] | ((unsigned)e[7] << 16);
    *(uint4*)(dst + (((long long)pc * kg_dst + tgg) * 128 + cl) * 8) = v;
  }
}
__global__ __launch_bounds__(256) void plane_c_to_t_kernel(const unsigned short* src, unsigned short* dst, long long T, long long kg_src, long long kg_dst) {
  plane_c_to_t_block(src, dst, T, kg_src, kg_dst, blockIdx.x, blockIdx.y);        // token panel, channel panel
}

strp_status plane_c_to_t(strp_ctx* ctx, const unsigned short* src, unsigned short* dst, int C, long long T) {
  ProfScope ps(ctx, "plane_c_to_t", 0.0, 4.0 * (double)C * (double)T);
  dim3 grid((unsigned)((T + 127) / 128), (unsigned)((C + 127) / 128));
  hipLaunchKernelGGL(plane_c_to_t_kernel, grid, dim3(256), 0, ctx->stream, src, dst, T, plane_kg(C), plane_kg(T));
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// Planes of a small matrix with, in the same launch, what a small module's step has to do for its residual at that point: turn a plane of it, or
// sum a product's partials.  All of them are the time of a launch and of one workgroup (2.8 to 4.7 us each by itself).
__global__ __launch_bounds__(256) void split_turn_kernel(const SplitJobs jobs, int split_end, const unsigned short* src, unsigned short* dst, long long T, long long kg_src,
                                                         long long kg_dst, int panels) {
  const int b = (int)blockIdx.x - split_end, pc = b / panels;
  if (b < 0) split_small_block(jobs);
  else plane_c_to_t_block(src, dst, T, kg_src, kg_dst, b - pc * panels, pc);
}
strp_status split_small_turn(strp_ctx* ctx, const SplitJob& job, const unsigned short* src, unsigned short* dst, int C, long long T) {
  const SplitJobs s = split_jobs(&job, 1);
  const int split_end = (int)((s.chunk0[3] + 255) / 256), panels = (int)((T + 127) / 128);
  ProfScope ps(ctx, "plane_c_to_t", 0.0, 4.0 * (double)C * (double)T);
  hipLaunchKernelGGL(split_turn_kernel, dim3(split_end + panels * ((C + 127) / 128)), dim3(256), 0, ctx->stream, s, split_end, src, dst, T, plane_kg(C), plane_kg(T), panels);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}
__global__ __launch_bounds__(256) void split_reduce_kernel(const SplitJobs jobs, int split_end, const ReduceP r) {
  const int b = (int)blockIdx.x - split_end, nx = (r.N + REDUCE_TILE_N - 1) / REDUCE_TILE_N;
  if (b < 0) split_small_block(jobs);
  else splitk_reduce_block(r, b % nx, b / nx, nx);
}
strp_status split_small_reduce(strp_ctx* ctx, const SplitJob& job, const ReduceP& r) {
  const SplitJobs s = split_jobs(&job, 1);
  const int split_end = (int)((s.chunk0[3] + 255) / 256);
  ProfScope ps(ctx, "splitk_reduce", 0.0, 2.0 * (double)r.splits * r.M * r.N);
  hipLaunchKernelGGL(split_reduce_kernel, dim3(split_end + reduce_blocks(r.M, r.N)), dim3(256), 0, ctx->stream, s, split_end, r);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

}  // namespace strp
