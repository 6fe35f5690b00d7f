// Factor and inverse factor of an SPD matrix in ONE launch.
//
// The matrix is cut into 64 x 64 tiles (N x N of them); workgroups take tasks from a counter, keep the tile they are making in
// registers, and wait in memory for the tiles it is made of.  One workgroup does nothing but the chain that everything
// else depends on, stage s = 0 .. N - 1:
//   L(s, s-1) = U(s, s-1) Linv(s-1, s-1)^T,  A(s, s) = U(s, s) - L(s, s-1) L(s, s-1)^T,  its factor and Linv(s, s)
// where U is A with the panels up to s - 2 applied.  Stage t of the tasks is what becomes possible once Linv(t, t) is there:
//   D(t + 2)   rows of tile row s = t + 2 for the chain: U(s, s-1) (two workgroups, 32 rows each), L(s, s-2) and U(s, s) (one)
//   G(i, t)    L(i, t), i > t + 2
//   V(t, c)    Linv(t, c) = -Linv(t, t) sum_j L(t, j) Linv(j, c), c < t
// The chain's workgroup runs its products and its pivots on four wavefronts; four others move its tiles.
#include "cojob.h"
#include "f64_tiles.h"

namespace strp {

// A task waits only for the chain and for tasks of smaller numbers, and numbers are given out in order to workgroups that run, so the
// lowest unfinished task never waits for anything that is not running: the launch ends whatever part of it the chip holds at a time.
// Should a wait outlast `limit` all the same, the launch gives up and says so in the status word.
struct FlowP {
  double* A; long long ld;         // L is left below the diagonal tiles
  double* V; long long ldv;        // Linv
  unsigned int* flags;             // counters, zero: lines of 64 bytes, 1 << row_lines of them in a row of the matrix
  int row_lines;
  int n, N;
  unsigned int tasks;              // besides the chain
  int lines_a, lines_v;            // no two tiles of the matrix share a cache line
  unsigned long long limit;        // of a wait, in ticks of the 100 MHz counter
  int32_t* status;
};

// Counters, a line each.  L(i, j) for j < i - 1 is finished when flow_l(i) > j; Linv(r, c), r > c, when flow_v(c) >= r.
constexpr int FLOW_COPIES = 8;     // of the chain's counters, which everybody reads: word 0: 4 for each Linv(t, t), word 1: 7 for each L(t, t-1)
__device__ __forceinline__ unsigned int* flow_line(const FlowP& p, int q) {
  return p.flags + 2 * (q >> p.row_lines) * p.ld + 16 * (q & ((1 << p.row_lines) - 1));
}
__device__ __forceinline__ unsigned int* flow_l(const FlowP& p, int i) { return flow_line(p, i); }
__device__ __forceinline__ unsigned int* flow_v(const FlowP& p, int c) { return flow_line(p, p.N + c); }
__device__ __forceinline__ unsigned int* flow_done(const FlowP& p, int s) { return flow_line(p, 2 * p.N + s); }     // halves of U(s, s-1); next word: U(s, s)
__device__ __forceinline__ unsigned int* flow_read(const FlowP& p, int s) { return flow_line(p, 3 * p.N + s); }     // ... that have read their part of A
__device__ __forceinline__ unsigned int* flow_chain(const FlowP& p, int copy) { return flow_line(p, 4 * p.N + copy); }
__device__ __forceinline__ unsigned int* flow_ticket(const FlowP& p) { return flow_line(p, 4 * p.N + FLOW_COPIES); }
__device__ __forceinline__ unsigned int* flow_unit(const FlowP& p) { return flow_line(p, 4 * p.N + FLOW_COPIES + 1); }
__device__ __forceinline__ unsigned int* flow_abort(const FlowP& p) { return flow_line(p, 4 * p.N + FLOW_COPIES + 2); }
static inline int flow_lines_needed(int N) { return 4 * N + FLOW_COPIES + 3; }

// What a wavefront waits for: up to three counters.  seen: the values they are known to have.
struct FlowWait {
  const unsigned int* word[3];
  unsigned int need[3], seen[3];
  __device__ __forceinline__ void set(int q, const unsigned int* w) { word[q] = w; seen[q] = need[q] = 0; }
  __device__ __forceinline__ bool ready() const { return seen[0] >= need[0] && seen[1] >= need[1] && seen[2] >= need[2]; }
};
// reads them once; -1: the launch has given up
__device__ __forceinline__ int flow_poll(const FlowP& p, FlowWait& w) {
  const int lane = threadIdx.x & 63;
  const unsigned int* q = lane == 0 ? w.word[0] : lane == 1 ? w.word[1] : lane == 2 ? w.word[2] : flow_abort(p);
  unsigned int v = 0;
  if (lane < 4) v = agent_get(q);
#pragma unroll
  for (int e = 0; e < 3; ++e) w.seen[e] = __builtin_amdgcn_readlane(v, e);
  const bool stop = __builtin_amdgcn_readlane(v, 3) != 0;
  asm volatile("" ::: "memory");          // what was waited for is read behind this
  return stop ? -1 : w.ready();
}
__device__ __forceinline__ bool flow_wait(const FlowP& p, FlowWait& w) {
  if (w.ready()) return true;
  unsigned long long t0 = 0;
  for (;;) {
    const int r = flow_poll(p, w);
    if (r) return r > 0;
    const unsigned long long now = wall_clock64();
    if (!t0) t0 = now;
    if (now - t0 > p.limit) {
      if ((threadIdx.x & 63) == 0) {
        agent_put(flow_abort(p), 1u);
        atomicCAS(p.status, 0, (int)STRP_EHIP);
      }
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}
__device__ __forceinline__ void flow_stored() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// rows [0, rv) and columns [0, cv) of a tile as a buffer: what lies past its last pair of elements reads as zero (ld is even)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t flow_buffer(const double* src, long long ld, int rv, int cv) {
  const int bytes = rv > 0 ? ((rv < NB ? rv : NB) - 1) * (int)ld * 8 + ((cv < NB ? cv : NB) + 1 & ~1) * 8 : 0;
  return __builtin_amdgcn_make_buffer_rsrc((void*)src, 0, bytes, 0x00027000);
}
// COHERENT: past the caches, like agent_get
template <bool COHERENT>
__device__ __forceinline__ doublex2 flow_get2(__amdgpu_buffer_rsrc_t buf, int off, int soff) {
  return __builtin_bit_cast(doublex2, __builtin_amdgcn_raw_buffer_load_b128(buf, off, soff, COHERENT ? 16 : 0));
}

// Tile rows of 64 columns by the 512 threads of a workgroup.  What another workgroup of the launch has written is read past the caches
// (coherent) where a line of it may have been read before, in its former state.
template <int ROWS>
struct FlowTile {
  static constexpr int NQ = ROWS / 16;
  doublex2 r[NQ];
  __device__ __forceinline__ void load(const double* src, long long ld, int rv, int cv, bool coherent) {
    const __amdgpu_buffer_rsrc_t buf = flow_buffer(src, ld, rv < ROWS ? rv : ROWS, cv);
    const int ch = threadIdx.x & 31, off = ((int)(threadIdx.x >> 5) * (int)ld + 2 * ch) * 8, step = 128 * (int)ld;
    if (coherent) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) r[q] = flow_get2<true>(buf, off, q * step);
    } else {
#pragma unroll
      for (int q = 0; q < NQ; ++q) r[q] = flow_get2<false>(buf, off, q * step);
    }
    if (cv < NB) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) r[q] = doublex2{2 * ch < cv ? r[q].x : 0.0, 2 * ch + 1 < cv ? r[q].y : 0.0};
    }
  }
  __device__ __forceinline__ void store_kc(double* img) const {
    const int ch = threadIdx.x & 31, row0 = threadIdx.x >> 5;
#pragma unroll
    for (int q = 0; q < NQ; ++q) *(doublex2*)(img + kc_off<NB>(2 * ch, row0 + 16 * q)) = r[q];
  }
  __device__ __forceinline__ void store_rc(double* img) const {
    const int ch = threadIdx.x & 31, row0 = threadIdx.x >> 5;
#pragma unroll
    for (int q = 0; q < NQ; ++q) *(doublex2*)(img + rc_off<NB>(row0 + 16 * q, 2 * ch)) = r[q];
  }
};

constexpr int FLOW_IMGS = 4;
struct FlowShared {
  union {
    double img[FLOW_IMGS][F64_IMG];
    struct {
      double u[F64_IMG];       // U(s, s-1)
      double inv[F64_IMG];     // Linv(s-1, s-1), then rows of Linv(s, s) as they are finished
      StepShared step;
      double x[10][256];       // U(s, s): the 16 x 16 blocks of its lower triangle by rows, a lane's elements 64 apart
    } chain;
  };
  double job[2][4][6];
  unsigned int ticket, unit;
};
static_assert(sizeof(FlowShared) <= 160 * 1024, "of the CU's LDS 3 KB are left: a workgroup has it to itself");

__device__ __forceinline__ double* flow_at(double* M, long long ld, int i, int k) { return M + (long long)i * NB * ld + (long long)k * NB; }

// rows row0 .. row0 + R - 1 of a KC image, by one wavefront, one row of 64 columns at a time
template <int R>
__device__ __forceinline__ void flow_rows_out(const double* img, double* dst, long long ld, int rv, int cv, int row0, int lane, bool lower) {
  double v[R];
#pragma unroll
  for (int q = 0; q < R; ++q) v[q] = img[kc_off<NB>(lane, row0 + q)];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int row = row0 + q;
    if (row < rv && lane < cv) agent_put(&dst[(long long)row * ld + lane], lower && lane > row ? 0.0 : v[q]);
  }
}

// a wavefront's part of the chain's tiles is in memory
__device__ __forceinline__ void flow_signal(const FlowP& p, int word, int lane) {
  flow_stored();
  if (lane < FLOW_COPIES) __hip_atomic_fetch_add(flow_chain(p, lane) + word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// this wavefront's 32 x 32 elements of L(s, s-1), columns 16 T0 .. and 16 T1 ..
template <int T0, int T1>
__device__ __forceinline__ void flow_l_out(const FlowP& p, double* dst, int jb, const doublex4 (&acc)[2][2], int wm, int l16, int lq) {
  const unsigned int step = (unsigned int)p.ld * 32u;
  unsigned int off = ((unsigned int)(wm + lq) * (unsigned int)p.ld + (unsigned int)l16) * 8u;
#pragma unroll
  for (int q = 0; q < 8; ++q, off += step) {
    if (jb < NB && wm + 4 * q + lq >= jb) continue;
    agent_put((double*)((char*)(dst + 16 * T0) + off), acc[q >> 2][0][q & 3]);
    agent_put((double*)((char*)(dst + 16 * T1) + off), acc[q >> 2][1][q & 3]);
  }
}
// The chain: wavefronts 0 .. 3 compute (their share of a 64 x 64 tile is 32 x 32), 4 .. 7 move.
__device__ __forceinline__ void flow_chain_workers(const FlowP& p, FlowShared& sh) {
  StepShared& st = sh.chain.step;
#pragma unroll 1
  for (int s = 0; s < p.N; ++s) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));          // no address of a stage is kept for the next one: there are no registers left for that
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = (wave >> 1) * 32, half = wave & 1, l16 = lane & 15, lq = lane >> 4;
    const int rows = p.n - s * NB, jb = rows < NB ? rows : NB;
    // 16 x 16 blocks of the diagonal tile's lower triangle: block (wave, 0), which the pivots begin with, and for wavefronts 0 .. 2
    // those that diag_block asks for
    const auto drow = [&](int q) { return q == 0 ? wave : q == 1 ? (wave < 3 ? 1 + wave : 3) : wave == 0 ? 2 : 3; };
    const auto dcol = [&](int q) { return q == 0 ? 0 : q == 1 ? 1 : wave < 2 ? 2 : 3; };
    doublex4 acc[2][2];
    if (s > 0) mma_lower_t(sh.chain.u, sh.chain.inv, wm, half, lane, acc);
    else zero_acc(acc);
    put_kc_tri(st.a, wm, half, lane, acc);
    if (s > 0 && wave < 3) {
      double* const dst = flow_at(p.A, p.ld, s, s - 1);
      if (half) flow_l_out<1, 2>(p, dst, jb, acc, wm, l16, lq);
      else flow_l_out<0, 3>(p, dst, jb, acc, wm, l16, lq);
    }
    lds_barrier();
    // rows of L past the edge are zero: what is put there stays
    auto block = [&](int q) {
      doublex4 u[2];
      u[0] = u[1] = doublex4{0.0, 0.0, 0.0, 0.0};
      doublex2 x[8], y[8];
      const double* const ax = st.a + kc_off<NB>(2 * lq, 16 * drow(q) + l16);
      const double* const ay = st.a + kc_off<NB>(2 * lq, 16 * dcol(q) + l16);
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) {
        x[cc] = *(const doublex2*)(ax + kc_off<NB>(8 * cc, 0));
        y[cc] = *(const doublex2*)(ay + kc_off<NB>(8 * cc, 0));
      }
      doublex4 v;
      const double* const xv = sh.chain.x[drow(q) * (drow(q) + 1) / 2 + dcol(q)] + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = xv[64 * r];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int cc = 0; cc < 8; ++cc) {
        u[0] = mma_f64(x[cc].x, y[cc].x, u[0]);
        u[1] = mma_f64(x[cc].y, y[cc].y, u[1]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * drow(q) + 4 * r + lq, k = 16 * dcol(q) + l16;
        if (jb < NB) v[r] = m < jb && k < jb ? v[r] : (m == k ? 1.0 : 0.0);
      }
      return v - (u[0] + u[1]);
    };
    const doublex4 c0 = block(0);
#pragma unroll
    for (int r = 0; r < 4; ++r) st.b[(16 * wave + 4 * r + lq) * SL + l16] = c0[r];
    lds_barrier();
    diag_block<true>(st, tid, sh.chain.inv, 0, jb, p.status, [&](int q, int, int) { return block(q); },
                     [&] { if (s > 0 && wave < 3) flow_signal(p, 1, lane); });
    lds_barrier();
  }
}
__device__ __forceinline__ void flow_chain_movers(const FlowP& p, FlowShared& sh) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) - 4, t = threadIdx.x - 256;
  // rows 16 i .. of Linv(s, s)
  auto inv_out = [&](int s, int i) {
    const int cv = p.n - s * NB;
    flow_rows_out<4>(sh.chain.inv, flow_at(p.V, p.ldv, s, s), p.ldv, cv, cv, 16 * i + 4 * w, lane, true);
  };
  // U(s, s-1) and U(s, s) into LDS: all loads first
  const int l16 = lane & 15, lq = lane >> 4, ld8 = 8 * (int)p.ld;
  auto load_u = [&](int s) {
    const int jb = p.n - s * NB;
    const __amdgpu_buffer_rsrc_t b1 = flow_buffer(flow_at(p.A, p.ld, s, s > 0 ? s - 1 : 0), p.ld, jb, s > 0 ? NB : jb);
    const __amdgpu_buffer_rsrc_t b0 = flow_buffer(flow_at(p.A, p.ld, s, s), p.ld, jb, jb);
    const int ch = t & 31, row0 = t >> 5, off1 = row0 * ld8 + 16 * ch, off0 = lq * ld8 + 8 * l16;
    doublex2 u[8];
    double v[3][4];
#pragma unroll
    for (int q = 0; q < 8; ++q) u[q] = flow_get2<true>(b1, off1, q * 8 * ld8);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int blk = w + 4 * q, row = blk > 5 ? 3 : blk > 2 ? 2 : blk > 0, col = blk - row * (row + 1) / 2;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        v[q][r] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(b0, off0, (16 * row + 4 * r) * ld8 + 128 * col, 16));
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) *(doublex2*)(sh.chain.u + kc_off<NB>(2 * ch, row0 + 8 * q)) = u[q];
#pragma unroll
    for (int q = 0; q < 3; ++q)
      if (w + 4 * q < 10)
#pragma unroll
        for (int r = 0; r < 4; ++r) sh.chain.x[w + 4 * q][64 * r + lane] = v[q][r];
  };
  // the part of L(s, s-1) that the wavefront with the pivots holds: rows 32 .., columns 16 .. 47
  auto l_out = [&](int s) {
    double v[4];
    const int row0 = 32 + 8 * w + (lane >> 5), k = 16 + (lane & 31);
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = sh.chain.step.a[kc_off<NB>(k, row0 + 2 * q)];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (row0 + 2 * q < p.n - s * NB) agent_put(&flow_at(p.A, p.ld, s, s - 1)[(long long)(row0 + 2 * q) * p.ld + k], v[q]);
  };
  FlowWait wait;
  load_u(0);
#pragma unroll 1
  for (int s = 0; s < p.N; ++s) {
    const bool next = s + 1 < p.N;
    bool have = !next;
    if (s > 0) inv_out(s - 1, 3);
    put_eye(sh.chain.step, t);
    if (s > 0) flow_signal(p, 0, lane);
    lds_barrier();
    if (s > 0) l_out(s);
    lds_barrier();
    // Between the seven barriers of diag_block a panel (about 1.5 us) and the short update behind it alternate: whatever takes time is
    // done beside a panel.  Rows of Linv(s, s) are finished beside the second, third and last panel and behind it.
    if (s > 0) flow_signal(p, 1, lane);
    lds_barrier();
    lds_barrier();
    if (next) {
      wait.set(0, flow_done(p, s + 1));
      wait.set(1, flow_done(p, s + 1) + 1);
      wait.set(2, flow_done(p, s + 1));
      wait.need[0] = s > 0 ? 2u : 0u;
      wait.need[1] = s > 0 ? 1u : 0u;
    }
    lds_barrier();
    lds_barrier();
    inv_out(s, 0);
    if (!have) flow_poll(p, wait);
    lds_barrier();
    lds_barrier();
    inv_out(s, 1);
    if (!have && (wait.ready() || flow_poll(p, wait) > 0)) {
      have = true;
      load_u(s + 1);
    }
    lds_barrier();
    inv_out(s, 2);
    if (!have) {
      if (!flow_wait(p, wait)) return;
      load_u(s + 1);
    }
    lds_barrier();
  }
  inv_out(p.N - 1, 3);
  flow_signal(p, 0, lane);
}

// L(row, j): which counter says that it is there, and what it has to say; coherent: the tile was read before in its former state
__device__ __forceinline__ void flow_need_l(const FlowP& p, FlowWait& w, int q, int row, int j, int copy) {
  if (j == row - 1) {
    w.word[q] = flow_chain(p, copy) + 1;
    w.seen[q] = 0;
    w.need[q] = 7u * row;
  } else {
    w.need[q] = (unsigned int)j + 1u;
  }
}
__device__ __forceinline__ bool flow_past_l(const FlowP& p, int row, int j) { return !p.lines_a || j >= row - 2; }

// 16 x 32 outputs per wavefront from here on
struct FlowLane {
  int lane, wave, wm, wn, l16, lq, copy;
  __device__ __forceinline__ FlowLane() {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    wm = (wave >> 1) * 16;
    wn = (wave & 1) * 32;
    l16 = lane & 15;
    lq = lane >> 4;
    copy = blockIdx.x & (FLOW_COPIES - 1);
  }
};
__device__ __forceinline__ void flow_put_inv(const FlowP& p, FlowTile<64>& t, int k) {
  t.load(flow_at(p.V, p.ldv, k, k), p.ldv, p.n - k * NB, p.n - k * NB, true);
}

// G(i, k): L(i, k), i > k + 2
__device__ __forceinline__ bool flow_l_task(const FlowP& p, FlowShared& sh, int i, int k) {
  const FlowLane id;
  const int rows = p.n - i * NB;
  FlowTile<64> ra, rb;
  doublex4 acc[1][2], c[1][2];
  zero_acc(acc);
  load_acc(flow_at(p.A, p.ld, i, k), p.ld, rows, NB, id.wm, id.wn, id.lane, c);
  FlowWait w;
  w.set(0, flow_l(p, i));
  w.set(1, flow_l(p, k));
  w.set(2, flow_chain(p, id.copy));
  auto need = [&](int j) {
    w.need[0] = (unsigned int)j + 1u;
    flow_need_l(p, w, 1, k, j, id.copy);
  };
  auto load = [&](int j) {
    ra.load(flow_at(p.A, p.ld, i, j), p.ld, rows, NB, !p.lines_a);
    rb.load(flow_at(p.A, p.ld, k, j), p.ld, NB, NB, flow_past_l(p, k, j));
  };
  if (k > 0) {
    need(0);
    if (!flow_wait(p, w)) return false;
    load(0);
  }
  for (int j = 0; j < k; ++j) {
    double* ia = sh.img[2 * (j & 1)];
    double* ib = sh.img[2 * (j & 1) + 1];
    ra.store_kc(ia);
    rb.store_kc(ib);
    lds_barrier();
    bool loaded = j + 1 >= k;
    if (!loaded) {
      need(j + 1);
      if (w.ready()) {
        load(j + 1);
        loaded = true;
      }
    }
    tile_mma<true>(ia, ib, id.wm, id.wn, id.lane, acc);
    if (!loaded) {
      if (!flow_wait(p, w)) return false;
      load(j + 1);
    }
  }
  double* ia = sh.img[2 * (k & 1)];
  double* ib = sh.img[2 * (k & 1) + 1];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) ia[kc_off<NB>(id.wn + 16 * j + id.l16, id.wm + 4 * r + id.lq)] = c[0][j][r] - acc[0][j][r];
  w.need[0] = w.need[1] = 0;
  w.need[2] = 4u * (k + 1);
  if (!flow_wait(p, w)) return false;
  flow_put_inv(p, rb, k);
  rb.store_kc(ib);
  lds_barrier();
  mma_lower_t(ia, ib, id.wm, id.wave & 1, id.lane, acc);
  double* out = flow_at(p.A, p.ld, i, k);
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = id.wm + 4 * r + id.lq;
      if (m < rows) agent_put(&out[(long long)m * p.ld + 16 * tri_tile(id.wave & 1, j) + id.l16], acc[0][j][r]);
    }
  flow_stored();
  lds_barrier();
  if (threadIdx.x == 0) agent_put(flow_l(p, i), (unsigned int)k + 1u);
  return true;
}

// acc[i] = M (rows 16 tri_tile(half, i), lower triangular, KC image) times T (columns wn .., RC image)
__device__ __forceinline__ void mma_lower_16(const double* im, const double* it, int half, int wn, int lane, doublex4 (&acc)[2]) {
  const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int mt = tri_tile(half, i);
    doublex4 s[2];
    s[0] = s[1] = doublex4{0.0, 0.0, 0.0, 0.0};
    for (int c2 = 0; c2 <= mt; ++c2)
#pragma unroll
      for (int c = 2 * c2; c < 2 * c2 + 2; ++c) {
        const int k = 8 * c + 2 * lq;
        const doublex2 a = *(const doublex2*)(im + kc_off<NB>(k, 16 * mt + l16));
        s[0] = mma_f64(a.x, it[rc_off<NB>(k, wn + l16)], s[0]);
        s[1] = mma_f64(a.y, it[rc_off<NB>(k + 1, wn + l16)], s[1]);
      }
    acc[i] = s[0] + s[1];
  }
}

// V(i, c): Linv(i, c), c < i, and the zeros of Linv(c, i)
__device__ __forceinline__ bool flow_v_task(const FlowP& p, FlowShared& sh, int i, int c) {
  const FlowLane id;
  const int rows = p.n - i * NB, tid = threadIdx.x;
  FlowTile<64> ra, rb;
  doublex4 acc[1][2];
  zero_acc(acc);
  {
    double* up = flow_at(p.V, p.ldv, c, i) + (tid & 63);
    if ((tid & 63) < rows)
      for (int r = tid >> 6; r < NB; r += 8) up[(long long)r * p.ldv] = 0.0;
  }
  FlowWait w;
  w.set(0, flow_l(p, i));
  w.set(1, flow_v(p, c));
  w.set(2, flow_chain(p, id.copy));
  auto need = [&](int j) {
    flow_need_l(p, w, 0, i, j, id.copy);
    w.need[1] = j > c ? (unsigned int)j : 0u;
    w.need[2] = 4u * (c + 1);
  };
  auto load = [&](int j) {
    ra.load(flow_at(p.A, p.ld, i, j), p.ld, rows, NB, flow_past_l(p, i, j));
    rb.load(flow_at(p.V, p.ldv, j, c), p.ldv, NB, NB, j == c || !p.lines_v);
  };
  need(c);
  if (!flow_wait(p, w)) return false;
  load(c);
  for (int j = c; j < i; ++j) {
    double* ia = sh.img[2 * (j & 1)];
    double* ib = sh.img[2 * (j & 1) + 1];
    ra.store_kc(ia);
    rb.store_rc(ib);
    lds_barrier();
    bool loaded = j + 1 >= i;
    if (!loaded) {
      need(j + 1);
      if (w.ready()) {
        load(j + 1);
        loaded = true;
      }
    }
    tile_mma<false>(ia, ib, id.wm, id.wn, id.lane, acc);
    if (!loaded) {
      if (!flow_wait(p, w)) return false;
      load(j + 1);
    }
  }
  double* ia = sh.img[2 * (i & 1)];
  double* ib = sh.img[2 * (i & 1) + 1];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) ib[rc_off<NB>(id.wm + 4 * r + id.lq, id.wn + 16 * j + id.l16)] = -acc[0][j][r];
  w.need[0] = w.need[1] = 0;
  w.need[2] = 4u * (i + 1);
  if (!flow_wait(p, w)) return false;
  flow_put_inv(p, ra, i);
  ra.store_kc(ia);
  lds_barrier();
  doublex4 o[2];
  mma_lower_16(ia, ib, id.wave >> 2, 16 * (id.wave & 3), id.lane, o);
  double* out = flow_at(p.V, p.ldv, i, c);
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = 16 * tri_tile(id.wave >> 2, q) + 4 * r + id.lq;
      if (m < rows) agent_put(&out[(long long)m * p.ldv + 16 * (id.wave & 3) + id.l16], o[q][r]);
    }
  flow_stored();
  lds_barrier();
  if (tid == 0) agent_put(flow_v(p, c), (unsigned int)i);
  return true;
}

// D(s), rows 32 h ..: U(s, s-1) for the chain.  16 x 16 outputs per wavefront.
__device__ __forceinline__ bool flow_u_task(const FlowP& p, FlowShared& sh, int s, int h) {
  const FlowLane id;
  const int lane = id.lane, l16 = id.l16, lq = id.lq, wr = (id.wave >> 2) * 16, ct = id.wave < 4 ? id.wave : 7 - id.wave, wc = ct * 16;
  const int rows = p.n - s * NB - 32 * h;       // may be below 0
  double* const a2 = flow_at(p.A, p.ld, s, s - 2) + (long long)32 * h * p.ld;
  double* const a1 = flow_at(p.A, p.ld, s, s - 1) + (long long)32 * h * p.ld;
  doublex4 u[2], v[2], c2, c1;
  u[0] = u[1] = v[0] = v[1] = c2 = c1 = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = wr + 4 * r + lq;
    if (m < rows) {
      c2[r] = a2[(long long)m * p.ld + wc + l16];
      c1[r] = a1[(long long)m * p.ld + wc + l16];
    }
  }
  flow_stored();
  lds_barrier();
  if (threadIdx.x == 0) atomicAdd(flow_read(p, s), 1u);
  FlowTile<32> ra;
  FlowTile<64> rb, rc;
  FlowWait w;
  w.set(0, flow_l(p, s));
  w.set(1, flow_l(p, s - 2));
  w.set(2, flow_l(p, s - 1));
  for (int j = 0; j < s - 2; ++j) {
    w.need[0] = w.need[2] = (unsigned int)j + 1u;
    flow_need_l(p, w, 1, s - 2, j, id.copy);
    if (!flow_wait(p, w)) return false;
    ra.load(flow_at(p.A, p.ld, s, j) + (long long)32 * h * p.ld, p.ld, rows, NB, !p.lines_a);
    rb.load(flow_at(p.A, p.ld, s - 2, j), p.ld, NB, NB, flow_past_l(p, s - 2, j));
    rc.load(flow_at(p.A, p.ld, s - 1, j), p.ld, NB, NB, flow_past_l(p, s - 1, j));
    lds_barrier();
    ra.store_kc(sh.img[0]);
    rb.store_kc(sh.img[1]);
    rc.store_kc(sh.img[2]);
    lds_barrier();
#pragma unroll 2
    for (int cc = 0; cc < 8; ++cc) {
      const int k = 8 * cc + 2 * lq;
      const doublex2 x = *(const doublex2*)(sh.img[0] + kc_off<NB>(k, wr + l16));
      const doublex2 y = *(const doublex2*)(sh.img[1] + kc_off<NB>(k, wc + l16)), z = *(const doublex2*)(sh.img[2] + kc_off<NB>(k, wc + l16));
      u[0] = mma_f64(x.x, y.x, u[0]);
      v[0] = mma_f64(x.x, z.x, v[0]);
      u[1] = mma_f64(x.y, y.y, u[1]);
      v[1] = mma_f64(x.y, z.y, v[1]);
    }
  }
  lds_barrier();
#pragma unroll
  for (int r = 0; r < 4; ++r) sh.img[0][kc_off<NB>(wc + l16, wr + 4 * r + lq)] = c2[r] - (u[0][r] + u[1][r]);
  w.set(0, flow_chain(p, id.copy));
  w.set(1, flow_chain(p, id.copy) + 1);
  w.need[2] = 0;
  w.need[0] = 4u * (s - 1);
  if (!flow_wait(p, w)) return false;
  flow_put_inv(p, rb, s - 2);
  rb.store_kc(sh.img[1]);
  lds_barrier();
  w.need[1] = 7u * (s - 1);
  if (!flow_wait(p, w)) return false;
  rc.load(flow_at(p.A, p.ld, s - 1, s - 2), p.ld, NB, NB, true);
  doublex4 l[1][2];
  switch (ct) {
    case 0: mma_lower_t_cols<1, 0, -1>(sh.img[0], sh.img[1], wr, lane, l); break;
    case 1: mma_lower_t_cols<1, 1, -1>(sh.img[0], sh.img[1], wr, lane, l); break;
    case 2: mma_lower_t_cols<1, 2, -1>(sh.img[0], sh.img[1], wr, lane, l); break;
    default: mma_lower_t_cols<1, 3, -1>(sh.img[0], sh.img[1], wr, lane, l); break;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) sh.img[3][kc_off<NB>(wc + l16, wr + 4 * r + lq)] = l[0][0][r];
  rc.store_kc(sh.img[2]);
  lds_barrier();
#pragma unroll
  for (int cc = 0; cc < 8; ++cc) {
    const int k = 8 * cc + 2 * lq;
    const doublex2 x = *(const doublex2*)(sh.img[3] + kc_off<NB>(k, wr + l16)), z = *(const doublex2*)(sh.img[2] + kc_off<NB>(k, wc + l16));
    v[0] = mma_f64(x.x, z.x, v[0]);
    v[1] = mma_f64(x.y, z.y, v[1]);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = wr + 4 * r + lq;
    if (m < rows) agent_put(&a1[(long long)m * p.ld + wc + l16], c1[r] - (v[0][r] + v[1][r]));
  }
  flow_stored();
  lds_barrier();
  if (threadIdx.x == 0) atomicAdd(flow_done(p, s), 1u);
  return true;
}

// D(s): L(s, s-2) and U(s, s).  The ten 16 x 16 blocks of its lower triangle, by wavefront (wavefronts w and w + 4 share a SIMD):
// (3, 0) and (0, 0), (3, 2) and (1, 0), (2, 0), (2, 2), (3, 1), (1, 1), (2, 1), (3, 3)
__device__ __forceinline__ bool flow_d_task(const FlowP& p, FlowShared& sh, int s) {
  const FlowLane id;
  const int rows = p.n - s * NB, jb = rows < NB ? rows : NB, nblk = id.wave < 2 ? 2 : 1;
  double* const a2 = flow_at(p.A, p.ld, s, s - 2);
  double* const a0 = flow_at(p.A, p.ld, s, s);
  const auto brow = [&](int q) { return q ? id.wave : (int)(0x32132233u >> (4 * id.wave) & 15u); };
  const auto bcol = [&](int q) { return q ? 0 : (int)(0x31112020u >> (4 * id.wave) & 15u); };
  FlowTile<64> ra, rb;
  doublex4 u[1][2], x[2], c2[1][2], c0[2];
  zero_acc(u);
  x[0] = x[1] = doublex4{0.0, 0.0, 0.0, 0.0};
  load_acc(a2, p.ld, rows, NB, id.wm, id.wn, id.lane, c2);
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int m = 16 * brow(q) + 4 * r + id.lq, k = 16 * bcol(q) + id.l16;
      m = m < jb ? m : jb - 1;
      k = k < jb ? k : jb - 1;
      c0[q][r] = a0[(long long)m * p.ld + k];
    }
  auto square = [&](const double* il) {      // x += L L^T
#pragma unroll
    for (int q = 0; q < 2; ++q)
      if (q < nblk) {
        doublex4 t = doublex4{0.0, 0.0, 0.0, 0.0};
        doublex2 a[8], b[8];
        const double* const ia = il + kc_off<NB>(2 * id.lq, 16 * brow(q) + id.l16);
        const double* const ib = il + kc_off<NB>(2 * id.lq, 16 * bcol(q) + id.l16);
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) {
          a[cc] = *(const doublex2*)(ia + kc_off<NB>(8 * cc, 0));
          b[cc] = *(const doublex2*)(ib + kc_off<NB>(8 * cc, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int cc = 0; cc < 8; ++cc) {
          x[q] = mma_f64(a[cc].x, b[cc].x, x[q]);
          t = mma_f64(a[cc].y, b[cc].y, t);
        }
        x[q] += t;
      }
  };
  FlowWait w;
  w.set(0, flow_l(p, s));
  w.set(1, flow_l(p, s - 2));
  w.set(2, flow_chain(p, id.copy));
  for (int j = 0; j < s - 2; ++j) {
    w.need[0] = (unsigned int)j + 1u;
    flow_need_l(p, w, 1, s - 2, j, id.copy);
    if (!flow_wait(p, w)) return false;
    ra.load(flow_at(p.A, p.ld, s, j), p.ld, rows, NB, !p.lines_a);
    rb.load(flow_at(p.A, p.ld, s - 2, j), p.ld, NB, NB, flow_past_l(p, s - 2, j));
    double* ia = sh.img[2 * (j & 1)];
    double* ib = sh.img[2 * (j & 1) + 1];
    ra.store_kc(ia);
    rb.store_kc(ib);
    lds_barrier();
    tile_mma<true>(ia, ib, id.wm, id.wn, id.lane, u);
    square(ia);
  }
  double* ia = sh.img[2 * (s & 1)];
  double* ib = sh.img[2 * (s & 1) + 1];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) ia[kc_off<NB>(id.wn + 16 * j + id.l16, id.wm + 4 * r + id.lq)] = c2[0][j][r] - u[0][j][r];
  w.set(1, flow_read(p, s));
  w.need[0] = 0;
  w.need[1] = 2u;
  w.need[2] = 4u * (s - 1);
  if (!flow_wait(p, w)) return false;
  flow_put_inv(p, rb, s - 2);
  rb.store_kc(ib);
  lds_barrier();
  doublex4 l[1][2];
  mma_lower_t(ia, ib, id.wm, id.wave & 1, id.lane, l);
  double* il = sh.img[2 * (~s & 1)];
  put_kc_tri(il, id.wm, id.wave & 1, id.lane, l);
  lds_barrier();
  square(il);
  // the chain waits for this tile
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (q < nblk)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * brow(q) + 4 * r + id.lq, k = 16 * bcol(q) + id.l16;
        if (m < jb && k < jb) agent_put(&a0[(long long)m * p.ld + k], c0[q][r] - x[q][r]);
      }
  flow_stored();
  lds_barrier();
  if (threadIdx.x == 0) agent_put(flow_done(p, s) + 1, 1u);
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = id.wm + 4 * r + id.lq;
      if (m < rows) agent_put(&a2[(long long)m * p.ld + 16 * tri_tile(id.wave & 1, j) + id.l16], l[0][j][r]);
    }
  flow_stored();
  lds_barrier();
  if (threadIdx.x == 0) agent_put(flow_l(p, s), (unsigned int)s - 1u);
  return true;
}

__device__ __forceinline__ void flow_ride(const FlowP& p, FlowShared& sh, const CoJob& job) {
  const int tid = threadIdx.x;
  if (tid == 0) sh.unit = atomicAdd(flow_unit(p), 2u);
  __syncthreads();
  unsigned int u = sh.unit;
  while (u < job.units) {
    __syncthreads();
    if (tid == 0) sh.unit = atomicAdd(flow_unit(p), 2u);
    const unsigned int mine = u + (tid >> 8);
    cojob_unit(job, mine, tid & 255, mine < job.units, sh.job[tid >> 8]);
    u = sh.unit;
  }
}

__global__ __launch_bounds__(512, 2) void chol_flow_kernel(const FlowP p, const CoJob job, int riders) {
  __shared__ __attribute__((aligned(16))) FlowShared sh;
  // every other workgroup of each XCD streams the ride-along job first
  if ((int)(blockIdx.x >> 3) % 2 < riders) flow_ride(p, sh, job);
  for (;;) {
    lds_barrier();
    if (threadIdx.x == 0) sh.ticket = atomicAdd(flow_ticket(p), 1u);
    if (agent_get(flow_abort(p))) return;
    lds_barrier();
    const unsigned int t = __builtin_amdgcn_readfirstlane(sh.ticket);
    if (t > p.tasks) break;
    if (t == 0) {
      if (threadIdx.x < 256) flow_chain_workers(p, sh);
      else flow_chain_movers(p, sh);
      return;
    }
    // N tasks in each of the first N - 2 stages, N - 2 and N - 1 in the last two
    const int e = (int)t - 1, whole = p.N > 2 ? p.N * (p.N - 2) : 0;
    bool ok;
    if (e >= whole) {
      const int q = e - whole, last = q >= p.N - 2;
      ok = flow_v_task(p, sh, last ? p.N - 1 : p.N - 2, last ? q - (p.N - 2) : q);
    } else {
      const int st = e / p.N, q = e - st * p.N;
      if (q < 2) ok = flow_u_task(p, sh, st + 2, q);
      else if (q == 2) ok = flow_d_task(p, sh, st + 2);
      else if (q < p.N - st) ok = flow_l_task(p, sh, st + q, st);
      else ok = flow_v_task(p, sh, st, q - (p.N - st));
    }
    if (!ok) return;
  }
  if (job.units) flow_ride(p, sh, job);
}

__global__ __launch_bounds__(256) void cojob_kernel(const CoJob job) { cojob_run(job, blockIdx.x, gridDim.x); }
strp_status launch_cojob(strp_ctx* ctx, const CoJob& job) {
  ProfScope ps(ctx, "pruned_rows", 0.0, (job.Z0 ? 16.0 : 12.0) * (double)job.nrows * (double)job.T);
  hipLaunchKernelGGL(cojob_kernel, dim3(job.units < 2048u ? job.units : 2048u), dim3(256), 0, ctx->stream, job);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

// the counters' lines in a row: columns 64 .. of rows 0 .. 63, which no task reads
static int flow_row_lines(int n) {
  int s = 0;
  while (s < 6 && (16 << s) <= n - NB) ++s;
  return s;
}
static bool flow_lines(const double* M, long long ld) { return ld % 16 == 0 && ((uintptr_t)M & 127) == 0; }
// Which way a system goes: by its order, so that the factor's bits depend neither on what else is done in the call nor on where the
// caller's factor lies, but in two ranges where a long pass that rides along (cojob.h) turns the comparison.
// us, a launch per panel / one launch, rows of whole cache lines:  n = 72 33.1 / 28.5,
// 136 47.0 / 39.1, 333 84 / 71, 600 133 / 114, 1000 211 / 175, 1408 293 / 237, 2048 505 / 383, 3072 953 / 856, 3600 1392 / 1312,
// 3968 1702 / 1549, 4416 2213 / 2214, 4912 2945 / 2730, 5312 3589 / 3273, 5888 4750 / 4710, 6272 5658 / 5407, 7168 8252 / 7446,
// 8192 12537 / 11973, 10240 24.7 / 19.1 ms; tiles that share cache lines, which are read past the caches:  1384 296 / 243,
// 1672 369 / 291, 2056 564 / 405, 3080 1011 / 898, 4915 3131 / 2729, 8600 15.8 / 13.3 ms.  The launch loses where the stages that its 255
// other workgroups hold at a time fall from four to three and from three to two (N tasks each), since what the chain waits
// for next is then handed out later:  4032 1770 / 1797, 4160 1902 / 1983, 4288 2056 / 2082; 5376 3685 / 3854, 5568 4092 / 4238,
// 5696 4373 / 4430.  With more tiles they bound it themselves, and at the third fall (8064 12.2 / 11.4 ms) it stays ahead.
// A pass runs beside the whole launch, or beside the chain's first one, so there it pays from about 1 and 4 GB on (bytes read and written):
// 3976, 0.5 GB 1849 / 1862, 1.0 1938 / 1932, 2.0 2233 / 2193, 8.0 3516 / 3136;  4200, 0.5 2104 / 2120, 1.0 2195 / 2162;  4096, 1.0 2052 / 2078, 2.0
// 2365 / 2333, 19 5225 / 4862;  5328, 2.0 4294 / 4354, 4.0 4694 / 4667, 8.0 5477 / 5197;  5560, 2.0 4744 / 4908, 4.0 5145 / 5137, 16 7499 / 6518;
// 5400, 4.0 4885 / 4982, 8.0 5612 / 5360, 17 6877 / 6166.  Elsewhere it widens the lead:  1000 of 2312 units over 30011 tokens 288 / 193, 3281 of 8192
// over 65536 1985 / 1691, 4912, 1.9 GB, 3403 / 3148.  With a pass beside
// them tiles that share lines cost the launch its lead (1000 331, 1544 744 / 728, 3281 2113 / 2043): a step pads its rows (system_ld).
bool chol_flow_ok(int n, double pass_bytes) {
  const int N = (n + NB - 1) / NB;
  if (n < NB + 8 || flow_lines_needed(N) > NB << flow_row_lines(n)) return false;
  if (N >= 63 && N <= 68) return pass_bytes >= 1e9;
  if (N >= 84 && N <= 90) return pass_bytes >= 4e9;
  return true;
}
bool chol_by_order(int n) { return chol_flow_ok(n, 0.0) == chol_flow_ok(n, 1e30); }

strp_status chol_flow(strp_ctx* ctx, double* A, int n, long long ld, double* Linv, long long ldv, int32_t* status, const CoJob& job) {
  FlowP p;
  memset(&p, 0, sizeof(p));
  p.A = A; p.ld = ld; p.V = Linv; p.ldv = ldv; p.flags = (unsigned int*)(A + NB); p.row_lines = flow_row_lines(n); p.n = n; p.N = (n + NB - 1) / NB; p.status = status;
  p.tasks = p.N > 1 ? (unsigned int)p.N * p.N - 3u : 0u;
  p.lines_a = flow_lines(A, ld);
  p.lines_v = flow_lines(Linv, ldv);
  p.limit = 1000000000ull;      // ten seconds
  const unsigned int wanted = 1 + p.tasks, most = ctx->flow_workers ? ctx->flow_workers : 256;
  const int grid = job.units ? 256 : (int)(wanted < most ? wanted : most);
  hipLaunchKernelGGL(chol_flow_kernel, dim3(grid), dim3(512), 0, ctx->stream, p, job, job.units ? 1 : 0);
  STRP_HIP(ctx, hipGetLastError());
  return STRP_OK;
}

}  // namespace strp
