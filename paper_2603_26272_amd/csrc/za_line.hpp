// Resident 1D kernels: a whole line stays on the chip for many RK3 steps.
//
// A 1D grid of a few thousand cells has too little work per stage to cover a
// launch: at N = 4096 a stage's sweep takes 6 us and the reduction launch
// that follows it 3.4 us, of which the fluxes are 1.4 us.  Here one launch
// runs up to a.nsteps steps.  Per stage, launches before -> resident now:
// advection 400 cells 7.7 -> 1.3 us, 1D Euler 200 cells 8.6 -> 2.5 us (one
// block: 2,900 cycles of fluxes, which four wavefronts on one CU issue at
// 4.9 cycles per instruction, and 1,800 of update, records and reduction),
// 1D Euler 4096 cells 9.7 -> 4.2 us (17 blocks: 2 us of it the round trip of
// the exchange through memory), 32000 cells 9.9 -> 4.9 us (126 blocks).  Thread t of a block owns cell c0 + t
// (its Q and Q^n stay in registers) and computes interface c0 + t; the
// records of the block's cells and of R halo cells per side sit in LDS.  Per
// stage: fluxes, one barrier, the update and the new records, the exchange
// of wave speeds (and, with several blocks, of the halo cells), one barrier.
//
// Several blocks exchange through global memory without fences: each 64-bit
// word carries 32 bits of payload and the exchange's 32-bit tag, is stored
// and polled with relaxed agent-scope atomics, and validates itself.  The
// words are double-buffered by the tag's parity: a block overwrites a word
// only after it has seen every block's next exchange, which each block
// publishes after it has read this one.  Every wait is bounded by a.spin
// ticks of the 100 MHz clock: a block that waits longer marks ctl->stuck and
// ends, the others follow, the result (in a workspace) is not committed, and
// the host repeats the steps with ordinary launches, which the context keeps
// from then on.  The limit is 1 s: the clock also runs while the device serves
// other processes, and a line that gave up too soon would lose its speed for
// good.
#pragma once
#include "za_kernels.hpp"

namespace za {

struct LineArgs {
  double* q;                 // state (one block: updated in place)
  double* out;               // result of a launch of several blocks (committed afterwards)
  DevCtl* ctl;
  unsigned long long* xch;   // exchange words (several blocks)
  Geom g;
  Phys ph;
  DevCtl init;               // one block: the sequence to start (arm), instead of *ctl
  int arm;
  int nsteps;                // steps of this launch, at most
  unsigned tag0;             // first exchange tag (several blocks)
  long long spin;            // wait limit, ticks of wall_clock64()
};

// Four such launches at once (one per hardware queue) still fit the chip: the
// host takes at most a quarter of the wavefronts that the device's CUs hold
// at the kernel's registers (of 256 CUs: 512 of 8 per CU, or 1024 of 16).
constexpr int LINE_MAX_BLOCKS = 128;
// Up to this many blocks every wavefront publishes its own maxima (one thread
// waits for each); beyond, the block's are reduced first, one barrier more.
constexpr int LINE_WAVE_BLOCKS = 64;
constexpr int LINE_MAX_WAVES = 16;
constexpr int LINE_HALO = 5;   // widest stencil half-width
// Wavefronts that one block takes before a second one joins: a second
// wavefront per SIMD costs the time of its fluxes, a second block the 2 us
// exchange.  Per stage, one block / several: Euler r = 3, 511 cells 3.7 /
// 4.1 us; advection, 1000 cells 1.9 / 2.5 us; Euler r = 5, 300 cells 8.0 /
// 7.1 us (so the wide and the general fluxes stop at one per SIMD).
constexpr int LINE_ONE_BLOCK_EULER = 8;
constexpr int LINE_ONE_BLOCK_WIDE = 4;
constexpr int LINE_ONE_BLOCK_SCALAR = 16;

// Exchange words of one parity: per wavefront its 3 wave-speed maxima, per
// block and side the R edge cells; two words per double.
constexpr int LINE_SPEED_WORDS = LINE_WAVE_BLOCKS * LINE_MAX_WAVES * 3 * 2;
constexpr int LINE_HALO_WORDS = LINE_MAX_BLOCKS * 2 * LINE_HALO * 3 * 2;
constexpr int LINE_WORDS = LINE_SPEED_WORDS + LINE_HALO_WORDS;

// Maxima of NV values over lanes 0 .. LANES - 1 (4, 16 or 64), wave-uniform.
// SIGNED = false: numbers >= 0 (or +inf), by words_max.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_max_f64(double x) {
  const int lo = (int)lo_word(x), hi = (int)hi_word(x);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, ROWS, 0xf, false);
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, ROWS, 0xf, false);
  return fmax(x, from_words((unsigned)l2, (unsigned)h2));
}
template <int LANES, int NV, bool SIGNED>
__device__ __forceinline__ void lanes_max(double (&v)[NV]) {
  if (SIGNED) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double x = dpp_max_f64<0x112, 0xf>(dpp_max_f64<0x111, 0xf>(v[i]));
      if (LANES > 4) x = dpp_max_f64<0x118, 0xf>(dpp_max_f64<0x114, 0xf>(x));
      if (LANES > 16) x = dpp_max_f64<0x143, 0xc>(dpp_max_f64<0x142, 0xa>(x));
      v[i] = from_words((unsigned)__builtin_amdgcn_readlane((int)lo_word(x), LANES - 1),
                        (unsigned)__builtin_amdgcn_readlane((int)hi_word(x), LANES - 1));
    }
  } else {
    unsigned hi[NV], lo[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) hi[i] = hi_word(v[i]);
    words_max<LANES, NV>(hi);
#pragma unroll
    for (int i = 0; i < NV; ++i) lo[i] = hi_word(v[i]) == hi[i] ? lo_word(v[i]) : 0u;
    words_max<LANES, NV>(lo);
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = from_words(lo[i], hi[i]);
  }
}

// Wave speeds of one cell (cell_speeds' values, with selects in place of its
// branch so that they interleave with the record of the same cell).
template <int SYS, int M, int NV>
__device__ __forceinline__ void line_cell_speeds(const double (&Q)[M], const Phys& ph, double (&v)[NV]) {
  if constexpr (SYS == SYS_EULER) {
    double u, w, p, c2;
    euler_cell_speed(Q[0], Q[1 % M], 0.0, Q[M - 1], ph, u, w, p, c2);
    const bool ok = Q[0] > 0.0 && p > 0.0 && c2 > 0.0 && c2 < __builtin_huge_val();
    const double c = __builtin_sqrt(c2);
    v[0] = ok ? fabs(u - c) : __builtin_huge_val();
    v[1] = ok ? fabs(u) : 0.0;
    v[2] = ok ? fabs(u + c) : 0.0;
  } else {
    const double u = Q[0];
    const bool ok = (u - u) == 0.0;
    if constexpr (SYS == SYS_BUCKLEY) {
      v[0] = ok ? u : __builtin_huge_val();
      v[1] = ok ? -u : -__builtin_huge_val();
    } else {
      v[0] = ok ? fabs(scalar_df<SYS>(u, ph.adv[0])) : __builtin_huge_val();
    }
  }
}

// x of the next lane (wave_shl 1); lane 63 gets `last`.
__device__ __forceinline__ double next_lane(double x, double last) {
  const int lo = __builtin_amdgcn_update_dpp((int)lo_word(last), (int)lo_word(x), 0x130, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp((int)hi_word(last), (int)hi_word(x), 0x130, 0xf, 0xf, false);
  return from_words((unsigned)lo, (unsigned)hi);
}

__device__ __forceinline__ unsigned long long line_word(double x, int half, unsigned tag) {
  return ((unsigned long long)tag << 32) | (half ? hi_word(x) : lo_word(x));
}
__device__ __forceinline__ double line_value(unsigned long long lo, unsigned long long hi) {
  return from_words((unsigned)lo, (unsigned)hi);
}
__device__ __forceinline__ void line_put(unsigned long long* p, unsigned long long w) {
  __hip_atomic_store(p, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long line_get(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Speeds that the sweeps of one stage need, from the global maxima: the LF
// speeds per field, max(|u| + c), and whether the state is admissible.
template <int SYS>
__device__ __forceinline__ void line_speeds(const double (&r)[3], const Phys& ph, SweepConst& sk, bool& bad) {
  bad = !(r[0] < __builtin_huge_val());
  if (SYS == SYS_BUCKLEY) {
    sk.smax = bad ? 0.0 : buckley_max_speed(-r[1], r[0], ph.bl_root);
    sk.al[0] = sk.smax;
  } else if (SYS == SYS_EULER) {
    sk.smax = wave_max(r[0], r[2]);
    sk.al[0] = ph.lf_scalar ? sk.smax : r[0];
    sk.al[1] = ph.lf_scalar ? sk.smax : r[1];
    sk.al[2] = sk.al[1];
    sk.al[3] = ph.lf_scalar ? sk.smax : r[2];
  } else {
    sk.smax = r[0];
    sk.al[0] = r[0];
  }
}

// One block's part of a line: its cells [c0, c0 + n), LDS records, and the
// exchange after each change of the state.
template <int SYS, int M, class T, int R, int LB>
struct LineBlock {
  static constexpr int NF = NumFields<SYS, M>::value;
  static constexpr int NV = SYS == SYS_EULER ? 3 : (SYS == SYS_BUCKLEY ? 2 : 1);   // maxima kept
  static constexpr bool SIGNED = SYS == SYS_BUCKLEY;
  static constexpr double NONE = SIGNED ? -__builtin_huge_val() : 0.0;   // below every speed
  static constexpr int RECN = LB + 2 * R;               // record slots: R halo, the cells, R halo
  struct Lds {
    T rec[NF * RECN];
    double fw[M][LB / 64 + 1];   // flux of each wavefront's first interface
    double sm[NV][16];           // maxima per wavefront
    double sb[NV][16];           // ... of the block's own cells
    int dead;
  };
  Lds& s;
  int tid, lane, wv, nw, P, b, n;
  bool own, has_l, has_r;

  // Publish the new state, build its records, and return the maxima over the
  // whole line; false if another block did not answer in time.
  __device__ __forceinline__ bool exchange(const LineArgs& a, const double (&q)[M], unsigned tag, double (&r)[3]) {
    double v[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = NONE;
    if (own) {
      line_cell_speeds<SYS, M, NV>(q, a.ph, v);
      if (P == 1) cell_record<SYS, M, 0, T>(q, a.ph, s.rec + R + tid, RECN);
    }
    lanes_max<64, NV, SIGNED>(v);
    if (P > 1) {
      unsigned long long* const base = a.xch + (size_t)(tag & 1) * LINE_WORDS;
      unsigned long long* const sp = base;
      unsigned long long* const hl = base + LINE_SPEED_WORDS;
      const bool per_block = P > LINE_WAVE_BLOCKS;
      if (per_block) {
        if (lane == 0) {
#pragma unroll
          for (int i = 0; i < NV; ++i) s.sb[i][wv] = v[i];
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = s.sb[i][lane & 15];
        lanes_max<16, NV, SIGNED>(v);
      }
      if (lane < 2 * NV && (!per_block || wv == 0)) {
        double x = v[0];
#pragma unroll
        for (int i = 1; i < NV; ++i) x = (lane >> 1) == i ? v[i] : x;
        line_put(sp + (per_block ? b : b * nw + wv) * 6 + lane, line_word(x, lane & 1, tag));
      }
      if (own && (tid < R || tid >= n - R)) {
        // side 0: the block's first R cells, side 1: its last R
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          const int k = side == 0 ? tid : tid - (n - R);
          if (k >= 0 && k < R) {
            unsigned long long* const w = hl + ((b * 2 + side) * LINE_HALO + k) * 6;
#pragma unroll
            for (int c = 0; c < M; ++c) {
              line_put(w + 2 * c, line_word(q[c], 0, tag));
              line_put(w + 2 * c + 1, line_word(q[c], 1, tag));
            }
          }
        }
      }
      if (own) cell_record<SYS, M, 0, T>(q, a.ph, s.rec + R + tid, RECN);
      // thread i waits for wavefront (block) i's maxima, threads 0 .. 2R - 1
      // also for the halo cells
      const bool need = tid < (per_block ? P : P * nw);
      const bool left = tid < R;
      const bool hneed = tid < 2 * R && (left ? has_l : has_r);
      const int hk = left ? tid : tid - R;
      const int nb = left ? (b == 0 ? P - 1 : b - 1) : (b == P - 1 ? 0 : b + 1);
      const unsigned long long* const ws = sp + (size_t)(need ? tid : 0) * 6;
      const unsigned long long* const wh = hl + (size_t)((nb * 2 + (left ? 1 : 0)) * LINE_HALO + (hneed ? hk : 0)) * 6;
      unsigned long long x[2 * NV], h[2 * M];
      const long long t0 = wall_clock64();
      bool dead = false;
      while (true) {
        bool ok = true;
        if (need) {
#pragma unroll
          for (int i = 0; i < 2 * NV; ++i) x[i] = line_get(ws + i);
#pragma unroll
          for (int i = 0; i < 2 * NV; ++i) ok = ok && (unsigned)(x[i] >> 32) == tag;
        }
        if (hneed) {
#pragma unroll
          for (int i = 0; i < 2 * M; ++i) h[i] = line_get(wh + i);
#pragma unroll
          for (int i = 0; i < 2 * M; ++i) ok = ok && (unsigned)(h[i] >> 32) == tag;
        }
        if (__all(ok)) break;
        if (wall_clock64() - t0 > a.spin) { dead = true; break; }
      }
      if (dead) {
        if (lane == 0) {
          s.dead = 1;
          __hip_atomic_store(&a.ctl->stuck, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } else {
        if (hneed) {
          double qh[M];
#pragma unroll
          for (int c = 0; c < M; ++c) qh[c] = line_value(h[2 * c], h[2 * c + 1]);
          cell_record<SYS, M, 0, T>(qh, a.ph, s.rec + (left ? hk : R + n + hk), RECN);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = need ? line_value(x[2 * i], x[2 * i + 1]) : NONE;
        lanes_max<64, NV, SIGNED>(v);
      }
    }
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i) s.sm[i][wv] = v[i];
    }
    __syncthreads();
    if (P > 1 && s.dead) return false;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = s.sm[i][lane & 15];
    if (nw <= 4) lanes_max<4, NV, SIGNED>(v);
    else lanes_max<16, NV, SIGNED>(v);
#pragma unroll
    for (int i = 0; i < 3; ++i) r[i] = v[i < NV ? i : 0];
    return true;
  }
};

template <int SYS, int M, class T, int WV, int R, int PP, int LB>
__global__ __launch_bounds__(LB) void k_line_solve(LineArgs a, CfgArg<T> cfg) {
  typedef LineBlock<SYS, M, T, R, LB> B;
  __shared__ typename B::Lds lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_id();
  const int N = a.g.nx, P = gridDim.x, b = blockIdx.x;
  const int c0 = (int)((long long)b * N / P), n = (int)((long long)(b + 1) * N / P) - c0;
  const bool per = a.g.bc_x == 0;
  B blk{lds, tid, lane, wv, (int)(blockDim.x >> 6), P, b, n, tid < n,
        P > 1 && (per || b > 0), P > 1 && (per || b < P - 1)};
  DevCtl st;
  if (a.arm) {
    st = a.init;
  } else {
    st = *a.ctl;
    // read before this block publishes anything: another block ends, and
    // block 0 rewrites the control block, only after that
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  }
  if (!st.active) return;
  if (tid < 16) {
#pragma unroll
    for (int i = 0; i < B::NV; ++i) lds.sm[i][tid] = lds.sb[i][tid] = B::NONE;
  }
  if (tid == 0) lds.dead = 0;
  // record slots of this thread's stencil (ghost cells by index)
  int off[2 * R];
#pragma unroll
  for (int j = 0; j < 2 * R; ++j) {
    int i = tid - R + j;
    if (P == 1) i = bc_map(i, N, a.g.bc_x);
    else if (!per) i = min(max(i, -c0), N - 1 - c0);
    off[j] = R + i;
  }
  double q[M], qn[M];
#pragma unroll
  for (int c = 0; c < M; ++c) q[c] = blk.own ? gptr(a.q)[(size_t)c * N + c0 + tid] : 1.0;
  __syncthreads();   // sm and dead initialised
  double r[3];
  unsigned tag = a.tag0;
  if (!blk.exchange(a, q, tag, r)) return;
  SweepConst sk;
  bool bad;
  int done = 0;
  while (true) {
    line_speeds<SYS>(r, a.ph, sk, bad);
#pragma unroll
    for (int c = 0; c < M; ++c) qn[c] = q[c];
    if (bad) { st.bad = 1; st.bad_step = st.steps; st.active = 0; break; }
    if (st.max_steps > 0 && st.steps >= st.max_steps) { st.active = 0; break; }
    if (st.t >= st.t_final) { st.active = 0; break; }
    double dt;
    if (st.dt_fixed > 0.0) dt = st.dt_fixed;
    else if (a.ph.dt_rule == 1) dt = a.ph.cfl * a.g.dx * a.g.dx;
    else dt = a.ph.cfl * a.g.dx / sk.smax;
    st.last = 0;
    if (st.t + dt >= st.t_final) { dt = st.t_final - st.t; st.last = 1; }
    st.dt = dt;
    sk.dt = dt;
    for (int s = 0; s < 3; ++s) {
      const double ca = s == 0 ? 0.0 : (s == 1 ? 0.75 : 1.0 / 3.0);
      const double cb = s == 0 ? 1.0 : (s == 1 ? 0.25 : 2.0 / 3.0);
      sk.mu = 0.0;
      if (PP) sk.mu = sk.smax > 0.0 ? dt * fma(sk.smax, a.g.inv_dx, 0.0) / sk.smax : 0.0;
      T F[M];
#pragma unroll
      for (int c = 0; c < M; ++c) F[c] = T(0);
      if (tid <= n) stencil_flux<SYS, M, 0, T, WV, R>(lds.rec, B::RECN, off, a.ph, sk, cfg.w, F);
      if (lane == 0) {
#pragma unroll
        for (int c = 0; c < M; ++c) lds.fw[c][wv] = (double)F[c];
      }
      __syncthreads();   // the records have been read, the first fluxes are in place
      const double kx = -(cb * dt) * a.g.inv_dx;
#pragma unroll
      for (int c = 0; c < M; ++c) {
        const double Fl = (double)F[c];
        const double Fr = next_lane(Fl, lds.fw[c][wv + 1]);
        q[c] = fma(ca, qn[c], fma(kx, Fr - Fl, cb * q[c]));
      }
      if (!blk.exchange(a, q, ++tag, r)) return;
      if (s < 2) {
        line_speeds<SYS>(r, a.ph, sk, bad);
        if (bad) break;
      }
    }
    if (bad) {
      // an inadmissible stage: the step does not count, Q^n stands
      st.bad = 1; st.bad_step = st.steps; st.active = 0;
#pragma unroll
      for (int c = 0; c < M; ++c) q[c] = qn[c];
      break;
    }
    st.t = st.last ? st.t_final : st.t + dt;
    st.steps += 1;
    st.dt_min = fmin(st.dt_min, dt);
    st.dt_max = fmax(st.dt_max, dt);
    if (st.last) st.active = 0;
    if (st.max_steps > 0 && st.steps >= st.max_steps) st.active = 0;
    if (!st.active || ++done == a.nsteps) break;
  }
  double* const dst = P == 1 ? a.q : a.out;
  if (blk.own) {
#pragma unroll
    for (int c = 0; c < M; ++c) gptr(dst)[(size_t)c * N + c0 + tid] = q[c];
  }
  if (b == 0 && tid == 0) {
    // every field but ctl->stuck, which any block may set
    DevCtl* const o = a.ctl;
    o->dt = st.dt; o->t = st.t; o->t_final = st.t_final; o->dt_fixed = st.dt_fixed;
    o->dt_min = st.dt_min; o->dt_max = st.dt_max;
    o->steps = st.steps; o->max_steps = st.max_steps; o->bad_step = st.bad_step;
    o->active = st.active; o->bad = st.bad; o->last = st.last;
    o->line_tag = a.tag0;
  }
}

// The result of a k_line_solve of several blocks, copied into the state if
// that launch (tag0) ran and no block gave up.
static __global__ __launch_bounds__(256) void k_line_commit(const double* __restrict__ from, double* __restrict__ to,
                                                            size_t n, const DevCtl* ctl, unsigned tag0) {
  if (ctl->stuck || ctl->line_tag != tag0) return;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) to[i] = from[i];
}

// The right-hand side of a line that one block holds: wave speeds, fluxes
// and differences in one launch.
template <int SYS, int M, class T, int WV, int R, int LB>
__global__ __launch_bounds__(LB) void k_line_rhs(LineArgs a, CfgArg<T> cfg) {
  typedef LineBlock<SYS, M, T, R, LB> B;
  __shared__ typename B::Lds lds;
  const int tid = threadIdx.x, lane = tid & 63, wv = wave_id();
  const int N = a.g.nx;
  B blk{lds, tid, lane, wv, (int)(blockDim.x >> 6), 1, 0, N, tid < N, false, false};
  if (tid < 16) {
#pragma unroll
    for (int i = 0; i < B::NV; ++i) lds.sm[i][tid] = lds.sb[i][tid] = B::NONE;
  }
  int off[2 * R];
#pragma unroll
  for (int j = 0; j < 2 * R; ++j) off[j] = R + bc_map(tid - R + j, N, a.g.bc_x);
  double q[M];
#pragma unroll
  for (int c = 0; c < M; ++c) q[c] = blk.own ? gptr(a.q)[(size_t)c * N + tid] : 1.0;
  __syncthreads();
  double r[3];
  blk.exchange(a, q, 0u, r);
  SweepConst sk;
  bool bad;
  line_speeds<SYS>(r, a.ph, sk, bad);
  sk.mu = 0.0;
  sk.dt = 0.0;
  if (tid == 0 && bad) {
    if (!a.ctl->bad) a.ctl->bad_step = a.ctl->steps;
    a.ctl->bad = 1;
  }
  T F[M];
#pragma unroll
  for (int c = 0; c < M; ++c) F[c] = T(0);
  if (tid <= N) stencil_flux<SYS, M, 0, T, WV, R>(lds.rec, B::RECN, off, a.ph, sk, cfg.w, F);
  if (lane == 0) {
#pragma unroll
    for (int c = 0; c < M; ++c) lds.fw[c][wv] = (double)F[c];
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < M; ++c) {
    const double Fl = (double)F[c];
    const double Fr = next_lane(Fl, lds.fw[c][wv + 1]);
    if (blk.own) gptr(a.out)[(size_t)c * N + tid] = -(Fr - Fl) * a.g.inv_dx;
  }
}

}  // namespace za
