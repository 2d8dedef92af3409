// libza: host side of the C ABI declared in include/za.h.
//
// One context = one problem shape on one device and stream.  It owns the
// RK3 stage states, the partial stage of paired sweeps (2D scalar laws and
// limited Euler stages), the wave-speed rows, partial sums, the exchange words
// of a resident line and the device control blocks (LF speeds, dt, t) that let
// whole RK3 steps run without host round trips.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <string>
#include <vector>

#include "za.h"
#include "za_kernels.hpp"
#include "za_internal.hpp"
#include "za_launch.hpp"

using namespace za;

namespace {

const char* kStatusStr[] = {"ok", "invalid argument", "out of device memory", "device error",
                            "non-finite or non-physical state", "unsupported", "busy"};

int ncomp_of(const za_problem& p) {
  if (p.system == ZA_EULER) return p.dim == 1 ? 3 : 4;
  return 1;
}

}  // namespace

// ---------------------------------------------------------------------------
// validation
// ---------------------------------------------------------------------------
za_status za_validate(const za_problem* p, std::string* why) {
  auto fail = [&](const char* m) { if (why) *why = m; return ZA_ERR_ARG; };
  if (!p) return fail("problem is NULL");
  if (p->dim != 1 && p->dim != 2) return fail("dim must be 1 or 2");
  if (p->system < ZA_ADVECTION || p->system > ZA_BUCKLEY) return fail("unknown system");
  if (p->nx < 1 || p->ny < 1) return fail("nx and ny must be >= 1");
  if (p->dim == 1 && p->ny != 1) return fail("ny must be 1 in 1D");
  if ((long long)p->nx * p->ny > (1LL << 31)) return fail("grid too large");
  if (!(p->xhi > p->xlo) || (p->dim == 2 && !(p->yhi > p->ylo))) return fail("empty domain");
  if (p->bc_x < 0 || p->bc_x > 1 || p->bc_y < 0 || p->bc_y > 1) return fail("unknown boundary condition");
  if (p->system == ZA_EULER && !(p->gamma > 1.0)) return fail("gamma must exceed 1");
  if (!(p->cfl > 0.0)) return fail("cfl must be positive");
  if (p->dt_rule < 0 || p->dt_rule > 1) return fail("unknown dt rule");
  if (p->precision < 0 || p->precision > 1) return fail("unknown precision");
  if (!(p->p >= 1.0)) return fail("p must be >= 1");
  if (!(p->eps > 0.0)) return fail("eps must be positive");
  if (p->affine_invariant && !(p->mu0 > 0.0)) return fail("mu0 must be positive");
  if (p->precision == ZA_FP32_RECON && (p->eps < 1e-37 || (p->affine_invariant && p->mu0 < 1e-18)))
    return fail("FP32 reconstruction needs eps >= 1e-37 and mu0 >= 1e-18 (normal FP32 range)");
  // 16 eps and (2 mu0)^2 must be normal FP64 numbers with a finite reciprocal
  if (p->precision == ZA_FP64 && (p->eps < 1e-300 || (p->affine_invariant && p->mu0 < 1e-150)))
    return fail("FP64 needs eps >= 1e-300 and mu0 >= 1e-150 (normal FP64 range)");
  if (p->order != 0 && (p->order < 2 || p->order > 5)) return fail("order r must be 2, 3, 4 or 5");
  if (p->pp_limiter != 0 && p->pp_limiter != 1) return fail("pp_limiter must be 0 or 1");
  if (p->alt_tau != 0 && p->alt_tau != 1) return fail("alt_tau must be 0 or 1");
  if (!(weight_L(*p) >= 0.0) || !(weight_L(*p) < 1e300)) return fail("weight_L must be finite and >= 0");
  if (!(weight_q(*p) >= 1.0) || !(weight_q(*p) < 1e300)) return fail("weight_q must be finite and >= 1");
  if (p->alt_tau && order_of(*p) != 3) {
    if (why) *why = "the alternative global indicator is defined here for r = 3 only";
    return ZA_ERR_UNSUPPORTED;
  }
  if (p->pp_limiter && p->system != ZA_EULER) return fail("the positivity limiter applies to the Euler equations");
  if (p->pp_limiter && (p->dt_rule != ZA_DT_CFL || p->cfl > 0.5))
    return fail("the positivity limiter needs the CFL time step with cfl <= 0.5");
  if (p->pp_limiter && order_of(*p) != 3) {
    if (why) *why = "the positivity limiter runs with r = 3 only";
    return ZA_ERR_UNSUPPORTED;
  }
  if (p->pp_limiter && p->precision != ZA_FP64) {
    if (why) *why = "the positivity limiter runs with FP64 reconstruction only";
    return ZA_ERR_UNSUPPORTED;
  }
  if (order_of(*p) != 3 && p->precision != ZA_FP64) {
    if (why) *why = "orders other than r = 3 run in FP64 only";
    return ZA_ERR_UNSUPPORTED;
  }
  return ZA_OK;
}

size_t za_state_count(const za_problem* p) {
  if (za_validate(p, nullptr) != ZA_OK) return 0;
  return (size_t)ncomp_of(*p) * p->nx * p->ny;
}

// device bytes of the partial sums, and of the rows and control blocks
static constexpr int SUM_BLOCKS = 6144;
static constexpr size_t kPartBytes = 4 * (size_t)SUM_BLOCKS * sizeof(double);   // per component
static constexpr size_t kRowsBytes = SP_SETS * SP_SET * sizeof(unsigned long long) + 1024;
static_assert(CTL_COPIES * sizeof(DevCtl) <= 1024, "the control blocks");

size_t za_workspace_bytes(const za_problem* p) {
  if (za_validate(p, nullptr) != ZA_OK) return 0;
  const size_t st = za_state_count(p) * sizeof(double);
  size_t b = 2 * st;                      // Q1, Q2
  if (p->dim == 2) b += st;               // the partial stage (counted for fused stages too)
  b += kPartBytes + kRowsBytes;            // partial sums, wave-speed rows, control blocks
  int lb, lw;
  line_shape(*p, 256, &lb, &lw);          // (fewer CUs only take fewer lines)
  b += line_bytes(lb);                    // exchange words of the resident 1D kernel
  return b;
}

const char* za_status_str(za_status s) {
  int i = (int)s;
  if (i < 0 || i > 6) return "unknown status";
  return kStatusStr[i];
}

const char* za_ctx_last_error(const za_ctx* c) { return c ? c->err.c_str() : "no context"; }

// ---------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------
static za_status hip_fail(za_ctx* c, hipError_t e, const char* what) {
  c->err = std::string(what) + ": " + hipGetErrorString(e);
  return e == hipErrorOutOfMemory ? ZA_ERR_NOMEM : ZA_ERR_DEVICE;
}

#define ZA_CHECK_LAUNCH(c, what)                              \
  do {                                                        \
    hipError_t e_ = hipGetLastError();                        \
    if (e_ != hipSuccess) return hip_fail((c), e_, (what));   \
  } while (0)


static void timed_begin(za_ctx* c, int cls) {
  if (!c->timing) return;
  hipEvent_t e;
  hipEventCreate(&e);
  hipEventRecord(e, c->stream);
  c->ev_open[cls] = e;
}
static void timed_end(za_ctx* c, int cls) {
  if (!c->timing) return;
  hipEvent_t e;
  hipEventCreate(&e);
  hipEventRecord(e, c->stream);
  c->events[cls].push_back({c->ev_open[cls], e});
}

void launch_x(za_ctx* c, int mode, const SweepArgs& a) {
  timed_begin(c, 0);
  if (order_of(c->prob) != 3) {
    launch_x_order(c, mode, a);
    timed_end(c, 0);
    return;
  }
  if (!general_weights(c->prob)) launch_x_wv<WV_Z1>(c, mode, a);
  else if (square_powers(c->prob)) launch_x_square(c, mode, a);
  else launch_x_general(c, mode, a);
  timed_end(c, 0);
}

void launch_y(za_ctx* c, int mode, const SweepArgs& a) {
  timed_begin(c, 1);
  if (order_of(c->prob) != 3) {
    launch_y_order(c, mode, a);
    timed_end(c, 1);
    return;
  }
  if (!general_weights(c->prob)) launch_y_wv<WV_Z1>(c, mode, a);
  else if (square_powers(c->prob)) launch_y_square(c, mode, a);
  else launch_y_general(c, mode, a);
  timed_end(c, 1);
}

// Stand-alone wave-speed pass over q, for steps (clear; start: which begin a
// stepping sequence from this control block) or a right-hand side.
void launch_speeds(za_ctx* c, const double* q, int clear, const DevCtl* start) {
  timed_begin(c, 2);
  const size_t ncell = (size_t)c->prob.nx * c->prob.ny;
  DevCtl v;
  std::memset(&v, 0, sizeof(v));
  if (start) v = *start;
  const dim3 grid(c->red_blocks), blk(c->red_threads);
  DevCtl* const ctl = start ? c->ctl : nullptr;
#define ZA_S(SYS, M) \
  hipLaunchKernelGGL((k_speed_rows<SYS, M>), grid, blk, 0, c->stream, q, ncell, c->ph, c->rows, clear, ctl, v)
  switch (c->prob.system) {
    case ZA_EULER:
      if (c->prob.dim == 1) ZA_S(SYS_EULER, 3); else ZA_S(SYS_EULER, 4);
      break;
    case ZA_ADVECTION: ZA_S(SYS_ADV, 1); break;
    case ZA_BURGERS: ZA_S(SYS_BURGERS, 1); break;
    default: ZA_S(SYS_BUCKLEY, 1); break;
  }
#undef ZA_S
  timed_end(c, 2);
}

__global__ void k_ctl_init(DevCtl* ctl, DevCtl v) {
  if (threadIdx.x == 0) *ctl = v;
}
__global__ void k_ctl_arm(DevCtl* ctl, double dt_fixed, double t_final, long long max_steps) {
  // start a new stepping sequence from the current (t, steps)
  if (threadIdx.x != 0) return;
  ctl->dt_fixed = dt_fixed;
  ctl->t_final = t_final;
  ctl->max_steps = max_steps;
  ctl->active = ctl->bad ? 0 : 1;
}

SweepArgs base_args(za_ctx* c) {
  SweepArgs a;
  std::memset(&a, 0, sizeof(a));
  a.ctl = c->ctl;
  a.g = c->geom;
  a.ph = c->ph;
  a.ytile = c->ytile;
  a.xl_chunks = c->xl_chunks;
  return a;
}

int device_cus(int device) {
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, device) == hipSuccess && n > 0) return n;
  (void)hipGetLastError();
  return 256;
}

// Rows per y-sweep block: split each 64-column strip into as many tiles as
// there are resident block slots per strip, so that one round of blocks
// covers the grid (no tail round at partial occupancy).
static int pick_ytile(za_ctx* c) {
  const za_problem& p = c->prob;
  if (p.dim != 2) return 64;
  int blocks_per_cu = c->fu_gx && !p.pp_limiter ? 3   // (flux output only)
                      : order_of(p) != 3    ? order_y_blocks_per_cu(p)
                      : !general_weights(p) ? y_blocks_per_cu_wv<WV_Z1>(p)
                      : square_powers(p)    ? square_y_blocks_per_cu(p)
                                            : general_y_blocks_per_cu(p);
  if (blocks_per_cu < 1) blocks_per_cu = 2;
  const long long strips = (p.nx + 63) / 64;
  const long long slots = (long long)blocks_per_cu * c->cus;
  long long tiles = std::max<long long>(1, slots / strips);
  // a tile of R rows computes R + 1 interface rows, YS_ROWS per step: take
  // the largest R with as many steps as the rows a tile needs
  const int need = (int)((p.ny + tiles - 1) / tiles);
  const int rows = YS_ROWS * ((need + YS_ROWS) / YS_ROWS) - 1;
  return std::max(rows, YS_TILE_MIN);
}

// Chunks per row segment of the looped x-sweep (stages in FP64, r = 3, Z
// weights with p = 1, no limiter; 0: the one-shot sweep).  A wavefront walks nc chunks of 64
// interfaces; the choice minimises rounds of resident wavefronts x chunks
// per wavefront (a record pass counted as 1/32 of a flux pass), i.e. the
// critical path when every SIMD slot is busy.
// ZA_XL_CHUNKS in the environment forces a value (0 disables the sweep).
static int pick_xl_chunks(za_ctx* c) {
  const za_problem& p = c->prob;
  if (p.precision != ZA_FP64 || order_of(p) != 3 || p.pp_limiter || general_weights(p) || c->fu_gx) return 0;
  if (const char* e = std::getenv("ZA_XL_CHUNKS")) {
    const int v = std::atoi(e);
    return v < 0 ? 0 : std::min(v, 256);
  }
  int blocks_per_cu = 0;
  const void* fn = p.system != ZA_EULER ? reinterpret_cast<const void*>(&k_sweep_xl<SYS_ADV, 1, WV_Z1, MODE_LX>)
                                        : reinterpret_cast<const void*>(&k_sweep_xl<SYS_EULER, 3, WV_Z1, MODE_STAGE>);
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks_per_cu, fn, 256, 0) != hipSuccess || blocks_per_cu < 1)
    blocks_per_cu = 3;
  const long long slots = 4LL * blocks_per_cu * c->cus;
  int best = 1;
  long long best_cost = -1;
  for (int nc = 1; nc <= 64; ++nc) {
    const long long seg = 64LL * nc - 1;
    const long long waves = xl_waves(p.nx, p.ny, nc);
    const long long cost = ((waves + slots - 1) / slots) * (32LL * nc + nc + 1);
    if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = nc; }
    if (seg >= p.nx) break;   // one segment per row from here on
  }
  return best;
}

// Sweeps of more blocks than this take their constants from a stage_begin
// launch (5 us) instead of each block's own (1 us, of which two rounds of
// resident blocks hide most): a 2048^2 right-hand side by one-shot sweeps of
// 16,900 blocks took 297 us with the one and 271 us with the other.
static constexpr long long kBeginBlocks = 3072;

// Whether the first sweep of a stage (mode) has that many blocks; then the
// launch, after which the sweeps read a.ctl.
static bool begin_apart(za_ctx* c, int mode, SweepArgs& a) {
  const long long nseg = (c->prob.nx + XS_CELLS - 1) / XS_CELLS;
  const bool looped = c->xl_chunks > 0 && (mode == MODE_LX || mode == MODE_STAGE);
  const long long waves = looped ? xl_waves(c->prob.nx, c->prob.ny, c->xl_chunks) : nseg * c->prob.ny;
  if (waves / 4 <= kBeginBlocks) return false;
  const dim3 one(1), blk(64);
  a.nblk = 1;
  switch (c->prob.system) {
    case ZA_EULER:
      if (c->prob.dim == 1) hipLaunchKernelGGL((k_stage_begin<SYS_EULER, 1>), one, blk, 0, c->stream, a, 1);
      else hipLaunchKernelGGL((k_stage_begin<SYS_EULER, 2>), one, blk, 0, c->stream, a, 2);
      break;
    case ZA_ADVECTION: hipLaunchKernelGGL((k_stage_begin<SYS_ADV, 2>), one, blk, 0, c->stream, a, c->prob.dim); break;
    case ZA_BURGERS: hipLaunchKernelGGL((k_stage_begin<SYS_BURGERS, 2>), one, blk, 0, c->stream, a, c->prob.dim); break;
    default: hipLaunchKernelGGL((k_stage_begin<SYS_BUCKLEY, 2>), one, blk, 0, c->stream, a, c->prob.dim); break;
  }
  a.sp_in = nullptr;
  a.check_run = a.kind != FIN_RHS;
  return true;
}

// One RK3 step on the stream (no host synchronisation): per stage one fused
// kernel, one 1D sweep, or an x-sweep and a y-sweep.  The kernel that writes
// a stage's new state also leaves the wave-speed maxima of that state, and the
// first kernel of a stage turns the maxima of its input into the stage's
// constants (stage_begin), so only the first step of an API call needs a
// stand-alone pass.  start: begin a stepping sequence from this control block
// (with the stand-alone pass).
static za_status enqueue_step(za_ctx* c, double* q, const DevCtl* start = nullptr) {
  const double ca[3] = {0.0, 0.75, 1.0 / 3.0};
  const double cb[3] = {1.0, 0.25, 2.0 / 3.0};
  const int kind[3] = {FIN_STAGE0, FIN_STAGEK, FIN_STAGE2};
  const double* in[3] = {q, c->q1, c->q2};
  double* out[3] = {c->q1, c->q2, q};
  for (int s = 0; s < 3; ++s) {
    if (s == 0 && !c->speeds_valid) launch_speeds(c, q, 1, start);
    SweepArgs a = base_args(c);
    a.q = in[s];
    a.qn = q;
    a.ca = ca[s];
    a.cb = cb[s];
    a.kind = kind[s];
    a.cin = c->ctl + s;
    a.ctl = c->ctl + (s + 1) % 3;
    a.sp_in = c->rows + s * SP_SET;
    a.sp_rows = SP_ROWS;
    a.sp_out = c->rows + (s + 1) % 3 * SP_SET;
    a.sp_zero = c->rows + (s + 2) % 3 * SP_SET;
    a.out = out[s];
    if (c->prob.dim == 1) {
      begin_apart(c, MODE_STAGE, a);
      launch_x(c, MODE_STAGE, a);
    } else if (c->fu_gx && !c->ph.pp) {
      timed_begin(c, 1);
      launch_fused(c, MODE_STAGE, a);
      timed_end(c, 1);
    } else {
      a.out = c->lx;
      begin_apart(c, MODE_LX, a);
      launch_x(c, MODE_LX, a);
      a.sp_in = nullptr;     // the x-sweep has left the stage's constants in ctl
      a.check_run = 1;
      a.lx = c->lx;
      a.out = out[s];
      launch_y(c, MODE_STAGE, a);
    }
  }
  c->speeds_valid = true;
  ZA_CHECK_LAUNCH(c, "step launch");
  return ZA_OK;
}

// n RK3 steps (start: as for enqueue_step).  After the first step of an API
// call (which needs the stand-alone wave-speed pass), runs of GRAPH_STEPS
// steps replay a hipGraph captured once per state pointer on a private
// capture stream; kernels read dt and the LF speeds from the device control
// block, so a graph is valid for any step.  Kernel timing (events) uses
// direct launches.
static constexpr int GRAPH_STEPS = 16;

static za_status enqueue_steps(za_ctx* c, double* q, int64_t n, const DevCtl* start) {
  za_status st;
  int64_t done = 0;
  if (n > 0 && !c->speeds_valid) {
    if ((st = enqueue_step(c, q, start)) != ZA_OK) return st;
    done = 1;
  }
  if (!c->timing && c->graphs_ok && n - done >= GRAPH_STEPS) {
    if (!c->graph_exec || c->graph_q != q) {
      if (c->graph_exec) { (void)hipGraphExecDestroy(c->graph_exec); c->graph_exec = nullptr; }
      if (!c->capture_stream && hipStreamCreate(&c->capture_stream) != hipSuccess) c->graphs_ok = false;
      if (c->graphs_ok) {
        hipStream_t user = c->stream;
        c->stream = c->capture_stream;
        hipGraph_t g = nullptr;
        bool ok = hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal) == hipSuccess;
        for (int i = 0; ok && i < GRAPH_STEPS; ++i) ok = enqueue_step(c, q) == ZA_OK;
        ok = (hipStreamEndCapture(c->stream, &g) == hipSuccess) && ok;
        c->stream = user;
        if (ok) ok = hipGraphInstantiate(&c->graph_exec, g, nullptr, nullptr, 0) == hipSuccess;
        if (g) (void)hipGraphDestroy(g);
        if (!ok) {
          c->graphs_ok = false;
          c->graph_exec = nullptr;
          (void)hipGetLastError();
        } else {
          c->graph_q = q;
        }
      }
    }
    while (c->graph_exec && n - done >= GRAPH_STEPS) {
      hipError_t e = hipGraphLaunch(c->graph_exec, c->stream);
      if (e != hipSuccess) return hip_fail(c, e, "graph launch");
      done += GRAPH_STEPS;
    }
  }
  for (; done < n; ++done) {
    if ((st = enqueue_step(c, q)) != ZA_OK) return st;
  }
  return ZA_OK;
}

static DevCtl fresh_ctl() {
  DevCtl v;
  std::memset(&v, 0, sizeof(v));
  v.t = 0.0;
  v.t_final = std::numeric_limits<double>::infinity();
  v.dt_min = std::numeric_limits<double>::infinity();
  v.dt_max = 0.0;
  v.bad_step = -1;
  v.active = 0;
  return v;
}

// The control block that starts a stepping sequence.
static DevCtl start_ctl(double dt_fixed, double t_final, int64_t max_steps) {
  DevCtl v = fresh_ctl();
  v.dt_fixed = dt_fixed;
  v.t_final = t_final;
  v.max_steps = max_steps;
  v.active = 1;
  return v;
}

static void launch_ctl(za_ctx* c, const DevCtl& v) {
  hipLaunchKernelGGL(k_ctl_init, dim3(1), dim3(64), 0, c->stream, c->ctl, v);
}

// The control block after everything enqueued so far (waits for it).
static za_status read_ctl(za_ctx* c, DevCtl* h) {
  hipError_t e = hipMemcpyWithStream(h, c->ctl, sizeof(DevCtl), hipMemcpyDeviceToHost, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "read control block");
  return ZA_OK;
}

// Whether the steps of this context run in the resident 1D kernel (event
// timing brackets the launches of single kernels instead).
static bool line_ready(const za_ctx* c) { return c->line_blocks > 0 && c->line_ok && !c->timing; }

// Steps between host checks: a resident launch retires steps beyond the end
// by itself and costs nothing extra per step; ordinary launches go on for
// nothing until the host has looked (64 times as long between checks where
// only an inadmissible state ends the steps early).
static int64_t steps_per_check(const za_ctx* c, bool equal_steps) {
  if (line_ready(c)) return 4096;
  return equal_steps ? 64 * 32 : 32;
}

// The next of at most n RK3 steps (those until the next host check; returned
// in *n) from the control block (start: from this one instead).  *h receives
// the control block afterwards, but if these are all n steps and !read_last.
// A resident launch of several blocks needs *h to hold the control block
// before the steps (or start), to go back to if a block waits too long for
// the others (another kernel kept one from being scheduled): the context
// stays with ordinary launches from there.
static za_status advance(za_ctx* c, double* q, int64_t* n, bool equal_steps, const DevCtl* start, bool read_last,
                         DevCtl* h) {
  za_status st;
  const int64_t all = *n;
  *n = std::min(all, steps_per_check(c, equal_steps));
  DevCtl before;
  if (line_ready(c) && c->line_blocks == 1) {
    launch_line(c, q, *n, start);
    ZA_CHECK_LAUNCH(c, "step launch");
    return read_last || *n < all ? read_ctl(c, h) : ZA_OK;
  }
  if (line_ready(c)) {
    before = start ? *start : *h;
    if (start) launch_ctl(c, *start);
    launch_line(c, q, *n, nullptr);
    ZA_CHECK_LAUNCH(c, "step launch");
    if ((st = read_ctl(c, h)) != ZA_OK) return st;
    if (!h->stuck) return ZA_OK;
    c->line_ok = false;
    c->speeds_valid = false;
    start = &before;
    *n = std::min(all, steps_per_check(c, equal_steps));
  }
  if ((st = enqueue_steps(c, q, *n, start)) != ZA_OK) return st;
  return read_last || *n < all ? read_ctl(c, h) : ZA_OK;
}

// Set in the environment to 0.  ZA_STEP_GRAPHS=0 runs the steps of za_solve
// as direct launches instead of replaying captured step graphs (results are
// identical).
static bool env_off(const char* name) {
  const char* e = std::getenv(name);
  return e && std::atoi(e) == 0;
}

// Whether steps may run in the resident 1D kernel: not with ZA_RESIDENT=0,
// and not where the environment asks for a form of the step launches (results
// are identical).
bool resident_wanted() {
  return !env_off("ZA_RESIDENT") && !env_off("ZA_STEP_GRAPHS") && !std::getenv("ZA_XL_CHUNKS");
}

// Everything a context derives from its problem without allocating: the
// geometry and physics constants, launch shapes and reduction sizes.
void init_shape(za_ctx* c, const za_problem* p, hipStream_t stream) {
  c->prob = *p;
  c->m = ncomp_of(*p);
  c->stream = stream;
  (void)hipGetDevice(&c->device);
  c->cus = device_cus(c->device);
  const size_t ncell = (size_t)p->nx * p->ny;
  c->geom.nx = p->nx;
  c->geom.ny = p->ny;
  c->geom.bc_x = p->bc_x;
  c->geom.bc_y = p->bc_y;
  c->geom.dx = (p->xhi - p->xlo) / p->nx;
  c->geom.dy = p->dim == 2 ? (p->yhi - p->ylo) / p->ny : 1.0;
  c->geom.inv_dx = 1.0 / c->geom.dx;
  c->geom.inv_dy = 1.0 / c->geom.dy;
  c->ph.gamma = p->gamma;
  c->ph.gm1 = p->gamma - 1.0;
  c->ph.adv[0] = p->adv_speed[0];
  c->ph.adv[1] = p->adv_speed[1];
  c->ph.cfl = p->cfl;
  c->ph.dt_rule = p->dt_rule;
  c->ph.lf_scalar = p->lf == ZA_LF_SCALAR ? 1 : 0;
  c->ph.pp = p->pp_limiter ? 1 : 0;
  buckley_roots(c->ph.bl_root);
  // stand-alone wave-speed pass: at most one block per CU
  c->red_threads = ncell <= 65536 ? 256 : 1024;
  c->red_blocks = (int)std::min<size_t>(SP_ROWS, (ncell + c->red_threads - 1) / c->red_threads);
  fused_shape(*p, c->cus, &c->fu_gx, &c->fu_gy);
  c->ytile = pick_ytile(c);
  c->xl_chunks = pick_xl_chunks(c);
  c->graphs_ok = !env_off("ZA_STEP_GRAPHS");
  // 1D problems that fit stay resident for many steps.  ZA_LINE_SPIN=ticks or
  // ticks:n (tests): the wait limit of the launches, from the n-th (0: first) on.
  line_shape(*p, c->cus, &c->line_blocks, &c->line_waves);
  if (!resident_wanted()) c->line_blocks = 0;
  if (const char* e = std::getenv("ZA_LINE_SPIN")) {
    char* end = nullptr;
    c->line_spin = std::strtoll(e, &end, 10);
    if (*end == ':') c->line_spin_from = std::atoll(end + 1);
  }
}

// A right-hand side or flux sweep of q, whose speeds are in c->rows.
SweepArgs rhs_args(za_ctx* c, const double* q, double* out) {
  SweepArgs a = base_args(c);
  a.q = q;
  a.out = out;
  a.kind = FIN_RHS;
  a.sp_in = c->rows;
  a.sp_rows = c->red_blocks;
  return a;
}

// rhs = L(q): one launch where one block holds the line, else the wave-speed
// pass and a fused kernel, a 1D sweep or a pair of sweeps.
void launch_rhs(za_ctx* c, const double* q, double* rhs) {
  if (line_ready(c) && c->line_blocks == 1) {
    launch_line_rhs(c, q, rhs);
    return;
  }
  launch_speeds(c, q, 0, nullptr);
  SweepArgs a = rhs_args(c, q, rhs);
  if (c->fu_gx) {
    timed_begin(c, 1);
    launch_fused(c, MODE_RHS, a);
    timed_end(c, 1);
    return;
  }
  begin_apart(c, MODE_RHS, a);
  launch_x(c, MODE_RHS, a);
  if (c->prob.dim == 2) {
    a.lx = rhs;
    launch_y(c, MODE_RHS, a);
  }
}

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

// Whether stages are pairs of sweeps with a partial stage between them (2D
// scalar laws and limited Euler stages; the others are fused).
static bool needs_lx(const za_problem& p) { return p.dim == 2 && (p.system != ZA_EULER || p.pp_limiter); }

za_status za_ctx_create(const za_problem* p, void* stream, za_ctx** out) {
  if (!out) return ZA_ERR_ARG;
  *out = nullptr;
  std::string why;
  za_status st = za_validate(p, &why);
  if (st != ZA_OK) return st;
  za_ctx* c = new za_ctx();
  init_shape(c, p, (hipStream_t)stream);
  const size_t st_bytes = (size_t)c->m * p->nx * p->ny * sizeof(double);
  hipError_t e;
  void* ptr = nullptr;
  if ((e = hipMalloc(&ptr, st_bytes)) != hipSuccess) { delete c; return ZA_ERR_NOMEM; }
  c->q1 = (double*)ptr;
  if ((e = hipMalloc(&ptr, st_bytes)) != hipSuccess) { za_ctx_destroy(c); return ZA_ERR_NOMEM; }
  c->q2 = (double*)ptr;
  if (needs_lx(*p)) {
    if ((e = hipMalloc(&ptr, st_bytes)) != hipSuccess) { za_ctx_destroy(c); return ZA_ERR_NOMEM; }
    c->lx = (double*)ptr;
  }
  // one allocation: partial sums, wave-speed rows, control blocks, exchange words
  if ((e = hipMalloc(&ptr, kPartBytes + kRowsBytes + line_bytes(c->line_blocks))) != hipSuccess) {
    za_ctx_destroy(c);
    return ZA_ERR_NOMEM;
  }
  c->part = (double*)ptr;
  c->rows = (unsigned long long*)((char*)ptr + kPartBytes);
  c->ctl = (DevCtl*)(c->rows + SP_SETS * SP_SET);
  c->line_xch = (unsigned long long*)((char*)ptr + kPartBytes + kRowsBytes);
  line_init(c);
  launch_ctl(c, fresh_ctl());
  if ((e = hipGetLastError()) != hipSuccess) { za_ctx_destroy(c); return ZA_ERR_DEVICE; }
  *out = c;
  return ZA_OK;
}

za_status za_ctx_destroy(za_ctx* c) {
  if (!c) return ZA_ERR_ARG;
  if (c->stream || true) hipStreamSynchronize(c->stream);
  for (int k = 0; k < 3; ++k) {
    for (auto& pr : c->events[k]) { hipEventDestroy(pr.first); hipEventDestroy(pr.second); }
  }
  if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
  if (c->capture_stream) (void)hipStreamDestroy(c->capture_stream);
  if (c->q1) hipFree(c->q1);
  if (c->q2) hipFree(c->q2);
  if (c->lx) hipFree(c->lx);
  if (c->part) hipFree(c->part);
  delete c;
  return ZA_OK;
}

za_status za_ctx_set_stream(za_ctx* c, void* stream) {
  if (!c) return ZA_ERR_ARG;
  c->stream = (hipStream_t)stream;
  return ZA_OK;
}

za_status za_rhs(za_ctx* c, const double* q, double* rhs) {
  if (!c || !q || !rhs || q == rhs) return ZA_ERR_ARG;
  c->speeds_valid = false;
  launch_rhs(c, q, rhs);
  ZA_CHECK_LAUNCH(c, "rhs launch");
  return ZA_OK;
}

za_status za_rhs_fluxes(za_ctx* c, const double* q, double* fx, double* fy) {
  if (!c || !q || !fx) return ZA_ERR_ARG;
  c->speeds_valid = false;
  launch_speeds(c, q, 0, nullptr);
  SweepArgs a = rhs_args(c, q, fx);
  begin_apart(c, MODE_FLUX, a);
  launch_x(c, MODE_FLUX, a);
  if (c->prob.dim == 2 && fy) {
    a.out = fy;
    launch_y(c, MODE_FLUX, a);
  }
  ZA_CHECK_LAUNCH(c, "flux launch");
  return ZA_OK;
}

za_status za_step(za_ctx* c, double* q, double dt, double* dt_used) {
  if (!c || !q) return ZA_ERR_ARG;
  c->speeds_valid = false;
  if (!(dt > 0.0) && !(dt <= 0.0)) return ZA_ERR_ARG;  // NaN
  const DevCtl v = start_ctl(dt > 0.0 ? dt : 0.0, std::numeric_limits<double>::infinity(), 1);
  za_status st;
  if (line_ready(c) && c->line_blocks == 1) {
    launch_line(c, q, 1, &v);
    ZA_CHECK_LAUNCH(c, "step launch");
  } else {
    if ((st = enqueue_step(c, q, &v)) != ZA_OK) return st;
  }
  if (dt_used) {
    DevCtl h;
    if ((st = read_ctl(c, &h)) != ZA_OK) return st;
    *dt_used = h.dt;
    if (h.bad) return ZA_ERR_NONFINITE;
  }
  return ZA_OK;
}

za_status za_solve(za_ctx* c, double* q, double t_final, int64_t max_steps, za_solve_info* info) {
  if (!c || !q) return ZA_ERR_ARG;
  c->speeds_valid = false;
  if (!(t_final > 0.0) && max_steps <= 0) return ZA_ERR_ARG;
  if (t_final != t_final) return ZA_ERR_ARG;
  const auto& p = c->prob;
  const double inf = std::numeric_limits<double>::infinity();
  DevCtl h;
  za_status st;
  if (t_final > 0.0 && p.dt_rule == ZA_DT_CFL_H2) {
    // fixed dt = cfl h^2: n equal steps, the last one lands on t_final
    const double h2 = p.dim == 2 ? std::min(c->geom.dx, c->geom.dy) : c->geom.dx;
    const double dt = p.cfl * h2 * h2;
    const int64_t n = (int64_t)std::ceil(t_final / dt * (1.0 - 1e-12));
    int64_t n_run = n;
    if (max_steps > 0 && max_steps < n) n_run = max_steps;
    const int64_t n_equal = std::min<int64_t>(n_run, n - 1);
    h = start_ctl(dt, inf, n_equal);
    const DevCtl v = h;
    if (n_equal < 1) launch_ctl(c, v);
    for (int64_t s = 0; s < n_equal;) {
      int64_t k = n_equal - s;
      if ((st = advance(c, q, &k, true, s == 0 ? &v : nullptr, false, &h)) != ZA_OK) return st;
      s += k;
      if (s < n_equal && h.bad) break;
    }
    if (n_run == n) {
      const double last = t_final - (double)(n - 1) * dt;
      hipLaunchKernelGGL(k_ctl_arm, dim3(1), dim3(64), 0, c->stream, c->ctl, last, inf, (long long)n);
      if ((st = enqueue_step(c, q)) != ZA_OK) return st;
    }
    if ((st = read_ctl(c, &h)) != ZA_OK) return st;
    if (n_run == n && !h.bad) h.t = t_final;
  } else {
    const double tf = t_final > 0.0 ? t_final : inf;
    const DevCtl v = start_ctl(0.0, tf, max_steps > 0 ? max_steps : 0);
    // A fixed step count is enqueued exactly; integrating to t_final
    // enqueues chunks and lets the device retire the steps beyond t_final.
    int64_t enqueued = 0;
    while (true) {
      int64_t n = t_final <= 0.0 ? max_steps - enqueued : std::numeric_limits<int64_t>::max();
      if ((st = advance(c, q, &n, false, enqueued == 0 ? &v : nullptr, true, &h)) != ZA_OK) return st;
      enqueued += n;
      if (!h.active || h.bad) break;
      if (t_final <= 0.0 && enqueued >= max_steps) break;
    }
  }
  if (info) {
    info->steps = h.steps;
    info->t = h.t;
    info->dt_min = h.dt_min;
    info->dt_max = h.dt_max;
    info->nonfinite_step = h.bad ? h.bad_step : -1;
  }
  return h.bad ? ZA_ERR_NONFINITE : ZA_OK;
}

za_status za_conserved_sums(za_ctx* c, const double* q, double* sums) {
  if (!c || !q || !sums) return ZA_ERR_ARG;
  c->speeds_valid = false;
  const size_t ncell = (size_t)c->prob.nx * c->prob.ny;
  const int nblk = (int)std::min<size_t>((size_t)SUM_BLOCKS, std::max<size_t>(1, (ncell + 4095) / 4096));
  const size_t chunk = (ncell + nblk - 1) / nblk;
  hipLaunchKernelGGL(k_sum_partial, dim3(nblk, c->m), dim3(256), 0, c->stream, q, ncell, chunk, c->part);
  ZA_CHECK_LAUNCH(c, "sum launch");
  std::vector<double> part((size_t)nblk * c->m);
  const hipError_t e =
      hipMemcpyWithStream(part.data(), c->part, part.size() * sizeof(double), hipMemcpyDeviceToHost, c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "copy sums");
  for (int comp = 0; comp < c->m; ++comp) {
    double s = 0.0;
    for (int b = 0; b < nblk; ++b) s += part[(size_t)comp * nblk + b];
    sums[comp] = s;
  }
  return ZA_OK;
}

za_status za_ctx_set_timing(za_ctx* c, int32_t enable) {
  if (!c) return ZA_ERR_ARG;
  c->timing = enable != 0;
  return ZA_OK;
}

za_status za_ctx_kernel_times(za_ctx* c, double* avg_ms, int64_t* counts) {
  if (!c || !avg_ms) return ZA_ERR_ARG;
  hipError_t e = hipStreamSynchronize(c->stream);
  if (e != hipSuccess) return hip_fail(c, e, "synchronise");
  for (int k = 0; k < 3; ++k) {
    double tot = 0.0;
    for (auto& pr : c->events[k]) {
      float ms = 0.f;
      hipEventElapsedTime(&ms, pr.first, pr.second);
      tot += ms;
      hipEventDestroy(pr.first);
      hipEventDestroy(pr.second);
    }
    const size_t n = c->events[k].size();
    avg_ms[k] = n ? tot / (double)n : 0.0;
    if (counts) counts[k] = (int64_t)n;
    c->events[k].clear();
  }
  return ZA_OK;
}

}  // extern "C"
