// Launches of the resident 1D kernels (za_line.hpp): which problems take
// them, in what shape, and the steps and right-hand sides they run.
#include "za_line.hpp"

#include <algorithm>
#include <cstring>

#include "za_internal.hpp"

using namespace za;

namespace {

// Threads a block may have: FP64 Euler and the wide stencils need more than
// the 128 registers that 1024 threads leave each.  (FP32 Euler with squared
// weights spills 14 there; with 512 threads it is no faster up to 32,704 cells
// and loses the lines beyond: 40,000 cells 8.0 -> 9.2 us a stage.)
template <int SYS, class T, int WV, int R>
constexpr int line_threads() {
  const bool wide = sizeof(T) == sizeof(double) && (SYS == SYS_EULER || R > 3 || WV != WV_Z1);
  return wide ? 512 : 1024;
}

// Calls f.run<SYS, M, T, WV, R, PP>() for the kernels that p takes; false
// if there is none: weights with pow() and everything outside 1D.
template <int SYS, int M, class F>
bool line_dispatch_sys(const za_problem& p, F& f) {
  const bool gp = general_weights(p);
  if (gp && !square_powers(p)) return false;
  const bool f32 = p.precision == ZA_FP32_RECON;
  if (order_of(p) != 3) {
    if (gp || f32) return false;
    switch (order_of(p)) {
      case 2: f.template run<SYS, M, double, WV_Z1, 2, 0>(); return true;
      case 4: f.template run<SYS, M, double, WV_Z1, 4, 0>(); return true;
      default: f.template run<SYS, M, double, WV_Z1, 5, 0>(); return true;
    }
  }
  if (gp) {
    if (p.pp_limiter) return false;
    if (f32) f.template run<SYS, M, float, WV_SQUARE, 3, 0>();
    else f.template run<SYS, M, double, WV_SQUARE, 3, 0>();
    return true;
  }
  if constexpr (SYS == SYS_EULER) {
    if (p.pp_limiter) {
      f.template run<SYS, M, double, WV_Z1, 3, 1>();
      return true;
    }
  }
  if (f32) f.template run<SYS, M, float, WV_Z1, 3, 0>();
  else f.template run<SYS, M, double, WV_Z1, 3, 0>();
  return true;
}

template <class F>
bool line_dispatch(const za_problem& p, F&& f) {
  if (p.dim != 1) return false;
  switch (p.system) {
    case ZA_EULER: return line_dispatch_sys<SYS_EULER, 3>(p, f);
    case ZA_ADVECTION: return line_dispatch_sys<SYS_ADV, 1>(p, f);
    case ZA_BURGERS: return line_dispatch_sys<SYS_BURGERS, 1>(p, f);
    default: return line_dispatch_sys<SYS_BUCKLEY, 1>(p, f);
  }
}

struct MaxThreads {
  int threads = 0;
  template <int SYS, int M, class T, int WV, int R, int PP>
  void run() { threads = line_threads<SYS, T, WV, R>(); }
};

struct Solve {
  za_ctx* c;
  const LineArgs& a;
  template <int SYS, int M, class T, int WV, int R, int PP>
  void run() {
    constexpr int LB = line_threads<SYS, T, WV, R>();
    hipLaunchKernelGGL((k_line_solve<SYS, M, T, WV, R, PP, LB>), dim3(c->line_blocks), dim3(64 * c->line_waves), 0,
                       c->stream, a, make_cfg<T>(c->prob));
  }
};

struct Rhs {
  za_ctx* c;
  const LineArgs& a;
  template <int SYS, int M, class T, int WV, int R, int PP>
  void run() {
    constexpr int LB = line_threads<SYS, T, WV, R>();
    hipLaunchKernelGGL((k_line_rhs<SYS, M, T, WV, R, LB>), dim3(1), dim3(64 * c->line_waves), 0, c->stream, a,
                       make_cfg<T>(c->prob));
  }
};

__global__ void k_words_clear(unsigned long long* w, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) w[i] = 0;
}

}  // namespace

void line_shape(const za_problem& p, int cus, int* blocks, int* waves) {
  *blocks = *waves = 0;
  MaxThreads mt;
  if (!line_dispatch(p, mt)) return;
  const int max_waves = mt.threads / 64;
  // one block up to LINE_ONE_BLOCK wavefronts, else four wavefronts (one per
  // SIMD) per block, more only where the block count would pass its limit
  const int one = p.nx / 64 + 1;   // wavefronts holding nx + 1 interfaces
  const int one_max = std::min(max_waves, p.system != ZA_EULER ? LINE_ONE_BLOCK_SCALAR
                                          : order_of(p) > 3 || general_weights(p) ? LINE_ONE_BLOCK_WIDE
                                                                                  : LINE_ONE_BLOCK_EULER);
  if (one <= one_max) {
    *blocks = 1;
    *waves = one;
    return;
  }
  for (int w = std::min(4, max_waves); w <= max_waves; w *= 2) {
    const int cells = 64 * w - 1;
    const long long n = ((long long)p.nx + cells - 1) / cells;
    // a quarter of the wavefronts that the CUs hold at the kernel's registers:
    // the blocks wait for each other, so all have to be resident at once
    if (n <= LINE_MAX_BLOCKS && 4 * n * w <= (long long)cus * max_waves) {
      *blocks = (int)n;
      *waves = w;
      return;
    }
  }
}

size_t line_bytes(int blocks) { return blocks > 1 ? 2 * (size_t)LINE_WORDS * sizeof(unsigned long long) : 0; }

void line_init(za_ctx* c) {
  if (c->line_blocks > 1)
    hipLaunchKernelGGL(k_words_clear, dim3(16), dim3(256), 0, c->stream, c->line_xch, 2 * LINE_WORDS);
}

// wait limit of one exchange: 1 s of the 100 MHz clock
static constexpr long long kLineSpin = 100000000LL;

void launch_line(za_ctx* c, double* q, int64_t n, const DevCtl* init) {
  LineArgs a;
  std::memset(&a, 0, sizeof(a));
  a.q = q;
  a.out = c->q1;
  a.ctl = c->ctl;
  a.xch = c->line_xch;
  a.g = c->geom;
  a.ph = c->ph;
  if (init) { a.init = *init; a.arm = 1; }
  a.nsteps = (int)n;
  a.tag0 = c->line_tag;
  a.spin = c->line_spin >= 0 && c->line_launches >= c->line_spin_from ? c->line_spin : kLineSpin;
  ++c->line_launches;
  line_dispatch(c->prob, Solve{c, a});
  if (c->line_blocks > 1) {
    const size_t count = (size_t)c->m * c->prob.nx;
    hipLaunchKernelGGL(k_line_commit, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, c->stream, c->q1, q, count,
                       c->ctl, a.tag0);
  }
  c->line_tag += 3u * (unsigned)n + 2u;   // one exchange at the start and one per stage
}

void launch_line_rhs(za_ctx* c, const double* q, double* rhs) {
  LineArgs a;
  std::memset(&a, 0, sizeof(a));
  a.q = const_cast<double*>(q);
  a.out = rhs;
  a.ctl = c->ctl;
  a.g = c->geom;
  a.ph = c->ph;
  line_dispatch(c->prob, Rhs{c, a});
}
