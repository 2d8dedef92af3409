// Separate sweeps of the fourth-, eighth- and tenth-order central-upwind schemes
// (r = 2, 4, 5; Appendix A) in FP64: the WENO-ZA6 kernels and launch shapes
// with the stencil half-width as a template parameter; Z weights with an
// occupancy target, the other weight variants (and flux output) through the
// general kernels.
#include "za_internal.hpp"

using namespace za;

namespace {

// resident wavefronts per SIMD requested for the Z-weight kernels
template <int R> struct OrderWaves;
template <> struct OrderWaves<2> { enum { x = 5, y = 3 }; };
template <> struct OrderWaves<4> { enum { x = 3, y = 2 }; };
template <> struct OrderWaves<5> { enum { x = 2, y = 2 }; };

// Z weights with p = 1 take the occupancy-targeted kernels; Ai, p != 1 and
// linear weights the general ones (without pow() where every exponent is 1
// or 2, which covers the flux output of Z weights).

template <int SYS, int M, int R, int WV>
void x_any(za_ctx* c, int mode, const SweepArgs& a, const CfgArg<double>& cfg, dim3 grid) {
  if (mode == MODE_FLUX) {
    hipLaunchKernelGGL((k_sweep_x_any<SYS, M, double, MODE_FLUX, WV, R>), grid, dim3(256), 0, c->stream, a, cfg);
    return;
  }
  if constexpr (SYS == SYS_EULER && M == 3 && R == 2 && WV == WV_GENERAL) {   // 130 registers, 128 give four
    if (mode == MODE_RHS)
      hipLaunchKernelGGL((k_sweep_x_r<SYS, M, double, MODE_RHS, WV, R, 4>), grid, dim3(256), 0, c->stream, a, cfg);
    else
      hipLaunchKernelGGL((k_sweep_x_r<SYS, M, double, MODE_STAGE, WV, R, 4>), grid, dim3(256), 0, c->stream, a, cfg);
  } else if constexpr (M != 4) switch (mode) {
    case MODE_RHS: hipLaunchKernelGGL((k_sweep_x_any<SYS, M, double, MODE_RHS, WV, R>), grid, dim3(256), 0, c->stream, a, cfg); break;
    case MODE_LX: hipLaunchKernelGGL((k_sweep_x_any<SYS, M, double, MODE_LX, WV, R>), grid, dim3(256), 0, c->stream, a, cfg); break;
    default: hipLaunchKernelGGL((k_sweep_x_any<SYS, M, double, MODE_STAGE, WV, R>), grid, dim3(256), 0, c->stream, a, cfg); break;
  }
}

template <int SYS, int M, int R>
void x_sys(za_ctx* c, int mode, SweepArgs a) {
  const CfgArg<double> cfg = make_cfg<double>(c->prob);
  const int nseg = (a.g.nx + XS_CELLS - 1) / XS_CELLS;
  const long long waves = (long long)a.g.ny * nseg;
  const dim3 grid((unsigned)((waves + 3) / 4)), blk(256);
  a.nblk = (int)grid.x;
  constexpr int XW = OrderWaves<R>::x;
  if constexpr (M != 4) if (!general_weights(c->prob) && mode != MODE_FLUX) {
    switch (mode) {
      case MODE_RHS: hipLaunchKernelGGL((k_sweep_x_r<SYS, M, double, MODE_RHS, WV_Z1, R, XW>), grid, blk, 0, c->stream, a, cfg); break;
      case MODE_LX: hipLaunchKernelGGL((k_sweep_x_r<SYS, M, double, MODE_LX, WV_Z1, R, XW>), grid, blk, 0, c->stream, a, cfg); break;
      default: hipLaunchKernelGGL((k_sweep_x_r<SYS, M, double, MODE_STAGE, WV_Z1, R, XW>), grid, blk, 0, c->stream, a, cfg); break;
    }
    return;
  }
  if (square_powers(c->prob)) x_any<SYS, M, R, WV_SQUARE>(c, mode, a, cfg, grid);
  else x_any<SYS, M, R, WV_GENERAL>(c, mode, a, cfg, grid);
}

template <int SYS, int M, int R, int WV>
void y_any(za_ctx* c, int mode, const SweepArgs& a, const CfgArg<double>& cfg, dim3 grid) {
  if (mode == MODE_FLUX) {
    if constexpr (SYS == SYS_EULER && M == 4 && R == 2 && WV == WV_GENERAL)   // 171 registers, 168 give three
      hipLaunchKernelGGL((k_sweep_y_r<SYS, M, double, MODE_FLUX, WV, R, 3>), grid, dim3(256), 0, c->stream, a, cfg);
    else
      hipLaunchKernelGGL((k_sweep_y_any<SYS, M, double, MODE_FLUX, WV, R>), grid, dim3(256), 0, c->stream, a, cfg);
    return;
  }
  if constexpr (M != 4) switch (mode) {
    case MODE_RHS: hipLaunchKernelGGL((k_sweep_y_any<SYS, M, double, MODE_RHS, WV, R>), grid, dim3(256), 0, c->stream, a, cfg); break;
    default: hipLaunchKernelGGL((k_sweep_y_any<SYS, M, double, MODE_STAGE, WV, R>), grid, dim3(256), 0, c->stream, a, cfg); break;
  }
}

template <int SYS, int M, int R>
void y_sys(za_ctx* c, int mode, const SweepArgs& a) {
  const CfgArg<double> cfg = make_cfg<double>(c->prob);
  const dim3 grid((unsigned)((a.g.nx + 63) / 64), (unsigned)((a.g.ny + a.ytile - 1) / a.ytile)), blk(256);
  constexpr int YW = OrderWaves<R>::y;
  if constexpr (M != 4) if (!general_weights(c->prob) && mode != MODE_FLUX) {
    if (mode == MODE_RHS)
      hipLaunchKernelGGL((k_sweep_y_r<SYS, M, double, MODE_RHS, WV_Z1, R, YW>), grid, blk, 0, c->stream, a, cfg);
    else
      hipLaunchKernelGGL((k_sweep_y_r<SYS, M, double, MODE_STAGE, WV_Z1, R, YW>), grid, blk, 0, c->stream, a, cfg);
    return;
  }
  if (square_powers(c->prob)) y_any<SYS, M, R, WV_SQUARE>(c, mode, a, cfg, grid);
  else y_any<SYS, M, R, WV_GENERAL>(c, mode, a, cfg, grid);
}

template <int R>
void x_order(za_ctx* c, int mode, const SweepArgs& a) {
  switch (c->prob.system) {
    case ZA_EULER:
      if (c->prob.dim == 1) x_sys<SYS_EULER, 3, R>(c, mode, a); else x_sys<SYS_EULER, 4, R>(c, mode, a);
      break;
    case ZA_ADVECTION: x_sys<SYS_ADV, 1, R>(c, mode, a); break;
    case ZA_BURGERS: x_sys<SYS_BURGERS, 1, R>(c, mode, a); break;
    default: x_sys<SYS_BUCKLEY, 1, R>(c, mode, a); break;
  }
}

template <int R>
void y_order(za_ctx* c, int mode, const SweepArgs& a) {
  switch (c->prob.system) {
    case ZA_EULER: y_sys<SYS_EULER, 4, R>(c, mode, a); break;
    case ZA_ADVECTION: y_sys<SYS_ADV, 1, R>(c, mode, a); break;
    case ZA_BURGERS: y_sys<SYS_BURGERS, 1, R>(c, mode, a); break;
    default: y_sys<SYS_BUCKLEY, 1, R>(c, mode, a); break;
  }
}

}  // namespace

void launch_x_order(za_ctx* c, int mode, const SweepArgs& a) {
  switch (order_of(c->prob)) {
    case 2: x_order<2>(c, mode, a); break;
    case 4: x_order<4>(c, mode, a); break;
    default: x_order<5>(c, mode, a); break;
  }
}

void launch_y_order(za_ctx* c, int mode, const SweepArgs& a) {
  switch (order_of(c->prob)) {
    case 2: y_order<2>(c, mode, a); break;
    case 4: y_order<4>(c, mode, a); break;
    default: y_order<5>(c, mode, a); break;
  }
}

// Resident blocks per CU of the stage y-sweep of this order (scalar laws;
// for the band height); 0 if unknown.
int order_y_blocks_per_cu(const za_problem& p) {
  const void* fn = nullptr;
  const bool gp = general_weights(p), sq = gp && square_powers(p);
#define ZA_YFN(R)                                                                                          \
  (sq   ? reinterpret_cast<const void*>(&k_sweep_y_any<SYS_ADV, 1, double, MODE_STAGE, WV_SQUARE, R>)  \
   : gp ? reinterpret_cast<const void*>(&k_sweep_y_any<SYS_ADV, 1, double, MODE_STAGE, WV_GENERAL, R>) \
        : reinterpret_cast<const void*>(&k_sweep_y_r<SYS_ADV, 1, double, MODE_STAGE, WV_Z1, R, OrderWaves<R>::y>))
  switch (order_of(p)) {
    case 2: fn = ZA_YFN(2); break;
    case 4: fn = ZA_YFN(4); break;
    default: fn = ZA_YFN(5); break;
  }
#undef ZA_YFN
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, 256, 0) != hipSuccess) return 0;
  return n;
}
