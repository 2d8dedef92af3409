// Sweep launches of one weight variant (WV), for every system, precision and
// mode.  Each variant's kernels are instantiated in a translation unit of its
// own: za_lib.hip (WV_Z1), za_square.hip (WV_SQUARE), za_general.hip
// (WV_GENERAL).
#pragma once
#include "za_internal.hpp"

namespace za {

// 2D Euler stages and right-hand sides are fused (za_fused.hpp): of the
// separate sweeps there remain the flux output and the limited stages.
template <int SYS, int M, class T, int WV>
static void launch_x_t(za_ctx* c, int mode, SweepArgs a) {
  const CfgArg<T> cfg = make_cfg<T>(c->prob);
  const int nseg = (a.g.nx + XS_CELLS - 1) / XS_CELLS;
  const long long waves = (long long)a.g.ny * nseg;
  const dim3 grid((unsigned)((waves + 3) / 4)), blk(256);
  a.nblk = (int)grid.x;
  if constexpr (SYS == SYS_EULER && sizeof(T) == sizeof(double)) {
    if (c->ph.pp && mode == (M == 3 ? MODE_STAGE : MODE_LX)) {
      hipLaunchKernelGGL((k_sweep_x_pp<M, (M == 3 ? MODE_STAGE : MODE_LX), WV>), grid, blk, 0, c->stream, a, cfg);
      return;
    }
  }
  if (mode == MODE_FLUX) {
    if constexpr (SYS == SYS_EULER && M == 4 && WV == WV_GENERAL && sizeof(T) == sizeof(float))
      // five wavefronts per SIMD: 97 registers where 96 give them
      hipLaunchKernelGGL((k_sweep_x_r<SYS, M, T, MODE_FLUX, WV, 3, 5>), grid, blk, 0, c->stream, a, cfg);
    else
      hipLaunchKernelGGL((k_sweep_x_any<SYS, M, T, MODE_FLUX, WV>), grid, blk, 0, c->stream, a, cfg);
    return;
  }
  if constexpr (M != 4) {
    if constexpr (sizeof(T) == sizeof(double) && WV == WV_Z1) {
      if ((mode == MODE_LX || mode == MODE_STAGE) && a.xl_chunks > 0) {
        const long long w = xl_waves(a.g.nx, a.g.ny, a.xl_chunks);
        const dim3 gl((unsigned)((w + 3) / 4));
        a.nblk = (int)gl.x;
        if constexpr (SYS != SYS_EULER) {
          if (mode == MODE_LX) {
            hipLaunchKernelGGL((k_sweep_xl<SYS, M, WV, MODE_LX>), gl, blk, 0, c->stream, a, cfg);
            return;
          }
        }
        hipLaunchKernelGGL((k_sweep_xl<SYS, M, WV, MODE_STAGE>), gl, blk, 0, c->stream, a, cfg);
        return;
      }
    }
    if constexpr (WV == WV_Z1) {
      if (mode == MODE_RHS)
        hipLaunchKernelGGL((k_sweep_x<SYS, M, T, MODE_RHS, WV>), grid, blk, 0, c->stream, a, cfg);
      else if (mode == MODE_STAGE)
        hipLaunchKernelGGL((k_sweep_x<SYS, M, T, MODE_STAGE, WV>), grid, blk, 0, c->stream, a, cfg);
      else if constexpr (SYS != SYS_EULER)
        hipLaunchKernelGGL((k_sweep_x<SYS, M, T, MODE_LX, WV>), grid, blk, 0, c->stream, a, cfg);
    } else if constexpr (SYS == SYS_EULER && WV == WV_GENERAL && sizeof(T) == sizeof(double)) {
      // three wavefronts per SIMD: 170 registers where 168 give them (line of
      // 4e6 cells, p = 3/2: 679 us a stage, 760 with two)
      if (mode == MODE_RHS)
        hipLaunchKernelGGL((k_sweep_x_r<SYS, M, T, MODE_RHS, WV, 3, 3>), grid, blk, 0, c->stream, a, cfg);
      else
        hipLaunchKernelGGL((k_sweep_x_r<SYS, M, T, MODE_STAGE, WV, 3, 3>), grid, blk, 0, c->stream, a, cfg);
    } else {
      if (mode == MODE_RHS)
        hipLaunchKernelGGL((k_sweep_x_any<SYS, M, T, MODE_RHS, WV>), grid, blk, 0, c->stream, a, cfg);
      else if (mode == MODE_STAGE)
        hipLaunchKernelGGL((k_sweep_x_any<SYS, M, T, MODE_STAGE, WV>), grid, blk, 0, c->stream, a, cfg);
      else if constexpr (SYS != SYS_EULER)
        hipLaunchKernelGGL((k_sweep_x_any<SYS, M, T, MODE_LX, WV>), grid, blk, 0, c->stream, a, cfg);
    }
  }
}

template <int SYS, int M, class T, int WV>
static void launch_y_t(za_ctx* c, int mode, const SweepArgs& a) {
  const CfgArg<T> cfg = make_cfg<T>(c->prob);
  const dim3 grid((unsigned)((a.g.nx + 63) / 64), (unsigned)((a.g.ny + a.ytile - 1) / a.ytile)), blk(256);
  if (mode == MODE_FLUX) {
    hipLaunchKernelGGL((k_sweep_y_any<SYS, M, T, MODE_FLUX, WV>), grid, blk, 0, c->stream, a, cfg);
    return;
  }
  if constexpr (SYS == SYS_EULER) {
    if constexpr (sizeof(T) == sizeof(double)) {
      if (mode == MODE_STAGE)   // limited
        hipLaunchKernelGGL((k_sweep_y_pp<MODE_STAGE, WV>), grid, blk, 0, c->stream, a, cfg);
    }
  } else if constexpr (WV == WV_Z1) {
    if (mode == MODE_RHS)
      hipLaunchKernelGGL((k_sweep_y<SYS, M, T, MODE_RHS, WV>), grid, blk, 0, c->stream, a, cfg);
    else
      hipLaunchKernelGGL((k_sweep_y<SYS, M, T, MODE_STAGE, WV>), grid, blk, 0, c->stream, a, cfg);
  } else {
    if (mode == MODE_RHS)
      hipLaunchKernelGGL((k_sweep_y_any<SYS, M, T, MODE_RHS, WV>), grid, blk, 0, c->stream, a, cfg);
    else
      hipLaunchKernelGGL((k_sweep_y_any<SYS, M, T, MODE_STAGE, WV>), grid, blk, 0, c->stream, a, cfg);
  }
}

template <int WV>
void launch_x_wv(za_ctx* c, int mode, const SweepArgs& a) {
  const bool f32 = c->prob.precision == ZA_FP32_RECON;
#define ZA_X(SYS, M) (f32 ? launch_x_t<SYS, M, float, WV>(c, mode, a) : launch_x_t<SYS, M, double, WV>(c, mode, a))
  switch (c->prob.system) {
    case ZA_EULER:
      if (c->prob.dim == 1) ZA_X(SYS_EULER, 3); else ZA_X(SYS_EULER, 4);
      break;
    case ZA_ADVECTION: ZA_X(SYS_ADV, 1); break;
    case ZA_BURGERS: ZA_X(SYS_BURGERS, 1); break;
    default: ZA_X(SYS_BUCKLEY, 1); break;
  }
#undef ZA_X
}

template <int WV>
void launch_y_wv(za_ctx* c, int mode, const SweepArgs& a) {
  const bool f32 = c->prob.precision == ZA_FP32_RECON;
#define ZA_Y(SYS, M) (f32 ? launch_y_t<SYS, M, float, WV>(c, mode, a) : launch_y_t<SYS, M, double, WV>(c, mode, a))
  switch (c->prob.system) {
    case ZA_EULER: ZA_Y(SYS_EULER, 4); break;
    case ZA_ADVECTION: ZA_Y(SYS_ADV, 1); break;
    case ZA_BURGERS: ZA_Y(SYS_BURGERS, 1); break;
    default: ZA_Y(SYS_BUCKLEY, 1); break;
  }
#undef ZA_Y
}

// Resident blocks per CU of the y-sweep that a stage of p launches (for the
// band height; Euler: the limited one); 0 if unknown.
template <int WV>
int y_blocks_per_cu_wv(const za_problem& p) {
  const void* fn;
  if (p.system != ZA_EULER) {
    if constexpr (WV == WV_Z1)
      fn = p.precision == ZA_FP32_RECON ? reinterpret_cast<const void*>(&k_sweep_y<SYS_ADV, 1, float, MODE_STAGE, WV>)
                                        : reinterpret_cast<const void*>(&k_sweep_y<SYS_ADV, 1, double, MODE_STAGE, WV>);
    else
      fn = p.precision == ZA_FP32_RECON
               ? reinterpret_cast<const void*>(&k_sweep_y_any<SYS_ADV, 1, float, MODE_STAGE, WV>)
               : reinterpret_cast<const void*>(&k_sweep_y_any<SYS_ADV, 1, double, MODE_STAGE, WV>);
  } else {
    fn = reinterpret_cast<const void*>(&k_sweep_y_pp<MODE_STAGE, WV>);
  }
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, 256, 0) != hipSuccess) return 0;
  return n;
}

}  // namespace za
