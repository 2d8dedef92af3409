// Launches of the fused 2D Euler stage for one weight variant and order; each
// translation unit that includes this instantiates its own kernels.
#pragma once
#include "za_fused.hpp"
#include "za_internal.hpp"

namespace za {

// Wavefronts per SIMD (= blocks per CU) that the registers and the LDS ring
// allow.  FP64 Z weights: 168 registers and 50 KB of LDS give three, FP32
// four; the general weights and the wider stencils hold two, both together
// (and pow()) one without spills.
template <class T, int WV, int R>
struct FuWaves {
  enum { f32 = sizeof(T) == sizeof(float),
         value = WV == WV_GENERAL ? (f32 ? 2 : 1)
                 : WV == WV_SQUARE ? (f32 ? 3 : (R > 3 ? 1 : 2))
                                   : (R == 3 ? (f32 ? 4 : 3) : (R == 2 ? 3 : 2)) };
};

template <class T, int WV, int R>
void launch_fused_t(za_ctx* c, int mode, const SweepArgs& a) {
  const CfgArg<T> cfg = make_cfg<T>(c->prob);
  const dim3 grid(c->fu_gx, c->fu_gy), blk(64 * FU_NW);
  constexpr int W = FuWaves<T, WV, R>::value;
  if (mode == MODE_STAGE)
    hipLaunchKernelGGL((k_fused<T, WV, R, MODE_STAGE, W>), grid, blk, 0, c->stream, a, cfg);
  else
    hipLaunchKernelGGL((k_fused<T, WV, R, MODE_RHS, W>), grid, blk, 0, c->stream, a, cfg);
}

}  // namespace za
