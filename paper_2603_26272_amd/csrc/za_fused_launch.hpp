// Launches of the fused 2D Euler stage for one weight variant and order; each
// translation unit that includes this instantiates its own kernels.
#pragma once
#include "za_fused.hpp"
#include "za_internal.hpp"

namespace za {

// Wavefronts per SIMD (= blocks per CU) of a launch that fills the device.
// FP64 Z weights: 168 registers and 50 KB of LDS give three, FP32 four; the
// general weights and the wider stencils hold two.  The squared weights at
// r = 4, 5 spill 37 and 113 registers to scratch at two, which still wins
// where blocks share CUs (us a stage, two against one: r = 4, 512^2 61 / 70,
// 2048^2 597 / 881; r = 5 99 / 97 and 1098 / 1229) and loses where none do
// (128^2: r = 4 21.5 / 20.2, r = 5 30.3 / 26.3): `alone` is the value for
// launches of at most one block per CU.  Weights with pow() (p = 3/2, us a
// stage of 1024^2; two sweeps per stage 403, 749, 938, 1442, FP32 348): r = 2
// 418 at two, 378 at three, r = 3 868 at one, 558 at two, r = 4 1124, 732,
// r = 5 1453, 944, FP32 382 at two, 298 at three, 357 at four.
template <class T, int WV, int R>
struct FuWaves {
  enum { f32 = sizeof(T) == sizeof(float),
         value = WV == WV_GENERAL ? (f32 || R == 2 ? 3 : 2)
                 : WV == WV_SQUARE ? (f32 ? 3 : 2)
                                   : (R == 3 ? (f32 ? 4 : 3) : (R == 2 ? 3 : 2)),
         alone = WV == WV_SQUARE && R > 3 ? 1 : (int)value };
};

template <class T, int WV, int R, int WAVES>
void launch_fused_w(za_ctx* c, int mode, const SweepArgs& a) {
  const CfgArg<T> cfg = make_cfg<T>(c->prob);
  const dim3 grid(c->fu_gx, c->fu_gy), blk(64 * FU_NW);
  if (mode == MODE_STAGE)
    hipLaunchKernelGGL((k_fused<T, WV, R, MODE_STAGE, WAVES>), grid, blk, 0, c->stream, a, cfg);
  else
    hipLaunchKernelGGL((k_fused<T, WV, R, MODE_RHS, WAVES>), grid, blk, 0, c->stream, a, cfg);
}

template <class T, int WV, int R>
void launch_fused_t(za_ctx* c, int mode, const SweepArgs& a) {
  typedef FuWaves<T, WV, R> W;
  if constexpr ((int)W::alone != (int)W::value) {
    if ((long long)c->fu_gx * c->fu_gy <= c->cus) {
      launch_fused_w<T, WV, R, W::alone>(c, mode, a);
      return;
    }
  }
  launch_fused_w<T, WV, R, W::value>(c, mode, a);
}

}  // namespace za
