// Launches of the fused 2D Euler stage for one weight variant and order; each
// translation unit that includes this instantiates its own kernels.
#pragma once
#include "za_fused.hpp"
#include "za_internal.hpp"

namespace za {

// Wavefronts per SIMD (= blocks per CU) of a launch that fills the device.
// FP64 Z weights: 168 registers and 50 KB of LDS give three, FP32 four; the
// general weights and the wider stencils hold two (r = 2 and FP32 with pow()
// three).  Three of these spill to scratch memory (bytes per lane: squared
// weights at r = 4 72, pow() at r = 4 and 2 112), which wins where blocks share
// CUs and loses where few do: `alone` is the value, free of scratch, for
// launches of at most that many blocks per CU.  At r = 5 two blocks would
// spill 280 and 304 bytes per lane, for which the runtime sets aside about 150
// MB per queue: those kernels take one.
//
// us a stage of 1024^2 (128^2), at one, two and three blocks per CU: squared r =
// 4 229, 163 (20.2, 21.5), r = 5 320, 283 (26.3, 30.3).  pow(), p = 3/2 (two
// sweeps: r = 2 403, r = 3 749, r = 4 938, r = 5 1442, FP32 348): r = 2 -, 418, 378
// (-, 41.6, 43.0), r = 3 868, 558, r = 4 1124, 732, r = 5 1314, 944, FP32 -, 382,
// 298 and 357 at four.
template <class T, int WV, int R>
struct FuWaves {
  enum { f32 = sizeof(T) == sizeof(float),
         value = WV == WV_Z1 ? (R == 3 ? (f32 ? 4 : 3) : (R == 2 ? 3 : 2))
                 : f32       ? 3
                 : R == 5    ? 1
                             : (WV == WV_GENERAL && R == 2 ? 3 : 2),
         alone = WV == WV_Z1 || f32              ? (int)value
                 : R == 4                        ? 1
                 : (WV == WV_GENERAL && R == 2)  ? 2
                                                 : (int)value };
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
    if ((long long)c->fu_gx * c->fu_gy <= (long long)W::alone * c->cus) {
      launch_fused_w<T, WV, R, W::alone>(c, mode, a);
      return;
    }
  }
  launch_fused_w<T, WV, R, W::value>(c, mode, a);
}

}  // namespace za
