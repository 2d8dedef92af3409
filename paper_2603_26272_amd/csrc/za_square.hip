// Sixth-order sweeps with general weights, exponents all 1 or 2 (WV_SQUARE).
#include "za_fused_launch.hpp"
#include "za_launch.hpp"

using namespace za;

void launch_x_square(za_ctx* c, int mode, const SweepArgs& a) { launch_x_wv<WV_SQUARE>(c, mode, a); }
void launch_y_square(za_ctx* c, int mode, const SweepArgs& a) { launch_y_wv<WV_SQUARE>(c, mode, a); }
int square_y_blocks_per_cu(const za_problem& p) { return y_blocks_per_cu_wv<WV_SQUARE>(p); }
void launch_fused_square(za_ctx* c, int mode, const SweepArgs& a) {
  if (c->prob.precision == ZA_FP32_RECON) launch_fused_t<float, WV_SQUARE, 3>(c, mode, a);
  else launch_fused_t<double, WV_SQUARE, 3>(c, mode, a);
}
