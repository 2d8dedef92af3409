// Sixth-order sweeps with general weights, any exponents (WV_GENERAL).
#include "za_fused_launch.hpp"
#include "za_launch.hpp"

using namespace za;

void launch_x_general(za_ctx* c, int mode, const SweepArgs& a) { launch_x_wv<WV_GENERAL>(c, mode, a); }
void launch_y_general(za_ctx* c, int mode, const SweepArgs& a) { launch_y_wv<WV_GENERAL>(c, mode, a); }
int general_y_blocks_per_cu(const za_problem& p) { return y_blocks_per_cu_wv<WV_GENERAL>(p); }
void launch_fused_general(za_ctx* c, int mode, const SweepArgs& a) {
  if (c->prob.precision == ZA_FP32_RECON) launch_fused_t<float, WV_GENERAL, 3>(c, mode, a);
  else launch_fused_t<double, WV_GENERAL, 3>(c, mode, a);
}
