// Fused 2D Euler stages of the fourth-, eighth- and tenth-order schemes (FP64).
#include "za_fused_launch.hpp"

using namespace za;

template <int R>
static void by_weights(za_ctx* c, int mode, const SweepArgs& a) {
  if (!general_weights(c->prob)) launch_fused_t<double, WV_Z1, R>(c, mode, a);
  else if (square_powers(c->prob)) launch_fused_t<double, WV_SQUARE, R>(c, mode, a);
  else launch_fused_t<double, WV_GENERAL, R>(c, mode, a);
}

void launch_fused_order(za_ctx* c, int mode, const SweepArgs& a) {
  switch (order_of(c->prob)) {
    case 2: by_weights<2>(c, mode, a); break;
    case 4: by_weights<4>(c, mode, a); break;
    default: by_weights<5>(c, mode, a); break;
  }
}
