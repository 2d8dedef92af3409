// Fused 2D Euler stages with Z weights at r = 3, and the launch shape of all
// of them.
#include "za_fused_launch.hpp"

using namespace za;

// The value of the kernel that p launches, by the conditions of launch_fused.
template <class T, int R>
static int fused_waves_t(const za_problem& p) {
  return !general_weights(p) ? FuWaves<T, WV_Z1, R>::value
         : square_powers(p)  ? FuWaves<T, WV_SQUARE, R>::value
                             : FuWaves<T, WV_GENERAL, R>::value;
}
int fused_waves(const za_problem& p) {
  if (p.precision == ZA_FP32_RECON) return fused_waves_t<float, 3>(p);
  switch (order_of(p)) {
    case 2: return fused_waves_t<double, 2>(p);
    case 3: return fused_waves_t<double, 3>(p);
    case 4: return fused_waves_t<double, 4>(p);
    default: return fused_waves_t<double, 5>(p);
  }
}

// Strips and bands: the band height that minimises the longest CU's work,
// counted in steps of one wavefront per SIMD.  A block of s steps covers
// 4 s - 1 rows.  n resident blocks per CU take n s steps of a CU's issue
// slots, times 1.5 for n = 1 and 1.15 for n = 2, which leave slots idle; a
// round of blocks adds 2 steps for its start (first loads and records) and
// the launch 1 more.  (Fitted over grids from 400^2 to 2048^2: FP64 stages
// take 9.5 us + 3.2 us per step; 1300 x 900: 76 us with the choice below, 98
// with one block per CU.)  Kernels of one block per CU take three to five
// times as long over a step, so half a step to start (2048^2, r = 5, squared
// weights: 1207 us with four rounds of 17 steps, 1229 with two of 35).
//
// A strip takes whole wavefronts however narrow it is: on grids of fewer than
// 8 columns (20 at r = 4, 5) an x-sweep and a y-sweep that packs four rows of
// 16 columns are faster (4 x 100000: 257 us a stage, fused 322), but there a
// state would not be the served one's bits.
void fused_shape(const za_problem& p, int cus, int* gx, int* gy) {
  *gx = *gy = 0;
  if (p.dim != 2 || p.system != ZA_EULER) return;
  const int res = fused_waves(p);   // resident blocks per CU of the kernel that p launches
  const int strips = (p.nx + FU_COLS - 1) / FU_COLS;
  const double start = res == 1 ? 0.5 : 2.0;
  double best = -1;
  // (bands of more than 256 steps only where the grid would have too many)
  for (long long s = 1;; s = s < 256 ? s + 1 : 2 * s) {
    const long long h = FU_NW * s - 1;   // rows of a band of s steps
    const long long nb = (p.ny + h - 1) / h;
    if (nb > 65535) continue;
    const long long m = (strips * nb + cus - 1) / cus;
    const long long full = m / res, rest = m % res;
    const double idle = rest == 1 ? 1.5 : (rest == 2 && res > 2 ? 1.15 : 1.0);
    const double cost = full * (res * s + start) + (rest ? idle * rest * s + start : 0.0);
    if (best < 0 || cost < best) { best = cost; *gx = strips; *gy = (int)nb; }
    if (m <= 1 || s >= 256) break;   // from here on only slower
  }
}

void launch_fused(za_ctx* c, int mode, SweepArgs a) {
  a.ytile = c->fu_gy;
  a.nblk = c->fu_gx * c->fu_gy;
  if (order_of(c->prob) != 3) launch_fused_order(c, mode, a);
  else if (!general_weights(c->prob)) {
    if (c->prob.precision == ZA_FP32_RECON) launch_fused_t<float, WV_Z1, 3>(c, mode, a);
    else launch_fused_t<double, WV_Z1, 3>(c, mode, a);
  } else if (square_powers(c->prob)) launch_fused_square(c, mode, a);
  else launch_fused_general(c, mode, a);
}
