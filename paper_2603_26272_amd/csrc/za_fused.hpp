// Fused 2D Euler stage: both sweeps of a stage in one kernel.
//
// A block of four wavefronts owns a strip of at most 63 columns and a band of
// rows, and marches up the band four interface rows per step.  The records
// of the 2R + 3 cell rows that one step's stencils touch (with R halo columns
// per side) sit in an LDS ring and serve both directions.  Wavefront
// w of a step computes the 63 y-interfaces of row k = k0 + w, then the 64
// x-interfaces of cell row r = k - 1, and completes that row's cells: the
// x-differences come from the next lane, the y-differences from the flux rows
// in LDS.
//
// Bound: FP64 vector issue (690 of 800 instructions per interface) and, over
// milliseconds, the board's power: data that vary everywhere run an eighth
// slower than constant quadrants (2.01 against 2.30 GHz).  Against an x-sweep
// that wrote a partial stage and a y-sweep that read it, HBM traffic per cell
// and stage falls from 181 to 85 bytes, records are built once, and a stage is
// one launch.  Per stage, before -> now (with the separate reduction launch
// before): 2048^2 FP64 277 -> 246 us, 512^2 39 -> 28 us, 128^2 24.7 -> 11.3 us;
// 2048^2 FP32 208 -> 174 us; 512^2 JS weights (without pow()) 53 -> 42 us,
// tenth order 72 -> 65 us.
//
// Shape.  64 x-interfaces take 63 columns; the y-interfaces of the same
// columns leave one lane idle.  Four wavefronts per block, one per SIMD: of
// six, two land on the same SIMDs in every block (2048^2: 375 us), and one
// block of eight or twelve stalls as a whole at its barriers (306, 300 us).
// Three blocks per CU need the records in 8 fields (with flux fields the ring
// fits twice: 267 us) and 168 registers, so the loads for the end of a step
// wait until its fluxes are done and cell i's flux is read twice.  The
// falling issue priority keeps the blocks of a CU level (without: 270 us).
#pragma once
#include "za_kernels.hpp"

namespace za {

constexpr int FU_COLS = 63;        // columns of a strip: 64 x-interfaces per row
constexpr int FU_NW = 4;           // wavefronts of a block, one per SIMD

// x of the next lane (wave_shl 1)
__device__ __forceinline__ double fu_next(double x) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)lo_word(x), 0x130, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)hi_word(x), 0x130, 0xf, 0xf, false);
  return from_words((unsigned)lo, (unsigned)hi);
}

template <class T, int WV, int R, int MODE>
__device__ __forceinline__ void fused_body(const SweepArgs& a, const CfgArg<T>& cfg, int bx, int by, int gx) {
  constexpr int NW = FU_NW, NF = Layout2<T>::NF;
  constexpr int FU_RECS = FU_COLS + 2 * R;                       // records per ring row
  constexpr int ROWS = NW + 2 * R - 1, RS = NF * FU_RECS;        // ring rows, row stride
  // FP32 records leave the registers to issue a step's loads before its
  // x-fluxes (1024^2 53.0 -> 51.1 us a stage, 2048^2 177 -> 174); FP64 just
  // fits them too and gains nothing (2048^2 251.3, 250.6).
  constexpr bool EARLY = sizeof(T) == sizeof(float) && WV == WV_Z1 && R == 3;
  constexpr bool REREAD = sizeof(T) == sizeof(double) && MODE == MODE_STAGE;
  static_assert(NW * 16 == 64 && 2 * R - 1 <= 16, "one wavefront loads a step's last halo columns");
  __shared__ T ring[ROWS * RS];
  __shared__ double fb[NW + 1][4][FU_COLS];
  __shared__ double sc[10];   // the stage's constants: speeds, dt, whether it runs
  const int lane = threadIdx.x & 63, w = wave_id();
  const int nx = a.g.nx, ny = a.g.ny;
  const size_t cs = (size_t)nx * ny;
  const int x0 = (int)((long long)bx * nx / gx), wc = (int)((long long)(bx + 1) * nx / gx) - x0;
  const int nb = a.ytile;            // bands
  const int y0 = (int)((long long)by * ny / nb), ylast = (int)((long long)(by + 1) * ny / nb);
  double rs[NPART];
#pragma unroll
  for (int t = 0; t < NPART; ++t) rs[t] = -__builtin_huge_val();
  // this lane's record columns: lane, and for the last few halo columns 64 + lane
  const bool in0 = lane < wc + 2 * R, in1 = lane + 64 < wc + 2 * R;
  const unsigned xa = bc_map_span(x0 - R + lane, x0 - R, 64, nx, a.g.bc_x);
  const unsigned xb = in1 ? bc_map(x0 - R + 64 + lane, nx, a.g.bc_x) : 0;
  const int xh = bc_map(x0 - R + 64 + (lane & 15), nx, a.g.bc_x);
  // The last wavefront prepares the stage's constants while the others build
  // the records of the first rows (all of them doing both: 128^2 12.4 us a
  // stage, now 11.7; 1024^2 FP32 54.6, 53.0).
  if (w == NW - 1) {
    StageLoads<SYS_EULER, 2> sl;
    stage_load(a, sl);
    SweepConst k0, k1;
    const bool run = stage_begin(a, sl, by * gx + bx, 2, k0, k1, lane, 64);
    if (lane == 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) { sc[s] = k0.al[s]; sc[4 + s] = k1.al[s]; }
      sc[8] = k0.dt;
      sc[9] = run ? 1.0 : 0.0;
    }
  } else {
    constexpr int NPRO = (ROWS + NW - 2) / (NW - 1);
    double qa[NPRO][4], qb[NPRO][4];
#pragma unroll
    for (int t = 0; t < NPRO; ++t) {
      const int i = w + (NW - 1) * t;
      if (i < ROWS) {
        const size_t row = (size_t)bc_map(y0 - R + i, ny, a.g.bc_y) * nx;
        if (in0) {
#pragma unroll
          for (int c = 0; c < 4; ++c) qa[t][c] = gptr(a.q + c * cs + row)[xa];
        }
        if (in1) {
#pragma unroll
          for (int c = 0; c < 4; ++c) qb[t][c] = gptr(a.q + c * cs + row)[xb];
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NPRO; ++t) {
      const int i = w + (NW - 1) * t;
      if (i < ROWS) {
        if (in0) euler_record2<T>(qa[t], (T)a.ph.gm1, ring + i * RS + lane, FU_RECS);
        if (in1) euler_record2<T>(qb[t], (T)a.ph.gm1, ring + i * RS + 64 + lane, FU_RECS);
      }
    }
  }
  __syncthreads();
  if (scalar_of(sc[9]) == 0.0) return;
  SweepConst kx_, ky_;
#pragma unroll
  for (int s = 0; s < 4; ++s) { kx_.al[s] = scalar_of(sc[s]); ky_.al[s] = scalar_of(sc[4 + s]); }
  kx_.dt = ky_.dt = scalar_of(sc[8]);
  const double kx = scalar_of(-(a.cb * kx_.dt) * a.g.inv_dx), ky = scalar_of(-(a.cb * ky_.dt) * a.g.inv_dy);
  int sb = w;                        // ring slot of row k - R
  int fk = w;                        // flux slot of interface row k
  const int nst = (ylast - y0) / NW + 1;
  for (int st = 0; st < nst; ++st) {
    progress_prio(st, nst);
    const int k = y0 + NW * st + w, r = k - 1;
    // the cell row this wavefront adds for the next step's stencils
    const int rn = k + NW + R - 1;
    const bool need = rn <= ylast + R - 1;
    int slot[2 * R];
#pragma unroll
    for (int j = 0; j < 2 * R; ++j) {
      const int t = sb + j;
      slot[j] = (t >= ROWS ? t - ROWS : t) * RS;
    }
    if (k <= ylast && lane < wc) {
      int off[2 * R];
#pragma unroll
      for (int j = 0; j < 2 * R; ++j) off[j] = slot[j] + lane + R;
      const T al[4] = {(T)ky_.al[0], (T)ky_.al[1], (T)ky_.al[2], (T)ky_.al[3]};
      T F[4];
      euler_flux<T, 4, WV, R, typename Layout2<T>::Y, REREAD>(ring, FU_RECS, off, (T)a.ph.gm1, al, cfg.w, F);
      fb[fk][0][lane] = (double)F[0];
      fb[fk][1][lane] = (double)F[2];
      fb[fk][2][lane] = (double)F[1];
      fb[fk][3][lane] = (double)F[3];
    }
    const bool row_in = r >= y0 && r < ylast;   // wave-uniform
    const bool upd = row_in && lane < wc;
    const size_t ro = (size_t)r * nx + x0;   // wave-uniform
    const unsigned ul = lane;
    // loads for the end of the step
    const int hrow = lane >> 4, rh = k - w + hrow + NW + R - 1;
    // the last halo columns of all the step's new rows: one wavefront in turn
    const bool hal = w == (st & (NW - 1)) && (lane & 15) + 64 < wc + 2 * R && rh <= ylast + R - 1;
    double qn[4], qa[4], qb[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) qn[c] = 0.0;
    auto loads = [&]() {
      if (MODE == MODE_STAGE && upd && a.ca != 0.0) {
#pragma unroll
        for (int c = 0; c < 4; ++c) qn[c] = gptr(a.qn + c * cs + ro)[ul];
      }
      if (need) {
        const size_t row = (size_t)bc_map_span(rn, rn, 1, ny, a.g.bc_y) * nx;
        if (in0) {
#pragma unroll
          for (int c = 0; c < 4; ++c) qa[c] = gptr(a.q + c * cs + row)[xa];
        }
      }
      if (hal) {
        const size_t o = (size_t)bc_map(rh, ny, a.g.bc_y) * nx + xh;
#pragma unroll
        for (int c = 0; c < 4; ++c) qb[c] = gptr(a.q)[c * cs + o];
      }
    };
    if (EARLY) loads();
    double part[4];
    if (row_in) {
      double qc[4];
      if (MODE == MODE_STAGE && upd) {
        if (sizeof(T) != sizeof(double)) {
#pragma unroll
          for (int c = 0; c < 4; ++c) qc[c] = gptr(a.q + c * cs + ro)[ul];
        }
      }
      T F[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) F[c] = T(0);
      if (lane <= wc) {
        int off[2 * R];
#pragma unroll
        for (int j = 0; j < 2 * R; ++j) off[j] = slot[R - 1] + lane + j;
        const T al[4] = {(T)kx_.al[0], (T)kx_.al[1], (T)kx_.al[2], (T)kx_.al[3]};
        euler_flux<T, 4, WV, R, typename Layout2<T>::X, REREAD>(ring, FU_RECS, off, (T)a.ph.gm1, al, cfg.w, F);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double Fl = (double)F[c];
        const double dF = fu_next(Fl) - Fl;
        if (MODE == MODE_RHS) {
          part[c] = -dF * a.g.inv_dx;
        } else {
          if (sizeof(T) == sizeof(double)) qc[c] = (double)ring[slot[R - 1] + c * FU_RECS + lane + R];
          part[c] = fma(kx, dF, a.cb * qc[c]);
        }
      }
    }
    // behind the fluxes: other blocks' wavefronts cover the loads
    if (!EARLY) loads();
    __syncthreads();   // the flux rows are in place, the ring has been read
    if (need) {
      // row rn takes the slot of row k - R
      if (in0) euler_record2<T>(qa, (T)a.ph.gm1, ring + sb * RS + lane, FU_RECS);
    }
    if (hal) {
      int hs = sb - w + hrow;   // the slot of row rh
      hs = hs < 0 ? hs + ROWS : (hs >= ROWS ? hs - ROWS : hs);
      euler_record2<T>(qb, (T)a.ph.gm1, ring + hs * RS + 64 + (lane & 15), FU_RECS);
    }
    if (upd) {
      const int fm = fk == 0 ? NW : fk - 1;
      double qnew[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double dF = fb[fk][c][lane] - fb[fm][c][lane];
        if (MODE == MODE_RHS) {
          gptr(a.out + c * cs + ro)[ul] = part[c] - dF * a.g.inv_dy;
        } else {
          qnew[c] = fma(ky, dF, fma(a.ca, qn[c], part[c]));
          gptr(a.out + c * cs + ro)[ul] = qnew[c];
        }
      }
      if (MODE == MODE_STAGE) cell_speeds<SYS_EULER, 4>(qnew, a.ph, rs);
    }
    __syncthreads();   // the new records are in place, the flux rows have been read
    sb += NW;
    sb = sb >= ROWS ? sb - ROWS : sb;
    fk -= 1;           // NW more, modulo NW + 1
    fk = fk < 0 ? NW : fk;
  }
  if (MODE == MODE_STAGE) block_speeds<SYS_EULER, 2, true>(rs, a.sp_out + ((by * gx + bx) % SP_ROWS) * SP_STRIDE);
}

template <class T, int WV, int R, int MODE, int WAVES>
__global__ __launch_bounds__(64 * FU_NW, WAVES) void k_fused(SweepArgs a, CfgArg<T> cfg) {
  fused_body<T, WV, R, MODE>(a, cfg, blockIdx.x, blockIdx.y, gridDim.x);
}

}  // namespace za
