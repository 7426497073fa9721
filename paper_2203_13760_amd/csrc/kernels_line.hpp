// Steps of a short 1D grid in one workgroup (gfx950).
//
// A grid with only x active and at most kLineCells cells is a few wavefronts of
// work per stage: as launches, a step is six or seven kernels of 3 to 5 us and
// their gaps, none of which the work needs. Here one workgroup holds the grid -
// the primitives with their halo in LDS, a lane's conservative values in
// registers - and runs the steps of a call, with the step size's reduction and
// the boundary images inside; the state is read and written once per launch.
// Bound by the serial chain of a stage (window from LDS, reconstruction, flux,
// update, two barriers). Sod's 200 cells, 50
// CFL steps: 1147 -> 320 us; 990 cells 1245 -> 818 us, so the limit is the
// workgroup's size.
#pragma once
#include "kernels_fwd.hpp"

namespace cfd {

constexpr int kLineNew = 62;   // cells a wavefront updates (its first two lanes only seed the shuffles)
constexpr int kLineWaves = 16;
constexpr int kLineCells = kLineNew * kLineWaves;
constexpr int kLineHalo = 3;   // halo cells held in LDS, whatever the state's halo width

template <int SCH, int PHYS>
__global__ void __launch_bounds__(64 * kLineWaves) k_line(double* __restrict__ U, Geom g, DevCtl* ctl, int steps,
                                                          double fixed_dt, double t_end, double* tp, double* dt_out) {
  __shared__ double P[5][kLineCells + 2 * kLineHalo];
  __shared__ double red[kLineWaves];
  const int lane = threadIdx.x & 63, wave = wave_in_block(), waves = (int)blockDim.x >> 6;
  const int n = g.n[0];
  const int f = wave * kLineNew - 1 + lane;    // the lane's face, between cells f-1 and f
  const int fl = min(f, n);                    // its reconstructed cell (window fl-2 .. fl+2)
  const int cell = f - 1;                      // the cell it updates
  const bool own = lane >= 2 && cell < n;
  const bool face = lane >= 1 && f <= n;
  double* Uc = U + g.h[0] + (own ? cell : 0);
  double u[5], un[5], w[6];
  double smax = 0.0;
  int bad = 0;
  auto publish = [&](bool rate) {  // primitives of u, with their halo images, into LDS
    const double ir = cons_to_prim(g, u, w);
    if (own) {
      bad |= health_bits(u, w[4]);
      if (rate) smax = cfl_rate(g, w, ir);
#pragma unroll
      for (int v = 0; v < 5; ++v) P[v][cell + kLineHalo] = w[v];
      const AxisImages X(cell, n, kLineHalo, g.bc[0], g.bc[1]);
      for (int m = 1; m < X.count(); ++m) {
        const int x = X.at(cell, m);
        const double sg = bc_sign(x, n, g.bc[0], g.bc[1]);
#pragma unroll
        for (int v = 0; v < 5; ++v) P[v][x + kLineHalo] = v == 1 ? sg * w[v] : w[v];
      }
    }
    __syncthreads();
  };
#pragma unroll
  for (int v = 0; v < 5; ++v) u[v] = Uc[v * g.vs];
  const bool cfl = !(fixed_dt > 0.0);
  double t = tp ? *tp : 0.0, dt = fixed_dt;
  publish(cfl);
  for (int s = 0; s < steps; ++s) {
    if (cfl) {
      const double m = wave_max(smax);
      if (lane == 0) red[wave] = m;
      __syncthreads();
      double r = 0.0;
      for (int i = 0; i < waves; ++i) r = fmax(r, red[i]);
      dt = step_size(g.cfl, r, 0.0, tp ? &t : nullptr, t_end);
      if (dt == 0.0) break;  // t_end reached
    }
    if (tp) t = t + dt;
#pragma unroll
    for (int v = 0; v < 5; ++v) un[v] = u[v];
    const int stages = g.rk2 ? 2 : 3;
    for (int k = 0; k < stages; ++k) {
      const double a = k == 0 ? 0.0 : (g.rk2 ? 0.5 : (k == 1 ? 0.75 : 1.0 / 3.0));
      const double b = k == 0 ? 1.0 : (g.rk2 ? 0.5 : (k == 1 ? 0.25 : 2.0 / 3.0));
      double q[5][5];
#pragma unroll
      for (int m = 0; m < 5; ++m)
#pragma unroll
        for (int v = 0; v < 5; ++v) q[m][v] = P[v][fl - 2 + m + kLineHalo];
      __syncthreads();  // every window is read before the next primitives are written
      double T[4] = {0.0, 0.0, 0.0, 0.0};
      if (with_heat<PHYS>(g)) {
#pragma unroll
        for (int m = 0; m < 4; ++m) T[m] = div_nr(q[m][4], q[m][0]);
      }
      double WL[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, WR[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      if (with_inviscid<PHYS>(g)) {
        double qr[5];
        recon_pair<SCH>(q, qr, WR);
#pragma unroll
        for (int v = 0; v < 5; ++v) WL[v] = lane_shr1(qr[v]);
        check_face_states(g, face, WL, WR, q[1], q[2], bad);
      }
      const double tf[3] = {0.0, 0.0, 0.0};  // no tangential axis is active
      double G[5];
      face_flux_states<0, SCH, PHYS>(g, WL, WR, q, T, tf, 0.0, G);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const double D = (G[v] - lane_shr1(G[v])) * g.idx[0];
        u[v] = a * un[v] + b * (u[v] + dt * -D);
      }
      publish(cfl && k == stages - 1);
    }
  }
  if (own) {
#pragma unroll
    for (int v = 0; v < 5; ++v) Uc[v * g.vs] = u[v];
  }
  if (bad) atomicOr(&ctl->status, bad);
  if (threadIdx.x == 0) {
    if (tp) *tp = t;
    if (dt_out) *dt_out = dt;
  }
}

}  // namespace cfd
