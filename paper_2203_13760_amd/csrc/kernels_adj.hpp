// Discrete adjoint of the right-hand side (gfx950).
//
//   1. the primitives P at the state (the forward kernels, or the buffers a
//      forward recompute of the stages leaves);
//   2. the face reverses: the face flux adjoint follows from Rbar
//      (R_i = -(G_{i+1/2} - G_{i-1/2})/dx gives Gbar_{i+1/2} =
//      (Rbar_{i+1} - Rbar_i)/dx); each face recomputes its forward flux and
//      reverses it (physics_adj.hpp), and its contributions go to Wbar
//      (rho,u,v,w,p,T~ of the stencil cells) and Dbar (the adjoints of the
//      centred derivatives) with hardware FP64 atomics. x faces
//      (k_xadj_inv/dis): one lane per cell or face of a row, inputs passed
//      between lanes and contributions summed per cell by wavefront shifts
//      (one atomic per cell and variable). y and z faces
//      (k_march_adj_inv/dis): marching wavefronts, the reverse of the forward
//      marches. On grids of 2^18 padded cells and more they are a launch each,
//      the inviscid and the dissipative ones on two streams; below, all of
//      them are one launch (k_faces_adj);
//   3. k_adj_halo: the transposed halo fill, every halo cell's Wbar (viscous:
//      with its transposed centred differences of Dbar; k_adj_fold adds the
//      interior cells' share) added to its interior source cell;
//   4. k_adj_fold: per interior cell, the transposed primitive map at the
//      state (from its primitives) gives Ubar.
// The atomics make the summation order, and so the last bits, vary between
// runs; everything else is deterministic.
#pragma once
#include "kernels_fwd.hpp"
#include "physics_adj.hpp"

namespace cfd {

__device__ __forceinline__ void atomic_add(double* p, double v) {
  if (v != 0.0) unsafeAtomicAdd(p, v);
}
__device__ __forceinline__ void atomic_add_at(double* base, unsigned off, double v) {
  atomic_add(reinterpret_cast<double*>(reinterpret_cast<char*>(base) + off), v);
}

// Face numbering for axis D: face f in [0, n_D] lies between cells f-1 and f.
// D = 0: f runs fastest, so the lanes of a wavefront hold consecutive faces of
// a row (col = the row) and also load consecutive cells; D = 1, 2: x runs
// fastest so that lanes load consecutive cells (col = -1: no two lanes of a
// wavefront share a column).
template <int D>
__device__ __forceinline__ bool face_coords(const Geom& g, int t, int& i, int& j, int& k, int& f, int& col) {
  if (D == 0) {
    const int F = g.n[0] + 1;
    col = t / F;
    f = t - col * F;
    k = col / g.n[1];
    j = col - k * g.n[1];
    i = f;
    return k < g.n[2];
  } else if (D == 1) {
    const int F = g.n[1] + 1;
    const int r = t / g.n[0];
    i = t - r * g.n[0];
    k = r / F;
    f = r - k * F;
    j = f;
    col = -1;
    return k < g.n[2];
  } else {
    const int r = t / g.n[0];
    i = t - r * g.n[0];
    f = r / g.n[1];
    j = r - f * g.n[1];
    k = f;
    col = -1;
    return f <= g.n[2];
  }
}

// Face adjoint Gbar from Rbar (read as rscale * Rbar, interior cells only).
template <int D>
__device__ __forceinline__ bool face_gbar(const Geom& g, const double* __restrict__ Rbar, double rscale, long long cf,
                                          int f, double* Gb) {
  const long long st = g.s[D];
  const bool hasL = f >= 1, hasR = f < g.n[D];
  double any = 0.0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double rl = hasL ? Rbar[v * g.vs + cf - st] : 0.0;
    const double rr = hasR ? Rbar[v * g.vs + cf] : 0.0;
    Gb[v] = rscale * (rr - rl) * g.idx[D];
    any += fabs(Gb[v]);
  }
  return any != 0.0;
}

// Reverse of the dissipative flux of one face (sub_dissipative_q), from the
// velocities u[0..3] and tangential sums t[0..3] of the four cells around it
// and Gbar, the adjoint of G = F - F^d: what the cells' adjoints are formed
// from - cell m takes cdn[m] d[v] + crc[m] f[v] for its velocities (in the order
// u_D, u_T1, u_T2), cdn[m] T for T~ and crc[m] t[k] for its tangential sums. The
// heat flux is linear in T~, so no T~ values are needed.
struct DisRev {
  double d[3], f[3], t[3], T;
};

template <int D, int PHYS>
__device__ __forceinline__ void dissipative_rev(const Geom& g, const double (*u)[3], const double (*t)[3],
                                                const double* Gb, DisRev& r) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const double i24 = g.idx[D] * (1.0 / 24.0);
  const double Eb = -Gb[4];
  if (with_viscous<PHYS>(g)) {
    auto dn = [&](int v) { return fma(27.0, u[2][v] - u[1][v], u[0][v] - u[3][v]) * i24; };
    auto rc = [&](int v) { return rc4(u[0][v], u[1][v], u[2][v], u[3][v]); };
    auto rt = [&](int k) { return rc4(t[0][k], t[1][k], t[2][k], t[3][k]); };
    const double tDD = g.mu * fma(4.0 / 3.0, dn(D), (-2.0 / 3.0) * rt(2));
    const double tD1 = g.mu * (rt(0) + dn(T1)), tD2 = g.mu * (rt(1) + dn(T2));
    const double bDD = g.mu * fma(Eb, rc(D), -Gb[1 + D]);
    const double bD1 = g.mu * fma(Eb, rc(T1), -Gb[1 + T1]), bD2 = g.mu * fma(Eb, rc(T2), -Gb[1 + T2]);
    r.d[0] = (4.0 / 3.0 * i24) * bDD;
    r.d[1] = i24 * bD1;
    r.d[2] = i24 * bD2;
    r.f[0] = (1.0 / 16.0) * (Eb * tDD);
    r.f[1] = (1.0 / 16.0) * (Eb * tD1);
    r.f[2] = (1.0 / 16.0) * (Eb * tD2);
    r.t[0] = (1.0 / 16.0) * bD1;
    r.t[1] = (1.0 / 16.0) * bD2;
    r.t[2] = (-2.0 / 48.0) * bDD;
  }
  r.T = g.kappa * i24 * Eb;
}
// cdn and crc without the factors dissipative_rev has applied.
constexpr double kCdn[4] = {1.0, -27.0, 27.0, -1.0}, kCrc[4] = {-1.0, 9.0, 9.0, -1.0};

// Component of Dbar a tangential sum's adjoint goes to: the mixed derivatives
// u_D along T1 and T2 in their own, and the sum of the two derivatives along
// their own axes in component (D, D), which fold_dbar hands to both.
template <int D>
__device__ __forceinline__ int dbar_comp(int k) {
  return D * 3 + (k == 0 ? (D + 1) % 3 : (k == 1 ? (D + 2) % 3 : D));
}

// ---------------------------------------------------------------------------
// x faces: one lane per slot of a row, as in the forward x sweep; the
// neighbouring cells of a row are neighbouring lanes, so a cell's inputs are
// loaded once and passed to the faces that use them, and the contributions to
// a cell are summed across lanes into the lane that owns it (DPP wavefront
// shifts, no LDS), which adds the sum to memory with one atomic per variable.
// Rows are taken in the band-major order of the forward x sweep.

// Inviscid part: the slots of a row are its cells -3 .. n+2 (every cell a
// reconstruction reaches). The lane of cell x forms the reconstruction pair
// of x (cells x-1 .. n have one, §3.3), reverses the HLLC flux of face x
// (between x-1 and x; its left state is the pair of x-1, one lane below), and
// then reverses the pair of x with the cotangents of its faces x (own) and
// x+1 (one lane above), into cells x-2 .. x+2 (lanes -2 .. +2). A wavefront
// takes 64 consecutive slots of which the middle kXInvNew reverse their
// pairs; kXInvCtx slots at each end overlap the neighbouring wavefronts and
// only supply values and collect sums. A lane loads its own cell only and the
// windows are formed by lane shifts, twice, which beats 50 loads of cached
// lines a lane: 128^3 296 us against 313 beside the dissipative reverses, the
// step and its reverse 3.47 -> 3.45 ms, the 40^3 rollout 8.09 -> 8.05 ms.
constexpr int kXInvCtx = 3;
constexpr int kXInvNew = 64 - 2 * kXInvCtx;

__device__ __forceinline__ void xadj_inv_body(const double* P, const double* __restrict__ Rbar, double rscale,
                                              double* Wbar, const Geom& g, int block) {
  const int lane = threadIdx.x & 63;
  const int wave = (block * kBlock + (int)threadIdx.x) >> 6;
  const int n = g.n[0];
  const int S = n + 6;
  const int total = S * g.n[1] * g.n[2];
  const int first = wave * kXInvNew;
  if (first >= total) return;  // uniform per wavefront
  const int gs = first - kXInvCtx + lane;
  const bool inrange = gs >= 0 && gs < total;
  int x = 0, j = 0, k = 0;
  if (inrange) {
    const int row = gs / S;
    x = gs - row * S - 3;
    x_row(g, row, j, k);
  }
  const bool pair = inrange && x >= -1 && x <= n;     // cell x has a reconstruction pair
  // face x, with the windows of cells x-1 and x in the wavefront
  const bool face = inrange && x >= 0 && x <= n && lane >= kXInvCtx && lane < 64 - 2;
  const bool rev = pair && lane >= kXInvCtx && lane < 64 - kXInvCtx;
  const long long cx = cell_at(g, x, j, k);
  // the cell's values; the other cells of its window come from the lanes beside
  double own[5];
  load_prims(P, g.vs, cx, own);
  auto window = [&](int v, double* q) {  // cells x-2 .. x+2
    q[2] = own[v];
    q[1] = lane_shr1(q[2]);
    q[0] = lane_shr1(q[1]);
    q[3] = lane_shl1(q[2]);
    q[4] = lane_shl1(q[3]);
  };
  const double gsc = rscale * g.idx[0];
  double WLb[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, WRb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  {
    double q[5][5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double s[5];
      window(v, s);
#pragma unroll
      for (int m = 0; m < 5; ++m) q[m][v] = s[m];
    }
    double qr[5], ql[5];
    recon_pair<SCH_JS>(q, qr, ql);  // right face of x (left state of face x+1), left face of x
    double WL[5], Gb[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const double r = inrange && x >= 0 && x < n ? Rbar[v * g.vs + cx] : 0.0;
      Gb[v] = gsc * (r - lane_shr1(r));  // (Rbar_x - Rbar_{x-1}) / dx
      WL[v] = lane_shr1(qr[v]);
    }
    if (face) hllc_rev<0>(g.gamma, g.gm1i, WL, ql, Gb, WLb, WRb);
  }
  // the windows are formed again below instead of being kept
#pragma unroll
  for (int v = 0; v < 5; ++v) pin(own[v]);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const double up = lane_shl1(WLb[v]);  // every lane takes part in the shift
    const double qrb = rev ? up : 0.0;    // face x+1: cotangent of the right-face value of x
    const double qlb = rev ? WRb[v] : 0.0;
    double gq[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    double q[5];
    window(v, q);
    // only whole windows of one row are reversed: the others (wavefront ends
    // with shifted-in zeros, row ends) can overflow in the normalisers, and a
    // zero cotangent times infinity is NaN
    if (rev) weno5_pair_rev(q[0], q[1], q[2], q[3], q[4], qrb, qlb, gq);
    pin(gq[0]);
    pin(gq[4]);
    // cell x receives gq[4] from lane - 2, gq[3] from lane - 1, gq[2] from
    // itself, gq[1] from lane + 1 and gq[0] from lane + 2
    const double lo = lane_shr1(lane_shr1(gq[4]) + gq[3]);
    const double hi = lane_shl1(lane_shl1(gq[0]) + gq[1]);
    if (inrange) atomic_add(Wbar + v * g.vs + cx, lo + gq[2] + hi);
  }
}

// Four wavefronts per SIMD: bound by the latency of its loads and atomics, and
// worth the 44 B of scratch a lane that 128 registers leave.
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4)))
k_xadj_inv(const double* P, const double* __restrict__ Rbar, double rscale, double* Wbar, Geom g) {
  xadj_inv_body(P, Rbar, rscale, Wbar, g, xcd_major_block(blockIdx.x, gridDim.x));
}

// Dissipative part: slot s of a row is face f = s - 3 (f = -3 .. n), and its
// lane loads the inputs of cell f+1 (u, v, w and the four tangential
// derivatives). Face f takes those of cells f-2 .. f+1 from itself and the
// three lanes below, and its contributions to those cells flow back down to
// them. A wavefront takes 64 consecutive slots; the first three overlap its
// predecessor and only supply inputs and collect sums. The heat flux is
// linear in T~, so its reverse needs no T~ values.
constexpr int kXDisCtx = 3;
constexpr int kXDisNew = 64 - kXDisCtx;

template <int PHYS>
__device__ __forceinline__ void xadj_dis_body(const double* __restrict__ P, const double* __restrict__ Rbar,
                                              double rscale, double* Wbar, double* Dbar, const Geom& g, int block) {
  const int lane = threadIdx.x & 63;
  const int wave = (block * kBlock + (int)threadIdx.x) >> 6;
  const int n = g.n[0];
  const int S = n + 1 + kXDisCtx;
  const int total = S * g.n[1] * g.n[2];
  const int first = wave * kXDisNew;
  if (first >= total) return;  // uniform per wavefront
  const int gs = first - kXDisCtx + lane;
  const bool inrange = gs >= 0 && gs < total;
  int f = 0, j = 0, k = 0;
  if (inrange) {
    const int row = gs / S;
    f = gs - row * S - kXDisCtx;
    x_row(g, row, j, k);
  }
  const bool face = inrange && f >= 0 && lane >= kXDisCtx;
  const long long co = cell_at(g, inrange ? f + 1 : 0, j, k);  // the lane's cell f+1
  // inputs of cell f+1, then of cells f, f-1, f-2 from the lanes below
  double u[4][3], d[4][3], r[3][5];
  const bool vis = with_viscous<PHYS>(g), heat = with_heat<PHYS>(g);
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    u[3][v] = vis ? P[(1 + v) * g.vs + co] : 0.0;
    d[3][v] = 0.0;
  }
  if (vis) {
    double x[4][4];
    tangential_load<0>(g, P, co, x);
    __builtin_amdgcn_sched_barrier(0);
    tangential_combine3<0>(g, x, d[3]);
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) r[0][v] = inrange && f + 1 >= 0 && f + 1 < n ? Rbar[v * g.vs + co] : 0.0;
#pragma unroll
  for (int m = 2; m >= 0; --m) {
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      u[m][v] = lane_shr1(u[m + 1][v]);
      d[m][v] = lane_shr1(d[m + 1][v]);
    }
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    r[1][v] = lane_shr1(r[0][v]);  // cell f
    r[2][v] = lane_shr1(r[1][v]);  // cell f-1
  }
  const double gsc = face ? rscale * g.idx[0] : 0.0;  // lanes without a face contribute zeros
  double Gb[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) Gb[v] = face ? gsc * (r[1][v] - r[2][v]) : 0.0;
  DisRev R;
  dissipative_rev<0, PHYS>(g, u, d, Gb, R);
  if (!face) {
#pragma unroll
    for (int v = 0; v < 3; ++v) R.d[v] = R.f[v] = R.t[v] = 0.0;
    R.T = 0.0;
  }
  // cell f+1 collects its share from faces f, f+1, f+2, f+3 (this lane and
  // the three above), up to the end of its row
  const bool above = inrange && f < n;
  auto gather = [&](double wd, const double* cd, double wf, const double* cf) {
    double a = fma(wd, cd[0], wf * cf[0]);
#pragma unroll
    for (int m = 1; m < 4; ++m) {
      const double b = lane_shl1(a);  // every lane takes part in the shift
      a = fma(wd, cd[m], fma(wf, cf[m], above ? b : 0.0));
    }
    return a;
  };
  if (vis) {
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      const double a = gather(R.d[v], kCdn, R.f[v], kCrc);
      if (inrange) atomic_add(Wbar + (1 + v) * g.vs + co, a);
    }
  }
  if (heat) {
    const double a = gather(R.T, kCdn, 0.0, kCrc);
    if (inrange) atomic_add(Wbar + 5 * g.vs + co, a);
  }
  if (vis) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (k < 2 && !g.act[1 + k]) continue;
      const double a = gather(0.0, kCdn, R.t[k], kCrc);
      if (inrange) atomic_add(Dbar + dbar_comp<0>(k) * g.vs + co, a);
    }
  }
}

template <int PHYS>
__global__ void __launch_bounds__(kBlock) k_xadj_dis(const double* __restrict__ P, const double* __restrict__ Rbar,
                                                     double rscale, double* Wbar, double* Dbar, Geom g) {
  xadj_dis_body<PHYS>(P, Rbar, rscale, Wbar, Dbar, g, xcd_major_block(blockIdx.x, gridDim.x));
}

// ---------------------------------------------------------------------------
// Marching face reverses along y and z (AX = 1, 2), the reverse counterparts
// of the forward marches: a wavefront holds 64 consecutive x of one column
// (other transverse coordinate, segment of `seg` cells along AX, chosen for
// each part on its own) and walks
// its faces in order, keeping the stencil window in registers, so every cell
// of the column is loaded once per segment instead of once per face that
// touches it, and a cell's adjoint is added to memory once, when the last
// face of the segment that touches it is done (one atomic per cell and
// variable; a cell near a segment end gets a share from each of the two
// segments). One-dimensional launch: blocks of 64 x along a row first, then
// four columns a block.

// Column, segment and first/last face of the marching wavefront, all uniform;
// false for a wavefront without a column. The lane's x is i (at or past the
// row's end in lanes without a cell). The segment of cells [s0, s1) owns faces
// s0 .. s1-1, and the last segment also face n (the upper boundary).
template <int AX>
__device__ __forceinline__ bool march_adj_column(const Geom& g, int block, int sl, int& i, int& o, int& s0, int& fe) {
  constexpr int OT = AX == 1 ? 2 : 1;
  const int gx = (g.n[0] + 63) / 64;
  const int by = block / gx, bx = block - by * gx;
  i = bx * 64 + (int)(threadIdx.x & 63);
  const int nseg = (g.n[AX] + sl - 1) / sl;
  const int col = uniform(by * (kBlock >> 6) + wave_in_block());
  if (col >= g.n[OT] * nseg) return false;
  o = uniform(col / nseg);
  s0 = (col - o * nseg) * sl;
  const int s1 = min(s0 + sl, g.n[AX]);
  fe = s1 == g.n[AX] ? s1 : s1 - 1;
  return true;
}

template <int AX>
__device__ __forceinline__ long long march_adj_cell(const Geom& g, int i, int o, int a) {
  return AX == 1 ? cell_at(g, i, a, o) : cell_at(g, i, o, a);
}

// Inviscid part. Face f (between cells f-1 and f) takes its left state from
// the reconstruction pair of cell f-1 and its right state from that of cell
// f (§3.3): the wavefront computes the pair of cell f at face f, reverses the
// HLLC flux of face f, and then reverses the pair of cell f-1, whose two
// cotangents (from faces f-1 and f) are both known, into cells f-3 .. f+1.
// A pair shared with the neighbouring segment is reversed in both, each with
// its own face's share of the cotangent (the reverse is linear in it).
// The window holds cells f-3 .. f+2 in registers, and the per-cell sums of
// the five cells a pair reverse touches live in a lane-private LDS ring. With
// scalar bases and the variables reversed one after another (pin) it fits two
// wavefronts per SIMD; before, at 384 registers, it ran one.
constexpr int kMarchRing = 5;

template <int AX>
__device__ __forceinline__ void march_adj_inv_body(const double* __restrict__ P, const double* __restrict__ Rbar,
                                                   double rscale, double* Wbar, const Geom& g, int seg, int block,
                                                   double* ring) {
  int i, o, s0, fe;
  if (!march_adj_column<AX>(g, block, seg, i, o, s0, fe)) return;
  const int tid = threadIdx.x;
#pragma unroll
  for (int e = 0; e < kMarchRing * 5; ++e) ring[e * kBlock + tid] = 0.0;
  const long long st = g.s[AX], vs = g.vs;
  const int n = g.n[AX];
  const double gs_scale = rscale * g.idx[AX];
  const long long c1 = march_adj_cell<AX>(g, 0, o, s0 - 3);  // window cell 0: cell f-3 of face f = s0, at x = 0
  const unsigned off = (unsigned)min(i, g.n[0] - 1) * 8u;
  const bool in = i < g.n[0];
  double w[6][5];
#pragma unroll
  for (int m = 0; m < 6; ++m)
#pragma unroll
    for (int v = 0; v < 5; ++v) w[m][v] = ld_at(P + v * vs + c1 + m * st, off);
  double WLc[5], WRbc[5], rl[5];
  {
    double unused[5];
    recon_pair<SCH_JS>(w, WLc, unused);  // cell s0-1: left state of face s0
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    WRbc[v] = 0.0;  // face s0-1 belongs to the previous segment
    rl[v] = s0 >= 1 ? ld_at(Rbar + v * vs + c1 + 2 * st, off) : 0.0;
  }
  int r0 = 0;  // ring slot of window cell 0
  for (int f = s0; f <= fe; ++f) {
    const long long c = c1 + uniform(f - s0) * st;
    // the entering cell (after the last face one already held)
    const long long ce = f < fe ? c + 6 * st : c + 5 * st;
    double nq[5], rr[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) nq[v] = ld_at(P + v * vs + ce, off);
#pragma unroll
    for (int v = 0; v < 5; ++v) rr[v] = f < n ? ld_at(Rbar + v * vs + c + 3 * st, off) : 0.0;
    // pair of cell f (window cells 1..5): left state of face f+1, right state of face f
    double nWL[5], WR[5];
    recon_pair<SCH_JS>(w + 1, nWL, WR);
    double Gb[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Gb[v] = gs_scale * (rr[v] - rl[v]);
    double WLb[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, WRb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    hllc_rev<AX>(g.gamma, g.gm1i, WLc, WR, Gb, WLb, WRb);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      pin(WLb[v]);
      pin(WRb[v]);
    }
    // pair of cell f-1 (window cells 0..4) with the cotangents of faces f and
    // f-1; cell f-3 is complete for this segment
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      double gq[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      pin(w[2][v]);
      weno5_pair_rev(w[0][v], w[1][v], w[2][v], w[3][v], w[4][v], WLb[v], WRbc[v], gq);
#pragma unroll
      for (int m = 0; m < 5; ++m) {
        const int slot = r0 + m < kMarchRing ? r0 + m : r0 + m - kMarchRing;
        double& a = ring[(slot * 5 + v) * kBlock + tid];
        if (m == 0) {
          if (in) atomic_add_at(Wbar + v * vs + c, off, a + gq[0]);
          a = 0.0;
        } else {
          a += gq[m];
        }
      }
    }
    r0 = r0 + 1 < kMarchRing ? r0 + 1 : 0;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
#pragma unroll
      for (int m = 0; m < 5; ++m) w[m][v] = w[m + 1][v];
      w[5][v] = nq[v];
      WLc[v] = nWL[v];
      WRbc[v] = WRb[v];
      rl[v] = rr[v];
    }
  }
  if (!in) return;
  // the pair of cell fe (window cells 0..4) with the cotangent of face fe only
  const long long c = c1 + (long long)(fe + 1 - s0) * st;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    double gq[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    weno5_pair_rev(w[0][v], w[1][v], w[2][v], w[3][v], w[4][v], 0.0, WRbc[v], gq);
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      const int slot = r0 + m < kMarchRing ? r0 + m : r0 + m - kMarchRing;
      atomic_add_at(Wbar + v * vs + c + m * st, off, ring[(slot * 5 + v) * kBlock + tid] + gq[m]);
    }
  }
}

template <int AX>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_march_adj_inv(const double* __restrict__ P, const double* __restrict__ Rbar, double rscale, double* Wbar, Geom g,
                int seg) {
  __shared__ double ring[kMarchRing * 5 * kBlock];
  march_adj_inv_body<AX>(P, Rbar, rscale, Wbar, g, seg, xcd_major_block(blockIdx.x, gridDim.x), ring);
}

// Dissipative part (viscous and heat flux). Face f reads window cells
// f-2 .. f+1 (u, v, w and the tangential sums of each, formed from P as in the
// forward marches); the adjoints of those inputs (Wbar u, v, w, T~ and Dbar)
// are summed in registers and cell f-2 is added to memory after face f.
template <int AX, int PHYS>
__device__ __forceinline__ void march_adj_dis_body(const double* __restrict__ P, const double* __restrict__ Rbar,
                                                   double rscale, double* Wbar, double* Dbar, const Geom& g, int seg,
                                                   int block) {
  constexpr int T1 = (AX + 1) % 3, T2 = (AX + 2) % 3;
  int i, o, s0, fe;
  if (!march_adj_column<AX>(g, block, seg, i, o, s0, fe)) return;
  const long long st = g.s[AX], vs = g.vs;
  const int n = g.n[AX];
  const double gs_scale = rscale * g.idx[AX];
  const long long c1 = march_adj_cell<AX>(g, 0, o, s0 - 2);  // window cell 0: cell f-2 of face f = s0, at x = 0
  const unsigned off = (unsigned)min(i, g.n[0] - 1) * 8u;
  const bool in = i < g.n[0];
  const bool vis = with_viscous<PHYS>(g), heat = with_heat<PHYS>(g);
  const long long sT1 = g.act[T1] ? g.s[T1] : 0, sT2 = g.act[T2] ? g.s[T2] : 0;
  const double w1 = g.act[T1] ? g.idx[T1] * (1.0 / 12.0) : 0.0, w2 = g.act[T2] ? g.idx[T2] * (1.0 / 12.0) : 0.0;
  double u[4][3], tg[4][3];  // cells f-2 .. f+1
  Diff4 d[4];
  auto tang_load = [&](long long cc) {
    d[0].load(P + (1 + AX) * vs + cc, sT1, off);
    d[1].load(P + (1 + T1) * vs + cc, sT1, off);
    d[2].load(P + (1 + AX) * vs + cc, sT2, off);
    d[3].load(P + (1 + T2) * vs + cc, sT2, off);
  };
  auto tang_sum = [&](double* t) {
    t[0] = d[0].diff() * w1;
    t[1] = d[2].diff() * w2;
    t[2] = fma(d[1].diff(), w1, d[3].diff() * w2);
  };
#pragma unroll
  for (int m = 0; m < 4; ++m) {
#pragma unroll
    for (int v = 0; v < 3; ++v) u[m][v] = vis ? ld_at(P + (1 + v) * vs + c1 + m * st, off) : 0.0;
    tg[m][0] = tg[m][1] = tg[m][2] = 0.0;
    if (vis) {
      tang_load(c1 + m * st);
      tang_sum(tg[m]);
    }
  }
  double ub[4][4], tb[4][3];  // adjoints of cells f-2 .. f+1: u_D, u_T1, u_T2, T~; the tangential sums
#pragma unroll
  for (int m = 0; m < 4; ++m) {
#pragma unroll
    for (int v = 0; v < 4; ++v) ub[m][v] = 0.0;
    tb[m][0] = tb[m][1] = tb[m][2] = 0.0;
  }
  double rl[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) rl[v] = s0 >= 1 ? ld_at(Rbar + v * vs + c1 + st, off) : 0.0;
  const int slot[4] = {1 + AX, 1 + T1, 1 + T2, 5};
  auto put = [&](long long cc, const double* b, const double* t) {
    if (!in) return;
#pragma unroll
    for (int v = 0; v < 4; ++v)
      if (v == 3 ? heat : vis) atomic_add_at(Wbar + slot[v] * vs + cc, off, b[v]);
    if (vis) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k == 2 || g.act[k == 0 ? T1 : T2]) atomic_add_at(Dbar + dbar_comp<AX>(k) * vs + cc, off, t[k]);
    }
  };
  for (int f = s0; f <= fe; ++f) {
    const long long c = c1 + uniform(f - s0) * st;
    const long long ce = f < fe ? c + 4 * st : c + 3 * st;  // the entering cell (after the last face one already held)
    double nq[3], rr[5];
    if (vis) {
#pragma unroll
      for (int v = 0; v < 3; ++v) nq[v] = ld_at(P + (1 + v) * vs + ce, off);
      tang_load(ce);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) rr[v] = f < n ? ld_at(Rbar + v * vs + c + 2 * st, off) : 0.0;
    __builtin_amdgcn_sched_barrier(0);
    double Gb[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Gb[v] = gs_scale * (rr[v] - rl[v]);
    DisRev r;
    dissipative_rev<AX, PHYS>(g, u, tg, Gb, r);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if (vis) {
#pragma unroll
        for (int v = 0; v < 3; ++v) {
          ub[m][v] = fma(kCdn[m], r.d[v], fma(kCrc[m], r.f[v], ub[m][v]));
          tb[m][v] = fma(kCrc[m], r.t[v], tb[m][v]);
        }
      }
      if (heat) ub[m][3] = fma(kCdn[m], r.T, ub[m][3]);
    }
    put(c, ub[0], tb[0]);  // cell f-2 is complete for this segment
#pragma unroll
    for (int m = 0; m < 3; ++m) {
#pragma unroll
      for (int v = 0; v < 4; ++v) ub[m][v] = ub[m + 1][v];
#pragma unroll
      for (int v = 0; v < 3; ++v) {
        tb[m][v] = tb[m + 1][v];
        tg[m][v] = tg[m + 1][v];
        u[m][v] = u[m + 1][v];
      }
    }
    ub[3][3] = 0.0;
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      ub[3][v] = tb[3][v] = 0.0;
      if (vis) u[3][v] = nq[v];
    }
    if (vis) tang_sum(tg[3]);
#pragma unroll
    for (int v = 0; v < 5; ++v) rl[v] = rr[v];
  }
  // cells fe-1 .. fe+1 (window cells 0..2) hold the rest of this segment's sums
  const long long c = c1 + (long long)(fe + 1 - s0) * st;
#pragma unroll
  for (int m = 0; m < 3; ++m) put(c + m * st, ub[m], tb[m]);
}

template <int AX, int PHYS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_march_adj_dis(const double* __restrict__ P, const double* __restrict__ Rbar, double rscale, double* Wbar,
                double* Dbar, Geom g, int seg) {
  march_adj_dis_body<AX, PHYS>(P, Rbar, rscale, Wbar, Dbar, g, seg, xcd_major_block(blockIdx.x, gridDim.x));
}

// All face reverses in one launch, for grids whose reverses take some
// microseconds each: block ranges in the order y and z inviscid, y and z
// dissipative, x inviscid, x dissipative (the longest chains first). One after
// another they would each leave most of the chip idle.
struct AdjBlocks {
  int end[6];  // cumulative
  int seg_inv[3], seg_dis[3];
};

template <int PHYS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_faces_adj(const double* __restrict__ P, const double* __restrict__ Rbar, double rscale, double* Wbar, double* Dbar,
            Geom g, AdjBlocks ab) {
  __shared__ double ring[kMarchRing * 5 * kBlock];
  const int b = blockIdx.x;
  if (b < ab.end[0]) return march_adj_inv_body<1>(P, Rbar, rscale, Wbar, g, ab.seg_inv[1], b, ring);
  if (b < ab.end[1]) return march_adj_inv_body<2>(P, Rbar, rscale, Wbar, g, ab.seg_inv[2], b - ab.end[0], ring);
  if constexpr (PHYS != PHYS_EULER) {
    if (b < ab.end[2])
      return march_adj_dis_body<1, PHYS>(P, Rbar, rscale, Wbar, Dbar, g, ab.seg_dis[1], b - ab.end[1]);
    if (b < ab.end[3])
      return march_adj_dis_body<2, PHYS>(P, Rbar, rscale, Wbar, Dbar, g, ab.seg_dis[2], b - ab.end[2]);
  }
  if (b < ab.end[4]) return xadj_inv_body(P, Rbar, rscale, Wbar, g, b - ab.end[3]);
  if constexpr (PHYS != PHYS_EULER)
    xadj_dis_body<PHYS>(P, Rbar, rscale, Wbar, Dbar, g, b - ab.end[4]);
}

// Transposed centred differences of Dbar at padded cell cc (coordinates q),
// added to wb[1..3]: phi_bar(m) += (Dbar(m+2) - 8 Dbar(m+1) + 8 Dbar(m-1) -
// Dbar(m-2)) / (12 dx_t), where the adjoint of du_t/dx_t is the sum of the
// (D, D) components of the other two face directions. CHECK selects the range
// checks a halo image needs; an interior cell's +-2 neighbours always lie
// inside the padded block.
template <bool CHECK>
__device__ __forceinline__ void fold_dbar(const Geom& g, const double* __restrict__ Dbar, long long cc,
                                          const int* q, double* wb) {
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    if (!g.act[t]) continue;
    const long long st = g.s[t];
    const int lo = -g.h[t], hi = g.n[t] + g.h[t];
    const int y = q[t];
    const double i12 = g.idx[t] * (1.0 / 12.0);
    // out of the padded block (CHECK): the cell's own entry with weight 0, so
    // that all loads go out together
    const bool h2 = !CHECK || y + 2 < hi, h1 = !CHECK || y + 1 < hi, l1 = !CHECK || y - 1 >= lo, l2 = !CHECK || y - 2 >= lo;
    const long long oh2 = h2 ? 2 * st : 0, oh1 = h1 ? st : 0, ol1 = l1 ? st : 0, ol2 = l2 ? 2 * st : 0;
    auto diff = [&](int comp) {
      const double* Db = Dbar + comp * g.vs + cc;
      const double x[4] = {Db[oh2], Db[oh1], Db[-ol1], Db[-ol2]};
      if (!CHECK) return fma(8.0, x[2] - x[1], x[0] - x[3]);
      return (h2 ? x[0] : 0.0) - (h1 ? 8.0 * x[1] : 0.0) + (l1 ? 8.0 * x[2] : 0.0) - (l2 ? x[3] : 0.0);
    };
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (a != t) {
        if (g.act[a]) wb[1 + a] += diff(a * 3 + t) * i12;       // du_a/dx_t, from the faces normal to a
        if (g.act[a]) wb[1 + t] += diff(a * 3 + a) * i12;       // du_t/dx_t, from the faces normal to a
      }
    }
  }
}

// Transposed halo fill of the primitive adjoints: every halo cell adds its
// adjoint - with Dbar its share of the transposed centred differences too
// (the interior cells' own share is formed in k_adj_fold) - to its interior
// source cell (the wall-normal velocity's through the image's sign at a
// reflecting wall), with atomics, since an edge cell can own several halo
// cells. One thread per halo cell, numbered as in the primitive halo refresh.
template <bool DBAR>
__global__ void __launch_bounds__(kBlock) k_adj_halo(double* Wbar, const double* __restrict__ Dbar, Geom g) {
  int i, j, k;
  if (!halo_cell(g, (long long)blockIdx.x * kBlock + threadIdx.x, i, j, k)) return;
  const int si = bc_source(i, g.n[0], g.bc[0], g.bc[1]);
  const int sj = bc_source(j, g.n[1], g.bc[2], g.bc[3]);
  const int sk = bc_source(k, g.n[2], g.bc[4], g.bc[5]);
  const long long c = cell_at(g, i, j, k), s = cell_at(g, si, sj, sk);
  double wb[6];
#pragma unroll
  for (int v = 0; v < 6; ++v) wb[v] = Wbar[v * g.vs + c];
  if constexpr (DBAR) {
    const int q[3] = {i, j, k};
    fold_dbar<true>(g, Dbar, c, q, wb);
  }
  const double f[6] = {1.0, bc_sign(i, g.n[0], g.bc[0], g.bc[1]), bc_sign(j, g.n[1], g.bc[2], g.bc[3]),
                       bc_sign(k, g.n[2], g.bc[4], g.bc[5]), 1.0, 1.0};
#pragma unroll
  for (int v = 0; v < 6; ++v) atomic_add(Wbar + v * g.vs + s, f[v] * wb[v]);
}

// The destination of a right-hand-side adjoint: out = a X + b Y + c Z + the
// folded adjoint at the interior cells (null terms are skipped; out may be
// one of X, Y, Z), and, with zero_halo, zeros at its halo cells (otherwise
// they are not touched). The linear combinations of the step adjoint's
// stages are formed here, in the pass that writes out anyway.
struct AdjOut {
  double* out;
  double a, b, c;
  const double* X;
  const double* Y;
  const double* Z;
  int zero_halo;
};

// Per cell s, after k_adj_halo:
// Wbar[s] plus (Dbar non-null) the transposed centred differences of Dbar at
// s, then the transposed primitive map at the state, given by its primitives
// P[s] (rho, u, v, w, p), into the destination o.
__global__ void __launch_bounds__(kBlock) k_adj_fold(const double* __restrict__ P, const double* __restrict__ Wbar,
                                                     const double* __restrict__ Dbar, AdjOut o, Geom g) {
  const PlaneIdx p = plane_index(g, true);
  if (!p.in) return;
  const long long s = p.c;
  if (p.i < 0 || p.i >= g.n[0] || p.j < 0 || p.j >= g.n[1] || p.k < 0 || p.k >= g.n[2]) {
    if (o.zero_halo)
#pragma unroll
      for (int v = 0; v < 5; ++v) o.out[v * g.vs + s] = 0.0;
    return;
  }
  double base[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const long long e = v * g.vs + s;
    double r = 0.0;
    if (o.X) r += o.a * o.X[e];
    if (o.Y) r += o.b * o.Y[e];
    if (o.Z) r += o.c * o.Z[e];
    base[v] = r;
  }
  double wb[6];
#pragma unroll
  for (int v = 0; v < 6; ++v) wb[v] = Wbar[v * g.vs + s];
  if (Dbar) {
    // an interior cell's +-2 neighbours lie inside the padded block
    const int q[3] = {p.i, p.j, p.k};
    fold_dbar<false>(g, Dbar, s, q, wb);
  }
  const double rho = P[s], pr = P[4 * g.vs + s];
  const double u[3] = {P[g.vs + s], P[2 * g.vs + s], P[3 * g.vs + s]};
  const double ir = div_nr(1.0, rho);
  const double gm1 = g.gamma - 1.0;
  // T~ = p / rho
  const double pb = wb[4] + wb[5] * ir;
  double rb = wb[0] - wb[5] * pr * ir * ir;
  // p = (gamma-1)(E - |m|^2 / (2 rho)), u_a = m_a / rho
  const double q2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  rb += pb * gm1 * 0.5 * q2;
  double mb[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    mb[a] = wb[1 + a] * ir - pb * gm1 * u[a];
    rb -= wb[1 + a] * u[a] * ir;
  }
  o.out[s] = base[0] + rb;
  o.out[g.vs + s] = base[1] + mb[0];
  o.out[2 * g.vs + s] = base[2] + mb[1];
  o.out[3 * g.vs + s] = base[3] + mb[2];
  o.out[4 * g.vs + s] = base[4] + pb * gm1;
}

// Coordinates along one axis (n cells, halo h) whose value in a state with
// filled halos is the image of interior coordinate c: m = 0 is c itself,
// m = 1 .. h the low halo cells -m and m = h+1 .. 2h the high halo cells
// n-1 .. n-1+h; false when halo cell m's boundary source is not c. sg is the
// factor the image applies to the axis's velocity (-1 through a wall).
__device__ __forceinline__ bool halo_preimage(int c, int n, int h, int bc_lo, int bc_hi, int m, int& x, double& sg) {
  if (m == 0) {
    x = c;
    sg = 1.0;
    return true;
  }
  x = m <= h ? -m : n - 1 + (m - h);
  if (bc_source(x, n, bc_lo, bc_hi) != c) return false;
  sg = bc_sign(x, n, bc_lo, bc_hi);
  return true;
}

// Adjoint of the initial state U = S(W) (primitive point values W, 5 x
// interior, to the padded conservative state with filled halos): per interior
// cell, the adjoint of the cell's conservative values gathers Ubar over the
// cell and all its halo images (the transpose of the halo fill, in a fixed
// order, so the result is deterministic), then the transposed map of
// (rho, u, v, w, p) -> (rho, rho u, rho v, rho w, p/(gamma-1) + rho |u|^2/2)
// at W is added to Wbar.
__global__ void __launch_bounds__(kBlock) k_state_init_adj(const double* __restrict__ W,
                                                           const double* __restrict__ Ubar,
                                                           double* __restrict__ Wbar, Geom g) {
  const PlaneIdx p = plane_index(g);
  if (!p.in || p.i < 0 || p.i >= g.n[0] || p.j < 0 || p.j >= g.n[1] || p.k < 0 || p.k >= g.n[2]) return;
  double ub[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int a = 0; a <= 2 * g.h[0]; ++a) {
    int x;
    double sx;
    if (!halo_preimage(p.i, g.n[0], g.h[0], g.bc[0], g.bc[1], a, x, sx)) continue;
    for (int b = 0; b <= 2 * g.h[1]; ++b) {
      int y;
      double sy;
      if (!halo_preimage(p.j, g.n[1], g.h[1], g.bc[2], g.bc[3], b, y, sy)) continue;
      for (int c = 0; c <= 2 * g.h[2]; ++c) {
        int z;
        double sz;
        if (!halo_preimage(p.k, g.n[2], g.h[2], g.bc[4], g.bc[5], c, z, sz)) continue;
        const long long e = cell_at(g, x, y, z);
        ub[0] += Ubar[e];
        ub[1] += sx * Ubar[g.vs + e];
        ub[2] += sy * Ubar[2 * g.vs + e];
        ub[3] += sz * Ubar[3 * g.vs + e];
        ub[4] += Ubar[4 * g.vs + e];
      }
    }
  }
  const long long ni = (long long)g.n[0] * g.n[1] * g.n[2];
  const long long s = ((long long)p.k * g.n[1] + p.j) * g.n[0] + p.i;
  const double rho = W[s], u = W[ni + s], v = W[2 * ni + s], w = W[3 * ni + s];
  Wbar[s] += ub[0] + u * ub[1] + v * ub[2] + w * ub[3] + 0.5 * (u * u + v * v + w * w) * ub[4];
  Wbar[ni + s] += rho * (ub[1] + u * ub[4]);
  Wbar[2 * ni + s] += rho * (ub[2] + v * ub[4]);
  Wbar[3 * ni + s] += rho * (ub[3] + w * ub[4]);
  Wbar[4 * ni + s] += ub[4] * g.gm1i;
}

}  // namespace cfd
