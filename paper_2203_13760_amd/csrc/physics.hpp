// Device building blocks of the finite-volume right-hand side (gfx950).
//
// Face-local arithmetic only: WENO5-JS reconstruction, HLLC flux with Einfeldt
// signal speeds, the fourth-order dissipative flux, and the cell-local
// primitive conversion. The sweep kernels feed these from registers; face
// fluxes never leave the register file.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace cfd {

// Grid geometry and physics constants, passed to every kernel by value.
struct Geom {
  int n[3];        // interior cells
  int h[3];        // halo width per axis (0 on inactive axes)
  int N[3];        // padded extents
  long long s[3];  // element strides of the padded block: 1, Nx, Nx*Ny
  long long vs;    // stride between variables: Nx*Ny*Nz
  double dx[3];
  double idx[3];   // 1/dx
  int act[3];      // axis active (n > 1)
  int bc[6];       // boundary types, x-, x+, y-, y+, z-, z+
  double gamma;
  double gm1i;     // 1/(gamma - 1)
  double mu;
  double kappa;    // gamma mu / ((gamma - 1) Pr): lambda grad T = kappa grad(p/rho)
  double cfl;
  double visc_rate;  // 2 max(4/3, gamma/Pr) sum_d dx_d^-2 (times mu/rho gives the diffusive rate)
  int inviscid, viscous, heat;
  int wenoz;       // WENO5-Z instead of WENO5-JS
  int roe;         // Roe flux splitting in characteristic space instead of HLLC
  int weno3;       // WENO3-JS instead of WENO5
  int rusanov;     // Rusanov flux instead of HLLC
  int rk2;         // TVD-RK2 instead of TVD-RK3
  int seg;         // cells per lane of the y / z marches
  int segx;        // rows per segment of a march with x faces
  int xg, xs;      // its wavefronts per segment; strips of single rows
  int nn;          // Rusanov-NN flux (with WENO3-JS): alpha per face from nna
  int safe;        // safe reconstruction: first-order states at faces with a non-positive rho or p
  const double* nnw;  // Rusanov-NN network weights (device, 2305 values)
  double* nna;        // Rusanov-NN alpha per face, [3][padded cells] at the face's left cell
};

// Convective schemes of the sweeps, a compile-time parameter: WENO5-JS or
// WENO5-Z on the primitives with HLLC (the high-order Godunov approach), or
// the flux-splitting approach with Roe eigenvalues and WENO5-JS in
// characteristic space (§3.3; the ROE setup of §5).
constexpr int SCH_JS = 0, SCH_Z = 1, SCH_ROE = 2;
// and the schemes of the implosion of §7.4: WENO3-JS with HLLC, WENO3-JS or
// WENO5-JS with the Rusanov flux
constexpr int SCH_W3 = 3, SCH_JS_RUS = 4, SCH_W3_RUS = 5;
// and the Rusanov-NN flux of §7.4 (WENO3-JS, Rusanov with the dissipation of a
// network, evaluated per face beforehand into Geom::nna)
constexpr int SCH_W3_NN = 6;
__host__ __device__ constexpr bool sch_weno3(int sch) { return sch == SCH_W3 || sch == SCH_W3_RUS || sch == SCH_W3_NN; }
__host__ __device__ constexpr bool sch_rusanov(int sch) {
  return sch == SCH_JS_RUS || sch == SCH_W3_RUS || sch == SCH_W3_NN;
}


// Flux terms of the sweeps, a compile-time parameter: the Euler equations, the
// full Navier-Stokes equations (convective, viscous and heat flux), or any
// other combination, read from the Geom flags at run time. The flags are
// uniform, but branching on them inside a march splits its loop into blocks
// that loads cannot be moved across and keeps zeroed windows live.
constexpr int PHYS_ANY = 0, PHYS_EULER = 1, PHYS_NS = 2;
template <int PHYS>
__host__ __device__ __forceinline__ bool with_inviscid(const Geom& g) { return PHYS != PHYS_ANY || g.inviscid; }
template <int PHYS>
__host__ __device__ __forceinline__ bool with_viscous(const Geom& g) {
  return PHYS == PHYS_NS || (PHYS == PHYS_ANY && g.viscous);
}
template <int PHYS>
__host__ __device__ __forceinline__ bool with_heat(const Geom& g) {
  return PHYS == PHYS_NS || (PHYS == PHYS_ANY && g.heat);
}

__host__ __device__ __forceinline__ double sq(double x) { return x * x; }

// a / b for denominators that are finite, normal and nonzero wherever the
// result is used: the hardware reciprocal estimate r ~ 1/b (v_rcp_f64,
// relative error below 2^-24 on gfx950) refined by one Newton-Raphson step
// r <- r + r (1 - b r) (error below 2^-48), then one residual correction of
// the quotient q <- q + r (a - b q) (Markstein 1990). It skips the range
// scaling and special-case fixup of the IEEE division sequence, about half of
// its instructions; on 4 194 304 random operand pairs (exponents -20 .. 20)
// it returned the correctly rounded a / b every time. The host pass (host-
// compiled tests of the face code) divides.
__host__ __device__ __forceinline__ double div_nr(double a, double b) {
#ifdef __HIP_DEVICE_COMPILE__
  double r = __builtin_amdgcn_rcp(b);
  const double e = fma(-b, r, 1.0);
  r = fma(e, r, r);
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
#else
  return a / b;
#endif
}

// 1 / b for the same denominators: the estimate r with error e = 1 - b r is
// corrected by r (e + e^2) (third order; error below 2^-72 before the final
// rounding, at most 1/2 ulp after it on 4 194 304 operands of 1e-94 to 1e306),
// one operation shorter than div_nr(1, b).
__host__ __device__ __forceinline__ double rcp_nr(double b) {
#ifdef __HIP_DEVICE_COMPILE__
  const double r = __builtin_amdgcn_rcp(b);
  const double e = fma(-b, r, 1.0);
  return fma(fma(e, e, e), r, r);
#else
  return 1.0 / b;
#endif
}

// sqrt(x) for a finite x >= 2^-767 (densities, pressures, squared sound
// speeds): the hardware reciprocal square root estimate y ~ 1/sqrt(x)
// (v_rsq_f64) refined by one Goldschmidt step on the pair g ~ sqrt(x),
// h ~ 1/(2 sqrt(x)) (r = 1/2 - g h, g += g r, h += h r) and one Newton
// correction of the root (g += (x - g^2) h). It has neither range scaling for
// tiny arguments nor fixups for 0 and infinity (x = 0 gives NaN, a negative x
// NaN as sqrt does), and on 4 194 304 random arguments it returned the
// correctly rounded root every time. The host pass takes sqrt.
__host__ __device__ __forceinline__ double sqrt_pos(double x) {
#ifdef __HIP_DEVICE_COMPILE__
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  return fma(fma(-g, g, x), h, g);
#else
  return sqrt(x);
#endif
}

// Keeps x where it stands in the order of the program: what x is formed from
// comes before, what uses it after. Without such points the compiler starts
// independent chains (the five variables of a reconstruction) together, and
// the marches' windows no longer fit the registers beside them.
__host__ __device__ __forceinline__ void pin(double& x) {
#ifdef __HIP_DEVICE_COMPILE__
  asm volatile("" : "+v"(x));
#else
  (void)x;
#endif
}

// Cell index of interior-relative coordinates (i,j,k) (halo cells negative).
__device__ __forceinline__ long long cell_at(const Geom& g, int i, int j, int k) {
  return (long long)(k + g.h[2]) * g.s[2] + (long long)(j + g.h[1]) * g.s[1] + (i + g.h[0]);
}

// Interior source coordinate of a (possibly halo) coordinate c on an axis with
// n cells: periodic image, zero-gradient clamp (§3.7), or the mirror image
// about a reflecting wall (the slip walls of the implosion, §7.4). Applying it
// per axis reproduces the axis-by-axis halo fill, corners included.
__device__ __forceinline__ int bc_source(int c, int n, int bc_lo, int bc_hi) {
  if (c < 0) return bc_lo == 0 ? c + n : (bc_lo == 2 ? -1 - c : 0);
  if (c >= n) return bc_hi == 0 ? c - n : (bc_hi == 2 ? 2 * n - 1 - c : n - 1);
  return c;
}

// Factor of the axis's velocity (momentum) component in the image of c: -1
// through a reflecting wall, else 1. Corner cells take the product over axes.
__device__ __forceinline__ double bc_sign(int c, int n, int bc_lo, int bc_hi) {
  return ((c < 0 && bc_lo == 2) || (c >= n && bc_hi == 2)) ? -1.0 : 1.0;
}

// ---------------------------------------------------------------------------
// WENO5-JS (Jiang & Shu 1996) value at the right face of the centre cell c of
// the stencil (a,b,c,d,e): smoothness indicators beta_k, candidates p_k,
// linear weights (0.1, 0.6, 0.3), alpha_k = d_k/(1e-6 + beta_k)^2, normalised.
// Evaluated with a single division: with s_k = (1e-6 + beta_k)^2 the weights
// are proportional to d_k * prod_{j != k} s_j, and the 1/6 of the candidate
// stencils is applied to the normaliser. Differences and increments on c as in
// weno5_pair. The products stay within FP64 range for |beta_k| up to ~1e70.
__host__ __device__ __forceinline__ double weno5(double a, double b, double c, double d, double e) {
  constexpr double k13 = 13.0 / 12.0;
  constexpr double eps = 1.0e-6;
  const double dm = c - b, dp = d - c;
  const double Db = dm - (b - a), Dc = dp - dm, Dd = (e - d) - dp;
  const double t0 = fma(0.5, Db, dm), t1 = 0.5 * (dm + dp), t2 = fma(-0.5, Dd, dp);
  const double s0 = sq(fma(t0, t0, fma(k13 * Db, Db, eps)));
  const double s1 = sq(fma(t1, t1, fma(k13 * Dc, Dc, eps)));
  const double s2 = sq(fma(t2, t2, fma(k13 * Dd, Dd, eps)));
  const double w0 = s1 * s2, w1 = 6.0 * (s0 * s2), w2 = 3.0 * (s0 * s1);
  const double n = fma(w0, fma(2.0, Db, 3.0 * dm), fma(w1, fma(2.0, dp, dm), w2 * fma(3.0, dp, -Dd)));
  return c + div_nr(n, 6.0 * (w0 + (w1 + w2)));
}

// WENO5-JS at both faces of the centre cell c of the stencil (a, b, c, d, e) =
// q_{i-2} .. q_{i+2}: qr at the right face i+1/2 (the left state there) and
// ql at the left face i-1/2 (the right state there). The two reconstructions
// share their three smoothness indicators in mirrored roles - the indicator
// of cells i-2..i is beta_0 of qr and beta_2 of ql - so each is formed once
// per cell, from the second differences Db, Dc, Dd centred at b, c, d and the
// first differences dm = c - b, dp = d - c:
//   beta_L = 13/12 Db^2 + (dm + Db/2)^2         (a - 4b + 3c = Db + 2 dm)
//   beta_C = 13/12 Dc^2 + ((dm + dp)/2)^2       (b - d = -(dm + dp))
//   beta_R = 13/12 Dd^2 + (dp - Dd/2)^2         (3c - 4d + e = Dd - 2 dp).
// With s_k = (1e-6 + beta_k)^2 the weights of qr are proportional to
// (s_C s_R, 6 s_L s_R, 3 s_L s_C), those of ql to (s_L s_C, 6 s_L s_R,
// 3 s_C s_R): the pairwise products are shared too. The candidates are taken
// as increments on c, six times
//   qr: 2 Db + 3 dm, 2 dp + dm, 3 dp - Dd;  ql: 2 Dd - 3 dp, -(2 dm + dp), -(3 dm + Db),
// one operation each from the differences (three to four from the cell
// values), and their rounding scales with the increment instead of with c;
// mirrored stencils give mirrored values bit for bit.
// Both quotients come from one reciprocal of the product of the two
// normalisers (in range for |beta| below ~1e38). Against candidates from the
// cell values and weights (0.1, 0.6, 0.3): 55 instead of 75 FP64 operations.
__host__ __device__ __forceinline__ void weno5_pair(double a, double b, double c, double d, double e, double& qr,
                                                   double& ql) {
  constexpr double k13 = 13.0 / 12.0;
  constexpr double eps = 1.0e-6;
  const double dm = c - b, dp = d - c;
  const double Db = dm - (b - a), Dc = dp - dm, Dd = (e - d) - dp;
  const double tL = fma(0.5, Db, dm), tC = 0.5 * (dm + dp), tR = fma(-0.5, Dd, dp);
  const double sL = sq(fma(tL, tL, fma(k13 * Db, Db, eps)));
  const double sC = sq(fma(tC, tC, fma(k13 * Dc, Dc, eps)));
  const double sR = sq(fma(tR, tR, fma(k13 * Dd, Dd, eps)));
  const double pCR = sC * sR, pLC = sL * sC;
  const double w1 = 6.0 * (sL * sR), w2 = 3.0 * pLC, v2 = 3.0 * pCR;
  const double X2 = fma(3.0, dp, -Dd), Y2 = fma(3.0, dm, Db);
  const double nr = fma(pCR, Y2 + Db, fma(w1, fma(2.0, dp, dm), w2 * X2));
  const double nl = fma(pLC, Dd - X2, -fma(w1, fma(2.0, dm, dp), v2 * Y2));
  const double dr = pCR + (w1 + w2), dl = pLC + (w1 + v2);
  const double r = rcp_nr(dr * dl) * (1.0 / 6.0);
  qr = fma(nr, dl * r, c);
  ql = fma(nl, dr * r, c);
}

// WENO5-Z (Borges, Carmona, Costa & Don 2008) at both faces of the centre cell,
// as weno5_pair: the same candidates and smoothness indicators, global
// indicator tau5 = |beta_L - beta_R|, weights alpha_k = d_k (1 + tau5 / e_k)
// with e_k = beta_k + 1e-40. With alpha_k = d_k (e_k + tau5) / e_k the weights
// are proportional to d_k (e_k + tau5) prod_{j != k} e_j, of which the two
// faces share all three products. A reciprocal per face keeps the range of
// |beta| (up to ~1e100).
__host__ __device__ __forceinline__ void weno5z_pair(double a, double b, double c, double d, double e, double& qr,
                                                    double& ql) {
  constexpr double k13 = 13.0 / 12.0;
  constexpr double eps = 1.0e-40;
  const double dm = c - b, dp = d - c;
  const double Db = dm - (b - a), Dc = dp - dm, Dd = (e - d) - dp;
  const double tL = fma(0.5, Db, dm), tC = 0.5 * (dm + dp), tR = fma(-0.5, Dd, dp);
  const double eL = fma(tL, tL, fma(k13 * Db, Db, eps));
  const double eC = fma(tC, tC, fma(k13 * Dc, Dc, eps));
  const double eR = fma(tR, tR, fma(k13 * Dd, Dd, eps));
  const double tau = fabs(eL - eR);
  const double a0 = (eL + tau) * (eC * eR), a2 = (eR + tau) * (eL * eC), w1 = 6.0 * ((eC + tau) * (eL * eR));
  const double w2 = 3.0 * a2, v2 = 3.0 * a0;
  const double X2 = fma(3.0, dp, -Dd), Y2 = fma(3.0, dm, Db);
  const double nr = fma(a0, Y2 + Db, fma(w1, fma(2.0, dp, dm), w2 * X2));
  const double nl = fma(a2, Dd - X2, -fma(w1, fma(2.0, dm, dp), v2 * Y2));
  qr = c + div_nr(nr, 6.0 * (a0 + (w1 + w2)));
  ql = c + div_nr(nl, 6.0 * (a2 + (w1 + v2)));
}

// WENO3-JS (Jiang & Shu 1996, r = 2) value at the right face of the centre
// cell b of the stencil (a, b, c): candidates (3b - a)/2 and (b + c)/2,
// smoothness indicators (b - a)^2 and (c - b)^2, linear weights (1/3, 2/3),
// alpha_k = d_k/(1e-6 + beta_k)^2, normalised; one division as in weno5.
__host__ __device__ __forceinline__ double weno3(double a, double b, double c) {
  constexpr double eps = 1.0e-6;
  const double s0 = sq(eps + sq(b - a)), s1 = sq(eps + sq(c - b));
  const double w0 = s1, w1 = 2.0 * s0;  // (1/3)/s0 : (2/3)/s1, times 3 s0 s1
  return div_nr(w0 * (3.0 * b - a) + w1 * (b + c), 2.0 * (w0 + w1));
}

// WENO3-JS at both faces of the centre cell b of (a, b, c): qr = weno3(a, b, c)
// at the right face and ql = weno3(c, b, a) at the left face, sharing the two
// indicators: s0 = (1e-6 + (b - a)^2)^2 and s1 = (1e-6 + (c - b)^2)^2 weigh
// the candidates (3b - a, b + c)/2 of qr as (s1, 2 s0) and (3b - c, b + a)/2
// of ql as (s0, 2 s1).
__host__ __device__ __forceinline__ void weno3_pair(double a, double b, double c, double& qr, double& ql) {
  constexpr double eps = 1.0e-6;
  const double s0 = sq(eps + sq(b - a)), s1 = sq(eps + sq(c - b));
  const double nr = s1 * (3.0 * b - a) + 2.0 * s0 * (b + c);
  const double nl = s0 * (3.0 * b - c) + 2.0 * s1 * (b + a);
  const double dr = s1 + 2.0 * s0, dl = s0 + 2.0 * s1;
  const double r = div_nr(1.0, 2.0 * (dr * dl));
  qr = nr * dl * r;
  ql = nl * dr * r;
}

// Rusanov (local Lax-Friedrichs) flux of §7.4 across a face normal to axis D
// from reconstructed primitive states: (F_L + F_R)/2 - alpha (U_R - U_L)/2 with
// alpha the largest |u -+ c| of the two states (u normal to the face), or the
// given alpha_in (GIVEN: the Rusanov-NN flux).
template <int D, bool GIVEN = false>
__host__ __device__ __forceinline__ void rusanov(double gamma, double gm1i, const double* WL, const double* WR,
                                                 double* F, double alpha_in = 0.0) {
  const double rL = WL[0], pL = WL[4], rR = WR[0], pR = WR[4];
  const double uL = WL[1 + D], uR = WR[1 + D];
  const double kL = 0.5 * rL * (WL[1] * WL[1] + WL[2] * WL[2] + WL[3] * WL[3]);
  const double kR = 0.5 * rR * (WR[1] * WR[1] + WR[2] * WR[2] + WR[3] * WR[3]);
  const double EL = pL * gm1i + kL, ER = pR * gm1i + kR;
  double alpha = alpha_in;
  if constexpr (!GIVEN) {
    const double cL = sqrt_pos(div_nr(gamma * pL, rL)), cR = sqrt_pos(div_nr(gamma * pR, rR));
    alpha = fmax(fmax(fabs(uL - cL), fabs(uL + cL)), fmax(fabs(uR - cR), fabs(uR + cR)));
  }
  const double UL[5] = {rL, rL * WL[1], rL * WL[2], rL * WL[3], EL};
  const double UR[5] = {rR, rR * WR[1], rR * WR[2], rR * WR[3], ER};
  double FL[5], FR[5];
  FL[0] = rL * uL;
  FR[0] = rR * uR;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    FL[1 + a] = FL[0] * WL[1 + a] + (a == D ? pL : 0.0);
    FR[1 + a] = FR[0] * WR[1 + a] + (a == D ? pR : 0.0);
  }
  FL[4] = uL * (EL + pL);
  FR[4] = uR * (ER + pR);
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] = 0.5 * (FL[v] + FR[v]) - 0.5 * alpha * (UR[v] - UL[v]);
}

// ---------------------------------------------------------------------------
// HLLC flux (Toro, Spruce & Speares 1994) with Einfeldt (1988) speeds across a
// face normal to axis D (a division, four reciprocals, five square roots). Inputs:
// reconstructed primitive states (rho, u, v, w, p) left/right. Output in
// physical slot order. The flux comes from one side K: the left one where
// 0 <= S_L or 0 <= S*, else the right one; it is that side's physical flux
// F_K, plus S_K (U*_K - U_K) inside the star region (S_L < 0 <= S* on the
// left, S* < 0 < S_R on the right). The side's values are selected first, so
// one physical flux and one star state are evaluated, and lanes never
// diverge.
template <int D>
__host__ __device__ __forceinline__ void hllc(double gamma, double gm1i, const double* WL, const double* WR, double* F) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const double rL = WL[0], uL = WL[1 + D], pL = WL[4];
  const double rR = WR[0], uR = WR[1 + D], pR = WR[4];
  const double c2L = gamma * pL * rcp_nr(rL), c2R = gamma * pR * rcp_nr(rR);
  const double cL = sqrt_pos(c2L), cR = sqrt_pos(c2R);
  // Einfeldt: Roe-averaged normal velocity and sound-speed bound. A negative
  // density (a face check_face_states reports) makes the averages NaN, which
  // fmin and fmax below pass over, so its 1/rho is not taken from its root.
  const double sL = sqrt_pos(rL), sR = sqrt_pos(rR);
  const double isum = rcp_nr(sL + sR);
  const double ubar = fma(sL, uL, sR * uR) * isum;
  const double dbar = sqrt_pos(isum * fma(0.5 * (sL * sR) * isum, sq(uR - uL), fma(sL, c2L, sR * c2R)));
  const double SL = fmin(uL - cL, ubar - dbar);
  const double SR = fmax(uR + cR, ubar + dbar);
  const double mL = rL * (SL - uL), mR = rR * (SR - uR);  // mass fluxes relative to the waves
  const double Ss = div_nr(pR - pL + uL * mL - uR * mR, mL - mR);
  const bool useL = 0.0 <= SL;
  const bool left = useL || 0.0 <= Ss;
  const bool star = left ? !useL : 0.0 < SR;
  const double r = left ? rL : rR, u = left ? uL : uR, p = left ? pL : pR;
  const double a = left ? WL[1 + T1] : WR[1 + T1], b = left ? WL[1 + T2] : WR[1 + T2];
  const double S = left ? SL : SR, m = left ? mL : mR;
  const double E = p * gm1i + 0.5 * r * (u * u + a * a + b * b);
  // star state U*_K = rho_K (S_K - u_K)/(S_K - S*) (1, S*, t1, t2, E_K/rho_K + (S*-u_K)(S* + p_K/(rho_K (S_K-u_K))));
  // the energy slot is rearranged so that no division by rho_K or m_K
  // remains; outside the star region it may be non-finite and is discarded
  const double i = rcp_nr(S - Ss);
  const double f = m * i;
  const double e = (S - u) * i * E + (Ss - u) * (f * Ss + p * i);
  const double F0 = r * u;
  const double Fk[5] = {F0, F0 * u + p, F0 * a, F0 * b, u * (E + p)};
  const double Uk[5] = {r, r * u, r * a, r * b, E};
  const double Us[5] = {f, f * Ss, f * a, f * b, e};
  double Fn[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) Fn[v] = star ? Fk[v] + S * (Us[v] - Uk[v]) : Fk[v];
  F[0] = Fn[0];
  F[1 + D] = Fn[1];
  F[1 + T1] = Fn[2];
  F[1 + T2] = Fn[3];
  F[4] = Fn[4];
}

// ---------------------------------------------------------------------------
// Stencil window of one face between window cells 2 and 3 (cells f-2 .. f+3
// along the face normal): primitive values q[c][v] (rho,u,v,w,p) and, for the
// four cells f-1 .. f+2, T~ = p/rho and the four tangential velocity
// derivatives the face needs (cell-centred, fourth order):
//   tg[c][0] = d u_D / d x_T1,  tg[c][1] = d u_T1 / d x_T1,
//   tg[c][2] = d u_D / d x_T2,  tg[c][3] = d u_T2 / d x_T2.
struct FaceWindow {
  double q[6][5];
  double T[4];
  double tg[4][4];
};

// Fourth-order central interpolation to the face between b and c (§3.4).
__host__ __device__ __forceinline__ double rc4(double a, double b, double c, double d) {
  return (-a + 9.0 * b + 9.0 * c - d) / 16.0;
}

// Subtracts the dissipative flux F^d (§3.4) across face i+1/2 from F: the
// primitives q[0..3] and T~[0..3] of cells i-1 .. i+2 (velocities and T~ for
// the fourth-order normal derivatives and the face velocities) and the face
// values tf of the tangential derivatives d u_D / d x_T1, d u_D / d x_T2 and
// d u_T1 / d x_T1 + d u_T2 / d x_T2 (the two enter only through div u).
template <int D, int PHYS = PHYS_ANY>
__host__ __device__ __forceinline__ void sub_dissipative_q(const Geom& g, const double (*q)[5], const double* T,
                                                           const double* tf, double* F) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const double i24 = g.idx[D] * (1.0 / 24.0);
  auto dn = [&](double a, double b, double c, double d) { return fma(27.0, c - b, a - d) * i24; };
  auto rc16 = [](double a, double b, double c, double d) { return fma(9.0, b + c, -(a + d)); };  // 16 x the face value
  if (with_viscous<PHYS>(g)) {
    // normal derivatives of the three velocity components
    const double dD = dn(q[0][1 + D], q[1][1 + D], q[2][1 + D], q[3][1 + D]);
    const double d1 = dn(q[0][1 + T1], q[1][1 + T1], q[2][1 + T1], q[3][1 + T1]);
    const double d2 = dn(q[0][1 + T2], q[1][1 + T2], q[2][1 + T2], q[3][1 + T2]);
    const double tDD = g.mu * fma(4.0 / 3.0, dD, (-2.0 / 3.0) * tf[2]);
    const double tD1 = g.mu * (tf[0] + d1);
    const double tD2 = g.mu * (tf[1] + d2);
    const double ufD = rc16(q[0][1 + D], q[1][1 + D], q[2][1 + D], q[3][1 + D]);
    const double uf1 = rc16(q[0][1 + T1], q[1][1 + T1], q[2][1 + T1], q[3][1 + T1]);
    const double uf2 = rc16(q[0][1 + T2], q[1][1 + T2], q[2][1 + T2], q[3][1 + T2]);
    F[1 + D] -= tDD;
    F[1 + T1] -= tD1;
    F[1 + T2] -= tD2;
    F[4] = fma(-1.0 / 16.0, fma(ufD, tDD, fma(uf1, tD1, uf2 * tD2)), F[4]);
  }
  if (with_heat<PHYS>(g)) F[4] = fma(-g.kappa, dn(T[0], T[1], T[2], T[3]), F[4]);
}

// ---------------------------------------------------------------------------
// Flux-splitting approach of §3.3 with the ROE setup of §5: convective flux
// across the face between window cells 2 and 3 (primitives q[0..5] = cells
// f-2 .. f+3). Roe average (sqrt(rho) weights) of cells 2 and 3: velocity u,
// total enthalpy H, sound speed c, c^2 = (gamma-1)(H - |u|^2/2). With
// b = (gamma-1)/c^2 and the waves ordered (u_D - c, entropy, shear T1,
// shear T2, u_D + c), the closed-form left eigenvectors (Toro 2009, §3.2)
// project cell j (velocity v, pressure p) to
//   A   = b (rho |v - u|^2 / 2 + p/(gamma-1)),  S = rho (u_D - v_D) / c,
//   V   = ((A + S)/2, rho - A, rho (v_T1 - u_T1), rho (v_T2 - u_T2), (A - S)/2),
// and, because the Euler flux is F = v_D U + p (0, e_D, v_D), the projected
// flux G = v_D V + p (l_D + l_E v_D) with the left eigenvectors' momentum-D
// and energy entries:
//   G   = v_D V + p (b (v_D - u_D)/2 - 1/(2c), -b (v_D - u_D), 0, 0, b (v_D - u_D)/2 + 1/(2c)).
// Each field is split, G+- = (G +- |lambda| V)/2, reconstructed with WENO5-JS
// (G+ from cells 0..4, G- mirrored from cells 5..1), summed, and transformed
// back with the right eigenvectors (columns (1, u - c e_D, H - u_D c),
// (1, u, |u|^2/2), (0, e_T1, u_T1), (0, e_T2, u_T2), (1, u + c e_D, H + u_D c)).
// No entropy fix (the splitting uses the moduli of the Roe eigenvalues as they are).
template <int D>
__host__ __device__ __forceinline__ void roe_flux(const Geom& g, const double (&q)[6][5], double* F) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const double gm1 = g.gamma - 1.0;
  const double sl = sqrt_pos(q[2][0]), sr = sqrt_pos(q[3][0]);
  const double isum = rcp_nr(sl + sr);
  const double al = sl * isum, ar = sr * isum;
  const double uD = al * q[2][1 + D] + ar * q[3][1 + D];
  const double u1 = al * q[2][1 + T1] + ar * q[3][1 + T1];
  const double u2 = al * q[2][1 + T2] + ar * q[3][1 + T2];
  const double kl = 0.5 * (q[2][1] * q[2][1] + q[2][2] * q[2][2] + q[2][3] * q[2][3]);
  const double kr = 0.5 * (q[3][1] * q[3][1] + q[3][2] * q[3][2] + q[3][3] * q[3][3]);
  const double hp = g.gamma * g.gm1i;  // gamma/(gamma-1): H = hp p/rho + |v|^2/2
  const double H = al * (hp * div_nr(q[2][4], q[2][0]) + kl) + ar * (hp * div_nr(q[3][4], q[3][0]) + kr);
  const double q2 = uD * uD + u1 * u1 + u2 * u2;
  const double c2 = gm1 * (H - 0.5 * q2);
  const double c = sqrt_pos(c2);
  const double ic = rcp_nr(c);
  const double b = gm1 * ic * ic;
  const double lam[5] = {fabs(uD - c), fabs(uD), fabs(uD), fabs(uD), fabs(uD + c)};
  // per cell: A and the pressure term of the projected fluxes; the fields are
  // then split and reconstructed one at a time, and S = rho (u_D - v_D) / c is
  // formed where it is used (fewer live registers: the marches hold two
  // wavefronts per SIMD)
  double A[6], pb[6];
  const double hic = 0.5 * ic;
#pragma unroll
  for (int j = 0; j < 6; ++j) {
    const double rho = q[j][0], p = q[j][4];
    const double dD = q[j][1 + D] - uD, d1 = q[j][1 + T1] - u1, d2 = q[j][1 + T2] - u2;
    A[j] = 0.5 * b * fma(0.5 * rho, fma(dD, dD, fma(d1, d1, d2 * d2)), p * g.gm1i);  // A / 2
    pb[j] = 0.5 * p * b * dD;
    pin(A[j]);
    pin(pb[j]);
  }
  double Gf[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    double Gp[6], Gm[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      const double rho = q[j][0], vD = q[j][1 + D];
      double V, G;
      if (k == 0) {
        V = fma(hic * rho, uD - vD, A[j]);
        G = fma(vD, V, fma(-hic, q[j][4], pb[j]));
      } else if (k == 1) {
        V = fma(-2.0, A[j], rho);
        G = fma(vD, V, -2.0 * pb[j]);
      } else if (k == 4) {
        V = fma(hic * rho, vD - uD, A[j]);
        G = fma(vD, V, fma(hic, q[j][4], pb[j]));
      } else {
        V = rho * (k == 2 ? q[j][1 + T1] - u1 : q[j][1 + T2] - u2);
        G = vD * V;
      }
      Gp[j] = 0.5 * (G + lam[k] * V);
      Gm[j] = 0.5 * (G - lam[k] * V);
    }
    Gf[k] = weno5(Gp[0], Gp[1], Gp[2], Gp[3], Gp[4]);
    pin(Gf[k]);
    Gf[k] += weno5(Gm[5], Gm[4], Gm[3], Gm[2], Gm[1]);
    pin(Gf[k]);
  }
  const double sac = Gf[0] + Gf[4], dac = Gf[4] - Gf[0];
  const double s3 = sac + Gf[1];
  F[0] = s3;
  F[1 + D] = uD * s3 + c * dac;
  F[1 + T1] = u1 * s3 + Gf[2];
  F[1 + T2] = u2 * s3 + Gf[3];
  F[4] = H * sac + uD * c * dac + 0.5 * q2 * Gf[1] + u1 * Gf[2] + u2 * Gf[3];
}

// Numerical flux from the window's primitives q[0..5] (cells i-2 .. i+3 around
// face i+1/2) with the Roe flux splitting, T~ of cells i-1 .. i+2 and the face
// values tf of the tangential derivatives (as in sub_dissipative_q). The
// scheme is a compile-time choice: a run-time branch between schemes
// multiplies the live registers of the sweeps.
template <int D, int PHYS>
__host__ __device__ __forceinline__ void roe_face_flux(const Geom& g, const double (&q)[6][5], const double* T,
                                                       const double* tf, double* G) {
  double F[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (with_inviscid<PHYS>(g)) roe_flux<D>(g, q, F);
#pragma unroll
  for (int v = 0; v < 5; ++v) pin(F[v]);
  sub_dissipative_q<D, PHYS>(g, q + 1, T, tf, F);
#pragma unroll
  for (int v = 0; v < 5; ++v) G[v] = F[v];
}

// Reconstructed states of the cell-centred schemes (all but the Roe flux
// splitting, which projects per face): from the primitives q[0..4] of cells
// i-2 .. i+2, the left state of face i+1/2 (qr) and the right state of face
// i-1/2 (ql), per variable.
template <int SCH>
__host__ __device__ __forceinline__ void recon_pair(double (*q)[5], double* qr, double* ql) {
  static_assert(SCH != SCH_ROE, "a face-by-face scheme");
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    pin(q[2][v]);
    if constexpr (sch_weno3(SCH)) weno3_pair(q[1][v], q[2][v], q[3][v], qr[v], ql[v]);
    else if constexpr (SCH == SCH_Z) weno5z_pair(q[0][v], q[1][v], q[2][v], q[3][v], q[4][v], qr[v], ql[v]);
    else weno5_pair(q[0][v], q[1][v], q[2][v], q[3][v], q[4][v], qr[v], ql[v]);
    pin(qr[v]);
    pin(ql[v]);
  }
}

// Numerical flux G = F - F^d across face i+1/2 (§3.3, §3.4) from its
// reconstructed states WL, WR, the primitives q[0..3] and T~[0..3] of cells
// i-1 .. i+2, the face values tf of the tangential derivatives (as in
// sub_dissipative_q) and, for the Rusanov-NN flux, the face's alpha.
template <int D, int SCH, int PHYS>
__host__ __device__ __forceinline__ void face_flux_states(const Geom& g, const double* WL, const double* WR,
                                                          const double (*q)[5], const double* T, const double* tf,
                                                          double alpha, double* G) {
  double F[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (with_inviscid<PHYS>(g)) {
    if constexpr (SCH == SCH_W3_NN) rusanov<D, true>(g.gamma, g.gm1i, WL, WR, F, alpha);
    else if constexpr (sch_rusanov(SCH)) rusanov<D>(g.gamma, g.gm1i, WL, WR, F);
    else hllc<D>(g.gamma, g.gm1i, WL, WR, F);
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) pin(F[v]);
  sub_dissipative_q<D, PHYS>(g, q, T, tf, F);
#pragma unroll
  for (int v = 0; v < 5; ++v) G[v] = F[v];
}

// Numerical flux G = F - F^d across the face (§3.3, §3.4) of a full window with
// the default scheme, each reconstruction on its own: what face_flux_rev
// reverses (used by its host check).
template <int D>
__host__ __device__ __forceinline__ void face_flux(const Geom& g, const FaceWindow& w, double* G) {
  double F[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, tf[3] = {0.0, 0.0, 0.0};
  if (g.inviscid) {
    double WL[5], WR[5];
    for (int v = 0; v < 5; ++v) {
      WL[v] = weno5(w.q[0][v], w.q[1][v], w.q[2][v], w.q[3][v], w.q[4][v]);
      WR[v] = weno5(w.q[5][v], w.q[4][v], w.q[3][v], w.q[2][v], w.q[1][v]);
    }
    hllc<D>(g.gamma, g.gm1i, WL, WR, F);
  }
  if (g.viscous) {
    auto face = [&](int k) { return rc4(w.tg[0][k], w.tg[1][k], w.tg[2][k], w.tg[3][k]); };
    tf[0] = face(0);
    tf[1] = face(2);
    tf[2] = face(1) + face(3);
  }
  sub_dissipative_q<D>(g, w.q + 1, w.T, tf, F);
  for (int v = 0; v < 5; ++v) G[v] = F[v];
}

}  // namespace cfd
