// Forward kernels of one right-hand-side evaluation / TVD-RK3 stage (gfx950).
//
// Primitives: U -> P = (rho,u,v,w,p) on the padded grid once per call, halos
// by gather from their interior source cells (so U's own halo is never read),
// plus the CFL rate max. After that the last sweep of a stage stores the
// primitives of the cells it updates, with their CFL rate and health bits, and
// either their halo images too (small grids) or a halo pass follows.
//
// Sweeps: each face flux is computed once in registers and differenced into
// its two cells, the tangential velocity derivatives of the viscous flux
// formed from P on the way.
//   cell-centred schemes, 3D: a z march (lanes along x, a register window
//     moving along z) that leaves -D_z in R, then a y march whose rows also
//     form their x faces between neighbouring lanes and that stores the new
//     state;
//   2D: that second sweep alone, with the whole update;
//   1D and the Roe splitting: one sweep per active axis (x: one lane per face,
//     lane shifts carry the left-face flux).
#pragma once
#include "physics.hpp"

namespace cfd {

// Device control block of a solver.
struct DevCtl {
  double dt;   // step of the current step (0: step disabled, t_end reached)
  int status;  // health bits, see cfd_check
  unsigned done;  // blocks of a step's last sweep that have published their CFL rate (0 between sweeps)
};

constexpr int kBlock = 256;
constexpr int kGradComps = 9;  // adjoint of d u_a / d x_b accumulated at component a*3+b

// What a sweep does with the divergence D of its axis: MODE_WRITE stores
// R = -D, MODE_ACC R -= D; the RK modes apply the stage update with R = -D
// (MODE_WRITE_RK) or R - D (MODE_ACC_RK) and store a new state and its
// primitives. The update stays in one place: with its share of the state formed
// in the first sweep (V = a Un + b (Uk - dt D_z) in R, the last sweep V - b dt D)
// the state is rounded once more a stage, and a step of a 3D box was 12 to 28 %
// further from its value in extended precision.
enum SweepMode { MODE_WRITE = 0, MODE_ACC = 1, MODE_ACC_RK = 2, MODE_WRITE_RK = 3 };
__host__ __device__ constexpr bool mode_rk(int m) { return m >= MODE_ACC_RK; }

struct StageIO {
  double* R;         // right-hand-side accumulator (padded layout)
  const double* Un;  // state at the start of the step
  const double* Uk;  // stage input state
  double* Uout;      // stage output state (may alias Un in the last stage)
  double a, b;       // Uout = a Un + b (Uk + dt R)
  const double* dtp; // step size on the device; nullptr: the fixed step dt
  double dt;
  double* Pn;        // primitives of Uout, interior cells (sweeps with PN set)
  double* partial;   // CFL rate slots (PN sweeps with PRIM_CFL in `what`)
  DevCtl* ctl;       // health bits (PN sweeps with PRIM_HEALTH in `what`)
  int what;
  int next;          // the sweep ends a step and forms the next one's size (dt_next)
  double cfl, t_end;
  double* t;
};

__device__ __forceinline__ double stage_dt(const StageIO& io) { return io.dtp ? *io.dtp : io.dt; }
__device__ __forceinline__ bool step_disabled(const double* dtp) { return dtp != nullptr && *dtp == 0.0; }

// Kernels over the padded grid use a plane-indexed launch: blockIdx.y is the
// padded z index, and threads cover the x-y plane with a 32-bit in-plane index.
struct PlaneIdx {
  int i, j, k;      // interior-relative coordinates (halo cells negative)
  long long c;      // padded cell index
  bool in;          // inside the padded grid
};

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2). The XCD-major order gives each XCD one contiguous range of logical
// blocks - consecutive planes - so the neighbour planes a stencil re-reads stay
// in that XCD's L2. XCD x receives the hardware blocks b = x, x+8, x+16, ...;
// the first nb % 8 XCDs get one block more, and the map is a permutation.
constexpr int kXcds = 8;

__device__ __forceinline__ int xcd_major_block(int b, int nb) {
  const int x = b % kXcds, local = b / kXcds;
  const int q = nb / kXcds, r = nb % kXcds;
  return x < r ? x * (q + 1) + local : r * (q + 1) + (x - r) * q + local;
}

// bx, by: block coordinates of a plane-indexed launch of gx x gy blocks.
__device__ __forceinline__ PlaneIdx plane_index_at(const Geom& g, int bx, int by, int gx, int gy, bool xcd_major) {
  PlaneIdx p;
  const int plane = g.N[0] * g.N[1];
  if (xcd_major) {
    const int logical = xcd_major_block(by * gx + bx, gx * gy);
    by = logical / gx;
    bx = logical - by * gx;
  }
  const int t = bx * kBlock + threadIdx.x;
  p.in = t < plane;
  const int jj = t / g.N[0];
  const int ii = t - jj * g.N[0];
  p.i = ii - g.h[0];
  p.j = jj - g.h[1];
  p.k = by - g.h[2];
  p.c = (long long)by * plane + t;
  return p;
}

__device__ __forceinline__ PlaneIdx plane_index(const Geom& g, bool xcd_major = false) {
  return plane_index_at(g, blockIdx.x, blockIdx.y, gridDim.x, gridDim.y, xcd_major);
}

// Number of blocks along x of a plane-indexed launch.
__host__ __device__ __forceinline__ int plane_blocks_x(const Geom& g) {
  return (g.N[0] * g.N[1] + kBlock - 1) / kBlock;
}

// ----------------------------------------------------------------------------
// Halo refresh of the primitives P after a sweep stored the
// interior ones, one thread per halo cell; skipped with the step. Halo cells
// are numbered slab by slab: the z halo planes (whole padded planes), then
// for interior z the y halo rows (whole padded rows), then for interior z and
// y the x halo cells.
__host__ __device__ __forceinline__ long long halo_cells(const Geom& g) {
  return 2LL * g.h[2] * g.N[0] * g.N[1] + 2LL * g.h[1] * g.N[0] * g.n[2] + 2LL * g.h[0] * g.n[1] * g.n[2];
}

__host__ __device__ __forceinline__ int halo_blocks(const Geom& g) {
  const long long n = halo_cells(g);
  return (int)(n > 0 ? (n + kBlock - 1) / kBlock : 1);
}

// Interior-relative coordinates of halo cell number t (numbered as above);
// false past the last halo cell.
__device__ __forceinline__ bool halo_cell(const Geom& g, long long t, int& i, int& j, int& k) {
  const long long zs = 2LL * g.h[2] * g.N[0] * g.N[1];
  const long long ys = 2LL * g.h[1] * g.N[0] * g.n[2];
  const long long xs = 2LL * g.h[0] * g.n[1] * g.n[2];
  if (t < zs) {
    const long long plane = (long long)g.N[0] * g.N[1];
    const int kk = (int)(t / plane);  // 0 .. 2h-1
    const long long r = t - kk * plane;
    j = (int)(r / g.N[0]) - g.h[1];
    i = (int)(r - (long long)(j + g.h[1]) * g.N[0]) - g.h[0];
    k = kk < g.h[2] ? kk - g.h[2] : g.n[2] + (kk - g.h[2]);
  } else if ((t -= zs) < ys) {
    const long long slab = 2LL * g.h[1] * g.N[0];
    k = (int)(t / slab);
    const long long r = t - k * slab;
    const int jj = (int)(r / g.N[0]);  // 0 .. 2h-1
    i = (int)(r - (long long)jj * g.N[0]) - g.h[0];
    j = jj < g.h[1] ? jj - g.h[1] : g.n[1] + (jj - g.h[1]);
  } else if ((t -= ys) < xs) {
    const long long row = 2LL * g.h[0];
    const long long kj = t / row;
    const int ii = (int)(t - kj * row);
    k = (int)(kj / g.n[1]);
    j = (int)(kj - (long long)k * g.n[1]);
    i = ii < g.h[0] ? ii - g.h[0] : g.n[0] + (ii - g.h[0]);
  } else {
    return false;
  }
  return true;
}

__device__ __forceinline__ void prim_halo_body(double* P, const Geom& g, long long t) {
  int i, j, k;  // interior-relative coordinates of the halo cell
  if (!halo_cell(g, t, i, j, k)) return;
  const int si = bc_source(i, g.n[0], g.bc[0], g.bc[1]);
  const int sj = bc_source(j, g.n[1], g.bc[2], g.bc[3]);
  const int sk = bc_source(k, g.n[2], g.bc[4], g.bc[5]);
  const long long c = cell_at(g, i, j, k), s = cell_at(g, si, sj, sk);
  const double sg[3] = {bc_sign(i, g.n[0], g.bc[0], g.bc[1]), bc_sign(j, g.n[1], g.bc[2], g.bc[3]),
                        bc_sign(k, g.n[2], g.bc[4], g.bc[5])};
#pragma unroll
  for (int v = 0; v < 5; ++v) P[v * g.vs + c] = (v >= 1 && v <= 3 ? sg[v - 1] : 1.0) * P[v * g.vs + s];
}

__global__ void __launch_bounds__(kBlock) k_prim_halo(double* P, Geom g, const double* dtp) {
  if (step_disabled(dtp)) return;
  prim_halo_body(P, g, (long long)blockIdx.x * kBlock + threadIdx.x);
}

// Halo refresh of a state U in place from its interior, one thread per halo cell.
__global__ void __launch_bounds__(kBlock) k_fill_halo(double* U, Geom g) {
  int i, j, k;
  if (!halo_cell(g, (long long)blockIdx.x * kBlock + threadIdx.x, i, j, k)) return;
  const int si = bc_source(i, g.n[0], g.bc[0], g.bc[1]);
  const int sj = bc_source(j, g.n[1], g.bc[2], g.bc[3]);
  const int sk = bc_source(k, g.n[2], g.bc[4], g.bc[5]);
  const long long c = cell_at(g, i, j, k), s = cell_at(g, si, sj, sk);
  const double sg[3] = {bc_sign(i, g.n[0], g.bc[0], g.bc[1]), bc_sign(j, g.n[1], g.bc[2], g.bc[3]),
                        bc_sign(k, g.n[2], g.bc[4], g.bc[5])};
#pragma unroll
  for (int v = 0; v < 5; ++v) U[v * g.vs + c] = (v >= 1 && v <= 3 ? sg[v - 1] : 1.0) * U[v * g.vs + s];
}

// Conservative interior state from primitive point values W (5 x interior, no halo).
__global__ void __launch_bounds__(kBlock) k_state_init(const double* W, double* U, Geom g) {
  const PlaneIdx p = plane_index(g);
  if (!p.in || p.i < 0 || p.i >= g.n[0] || p.j < 0 || p.j >= g.n[1] || p.k < 0 || p.k >= g.n[2]) return;
  const long long ni = (long long)g.n[0] * g.n[1] * g.n[2];
  const long long s = ((long long)p.k * g.n[1] + p.j) * g.n[0] + p.i;
  const double rho = W[s], u = W[ni + s], v = W[2 * ni + s], w = W[3 * ni + s], pr = W[4 * ni + s];
  U[p.c] = rho;
  U[g.vs + p.c] = rho * u;
  U[2 * g.vs + p.c] = rho * v;
  U[3 * g.vs + p.c] = rho * w;
  U[4 * g.vs + p.c] = pr / (g.gamma - 1.0) + 0.5 * rho * (u * u + v * v + w * w);
}

__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
  return x;
}

// Block maximum (wavefront shuffles, then across the block's wavefronts via
// LDS); the result is valid in thread 0.
__device__ __forceinline__ double block_max(double x) {
  __shared__ double part[kBlock / 64];
  x = wave_max(x);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) part[w] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) x = fmax(x, part[i]);
  }
  __syncthreads();  // part[] may be reused by the block's next reduction
  return x;
}

// CFL rate of an interior cell from its primitives w = (rho, u, v, w, p, p/rho)
// and ir = 1/rho: max(sum_d (|u_d| + c)/dx_d, (mu/rho) visc_rate), c^2 = gamma p/rho.
__device__ __forceinline__ double cfl_rate(const Geom& g, const double* w, double ir) {
  const double c = sqrt_pos(g.gamma * w[5]);
  double s = 0.0;
#pragma unroll
  for (int d = 0; d < 3; ++d)
    if (g.act[d]) s += (fabs(w[1 + d]) + c) * g.idx[d];
  if (g.viscous || g.heat) s = fmax(s, (g.mu * ir) * g.visc_rate);
  return s;
}

// CFL rate maxima are kept in kCflSlots slots (the bits of non-negative
// doubles order like unsigned integers, so atomicMax on the bits is a max).
// Each block folds its maximum into slot (block index mod kCflSlots), which
// spreads the atomics; k_dt reduces the slots and clears them for the next step.
constexpr int kCflSlots = 256;

__device__ __forceinline__ void publish_rate(double* slots, int block_index, double s) {
  s = block_max(s);
  if (threadIdx.x == 0 && s > 0.0)
    atomicMax(reinterpret_cast<unsigned long long*>(slots) + (block_index & (kCflSlots - 1)),
              (unsigned long long)__double_as_longlong(s));
}

// Primitive variables w = (rho, u, v, w, p, p/rho) of conservative values q;
// returns 1/rho.
__device__ __forceinline__ double cons_to_prim(const Geom& g, const double* q, double* w) {
  const double rho = q[0];
  w[0] = rho;
  const double ir = div_nr(1.0, rho);
  w[1] = q[1] * ir;
  w[2] = q[2] * ir;
  w[3] = q[3] * ir;
  w[4] = (g.gamma - 1.0) * (q[4] - 0.5 * (q[1] * w[1] + q[2] * w[2] + q[3] * w[3]));
  w[5] = w[4] * ir;
  return ir;
}

// Health bits of a cell: 1 non-finite conservative value, 2 rho <= 0, 4 p <= 0;
// and of a face: 8 a reconstructed state with rho <= 0 or p <= 0.
constexpr int kBadFace = 8;

// Face check of the cell-centred schemes: a reconstructed state of the face
// with a non-positive (or non-finite) density or pressure sets kBadFace in
// bad; with safe reconstruction both states then take the values of the two
// cells next to the face (qa left, qb right: the first-order reconstruction).
__device__ __forceinline__ void check_face_states(const Geom& g, bool use, double* WL, double* WR,
                                                  const double* qa, const double* qb, int& bad) {
  const bool ok = !use || (WL[0] > 0.0 && WL[4] > 0.0 && WR[0] > 0.0 && WR[4] > 0.0);
  if (__builtin_expect(__any(!ok), 0)) {  // a branch of the whole wavefront, hardly ever taken
    bad |= ok ? 0 : kBadFace;
    if (g.safe) {
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        WL[v] = ok ? WL[v] : qa[v];
        WR[v] = ok ? WR[v] : qb[v];
      }
    }
  }
}

// Health bits of a cell: 1 non-finite conservative value, 2 rho <= 0, 4 p <= 0.
__device__ __forceinline__ int health_bits(const double* q, double p) {
  int bad = 0;
  if (!isfinite(q[0]) || !isfinite(q[1]) || !isfinite(q[2]) || !isfinite(q[3]) || !isfinite(q[4])) bad |= 1;
  if (!(q[0] > 0.0)) bad |= 2;
  if (!(p > 0.0)) bad |= 4;
  return bad;
}

// Primitive variables on the padded grid, gathered through the boundary map.
// Over interior cells, `what` bit 0 adds the CFL rate (block maxima written
// to partial[], one per block) and bit 1 the health bits.
// Bit 2 also stores T~ = p/rho (component 5), which no kernel reads: the
// sweeps form it from their windows.
constexpr int PRIM_CFL = 1, PRIM_HEALTH = 2, PRIM_T = 4;

__device__ __forceinline__ void prim_body(const double* __restrict__ U, double* __restrict__ P, const Geom& g,
                                          DevCtl* ctl, int what, double* __restrict__ partial, const PlaneIdx& q,
                                          int part_index) {
  double smax = 0.0;
  if (q.in) {
    const int si = bc_source(q.i, g.n[0], g.bc[0], g.bc[1]);
    const int sj = bc_source(q.j, g.n[1], g.bc[2], g.bc[3]);
    const int sk = bc_source(q.k, g.n[2], g.bc[4], g.bc[5]);
    const long long s = cell_at(g, si, sj, sk);
    const long long c = q.c;
    double u[5], w[6];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = U[v * g.vs + s];
    u[1] *= bc_sign(q.i, g.n[0], g.bc[0], g.bc[1]);
    u[2] *= bc_sign(q.j, g.n[1], g.bc[2], g.bc[3]);
    u[3] *= bc_sign(q.k, g.n[2], g.bc[4], g.bc[5]);
    const double ir = cons_to_prim(g, u, w);
#pragma unroll
    for (int v = 0; v < 5; ++v) P[v * g.vs + c] = w[v];
    if (what & PRIM_T) P[5 * g.vs + c] = w[5];
    if (what && s == c) {
      if (what & PRIM_CFL) smax = cfl_rate(g, w, ir);
      if (what & PRIM_HEALTH) {
        const int bad = health_bits(u, w[4]);
        if (bad) atomicOr(&ctl->status, bad);
      }
    }
  }
  if (what & PRIM_CFL) publish_rate(partial, part_index, smax);
}

__global__ void __launch_bounds__(kBlock) k_prim(const double* __restrict__ U, double* __restrict__ P,
                                                 Geom g, DevCtl* ctl, int what, const double* dtp,
                                                 double* __restrict__ partial) {
  if (step_disabled(dtp)) return;
  prim_body(U, P, g, ctl, what, partial, plane_index(g), blockIdx.y * gridDim.x + blockIdx.x);
}

// Prologue of a right-hand side in one pass over the padded grid: the
// primitives of U, its halo cells refreshed in place from the interior cells
// that are read for them anyway, and the halo cells of R set to zero (the
// sweeps write R's interior).
__global__ void __launch_bounds__(kBlock) k_prim_rhs(double* U, double* __restrict__ P, double* __restrict__ R, Geom g) {
  const PlaneIdx q = plane_index(g);
  if (!q.in) return;
  const int si = bc_source(q.i, g.n[0], g.bc[0], g.bc[1]);
  const int sj = bc_source(q.j, g.n[1], g.bc[2], g.bc[3]);
  const int sk = bc_source(q.k, g.n[2], g.bc[4], g.bc[5]);
  const long long s = cell_at(g, si, sj, sk), c = q.c;
  double u[5], w[6];
#pragma unroll
  for (int v = 0; v < 5; ++v) u[v] = U[v * g.vs + s];
  u[1] *= bc_sign(q.i, g.n[0], g.bc[0], g.bc[1]);
  u[2] *= bc_sign(q.j, g.n[1], g.bc[2], g.bc[3]);
  u[3] *= bc_sign(q.k, g.n[2], g.bc[4], g.bc[5]);
  if (s != c) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      U[v * g.vs + c] = u[v];
      R[v * g.vs + c] = 0.0;
    }
  }
  cons_to_prim(g, u, w);
#pragma unroll
  for (int v = 0; v < 5; ++v) P[v * g.vs + c] = w[v];
}

// CFL rate maxima of a state (interior cells only), for cfd_compute_dt.
__global__ void __launch_bounds__(kBlock) k_cfl(const double* __restrict__ U, Geom g,
                                                double* __restrict__ partial) {
  const PlaneIdx q = plane_index(g);
  double smax = 0.0;
  if (q.in && q.i >= 0 && q.i < g.n[0] && q.j >= 0 && q.j < g.n[1] && q.k >= 0 && q.k < g.n[2]) {
    double u[5], w[6];
#pragma unroll
    for (int v = 0; v < 5; ++v) u[v] = U[v * g.vs + q.c];
    const double ir = cons_to_prim(g, u, w);
    smax = cfl_rate(g, w, ir);
  }
  publish_rate(partial, blockIdx.y * gridDim.x + blockIdx.x, smax);
}

// Step size from the CFL rate maximum m (or the fixed one), clipped to end at
// t_end (> 0) and zero once t has reached it.
__device__ __forceinline__ double step_size(double cfl, double m, double fixed_dt, const double* t, double t_end) {
  double dt = fixed_dt > 0.0 ? fixed_dt : cfl / m;
  if (t != nullptr && t_end > 0.0) {
    const double rem = t_end - *t;
    dt = rem > 0.0 ? fmin(dt, rem) : 0.0;
  }
  return dt;
}

// Size of the next step: fixed, or cfl / (max of the npart CFL rate slots,
// which are cleared); clipped to t_end (> 0) and zero once t has reached it.
// One block of kBlock threads.
__device__ __forceinline__ void dt_body(DevCtl* ctl, double cfl, double fixed_dt, double t_end, const double* t,
                                        double* dt_out, double* __restrict__ partial, int npart) {
  double m = 0.0;
  if (!(fixed_dt > 0.0)) {
    for (int i = threadIdx.x; i < npart; i += blockDim.x) m = fmax(m, partial[i]);
    m = block_max(m);  // every slot has been read once this returns
    for (int i = threadIdx.x; i < npart; i += blockDim.x) partial[i] = 0.0;
  }
  if (threadIdx.x != 0) return;
  const double dt = step_size(cfl, m, fixed_dt, t, t_end);
  ctl->dt = dt;
  if (dt_out != nullptr) *dt_out = dt;
}

__global__ void __launch_bounds__(kBlock) k_dt(DevCtl* ctl, double cfl, double fixed_dt, double t_end,
                                               const double* t, double* dt_out, double* __restrict__ partial,
                                               int npart) {
  dt_body(ctl, cfl, fixed_dt, t_end, t, dt_out, partial, npart);
}

// ----------------------------------------------------------------------------
// Loads and stores at a wavefront-uniform base plus a 32-bit byte offset per
// lane: the base of every (variable, neighbour) pair stays in scalar
// registers and all of a lane's accesses share one offset register.
__device__ __forceinline__ double ld_at(const double* base, unsigned off) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + off);
}
__device__ __forceinline__ void st_at(double* base, unsigned off, double x) {
  *reinterpret_cast<double*>(reinterpret_cast<char*>(base) + off) = x;
}

// A value that is the same in all lanes, kept in a scalar register. A march
// forms its cell index from uniform(f): without it the loop passes turn
// base + offset back into one 64-bit address per lane and access.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ int wave_in_block() { return uniform((int)threadIdx.x >> 6); }

// Face window loads.
__device__ __forceinline__ void load_prims(const double* __restrict__ P, long long vs, long long c,
                                           double* q) {
#pragma unroll
  for (int v = 0; v < 5; ++v) q[v] = P[v * vs + c];
}

// Tangential velocity derivatives at a cell for faces normal to D,
// fourth-order central differences of the primitives across the cell (§3.4):
// d u_D / d x_T1, d u_T1 / d x_T1, d u_D / d x_T2, d u_T2 / d x_T2. The
// tangential coordinates of every cell a face stencil touches are interior, so
// the +-2 neighbours lie inside the padded block.
//
// In two halves: the sixteen loads, and the arithmetic, without branches. An
// inactive axis gets stride 0 and weight 0 (the difference of a cell with
// itself is exactly 0). Callers issue all loads before any use (a scheduling
// barrier keeps the compiler from interleaving loads and uses, which
// serialises their latencies).
template <int D>
__device__ __forceinline__ void tangential_load(const Geom& g, const double* __restrict__ P, long long c,
                                                double (&x)[4][4]) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const long long s1 = g.act[T1] ? g.s[T1] : 0, s2 = g.act[T2] ? g.s[T2] : 0;
  const double* q[4] = {P + (1 + D) * g.vs + c, P + (1 + T1) * g.vs + c, P + (1 + D) * g.vs + c,
                        P + (1 + T2) * g.vs + c};
  const long long st[4] = {s1, s1, s2, s2};
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    x[m][0] = q[m][-2 * st[m]];
    x[m][1] = q[m][-st[m]];
    x[m][2] = q[m][st[m]];
    x[m][3] = q[m][2 * st[m]];
  }
}

// The three sums the cell-centred sweeps carry (layout of sub_dissipative_q):
// the two derivatives along their own axes enter the flux only as a sum.
template <int D>
__device__ __forceinline__ void tangential_combine3(const Geom& g, const double (&x)[4][4], double* tg) {
  constexpr int T1 = (D + 1) % 3, T2 = (D + 2) % 3;
  const double w1 = g.act[T1] ? g.idx[T1] * (1.0 / 12.0) : 0.0, w2 = g.act[T2] ? g.idx[T2] * (1.0 / 12.0) : 0.0;
  auto diff = [](const double* y) { return fma(8.0, y[2] - y[1], y[0] - y[3]); };
  tg[0] = diff(x[0]) * w1;
  tg[1] = diff(x[2]) * w2;
  tg[2] = fma(diff(x[1]), w1, diff(x[3]) * w2);
}

template <int D>
__device__ __forceinline__ void tangential_at3(const Geom& g, const double* __restrict__ P, long long c, double* tg) {
  double x[4][4];
  tangential_load<D>(g, P, c, x);
  tangential_combine3<D>(g, x, tg);
}

// Halo images of one axis of an interior coordinate c: the low halo cells
// [lo, lo + nlo) and the high ones [hi, hi + nhi) whose boundary source is c.
struct AxisImages {
  int lo, nlo, hi, nhi;
  __device__ __forceinline__ AxisImages(int c, int n, int h, int bc_lo, int bc_hi) {
    const bool first = c < h, last = c >= n - h;
    nlo = bc_lo == 0 ? last : (bc_lo == 2 ? first : (c == 0 ? h : 0));
    lo = bc_lo == 0 ? c - n : (bc_lo == 2 ? -1 - c : -h);
    nhi = bc_hi == 0 ? first : (bc_hi == 2 ? last : (c == n - 1 ? h : 0));
    hi = bc_hi == 0 ? c + n : (bc_hi == 2 ? 2 * n - 1 - c : n);
  }
  __device__ __forceinline__ int count() const { return 1 + nlo + nhi; }
  __device__ __forceinline__ int at(int c, int m) const { return m == 0 ? c : (m <= nlo ? lo + m - 1 : hi + m - 1 - nlo); }
};

// Stores the primitives w of interior cell (i, j, k) at its halo images: what
// the halo pass copies, without its launch. Worth it on grids whose sweeps
// take a few microseconds; on large ones the scattered stores cost the sweep
// what the pass costs.
__device__ __forceinline__ void store_images(double* P, const Geom& g, int i, int j, int k, const double* w) {
  const bool edge = (g.act[0] && (i < g.h[0] || i >= g.n[0] - g.h[0])) ||
                    (g.act[1] && (j < g.h[1] || j >= g.n[1] - g.h[1])) ||
                    (g.act[2] && (k < g.h[2] || k >= g.n[2] - g.h[2]));
  if (!edge) return;
  const AxisImages X(i, g.n[0], g.h[0], g.bc[0], g.bc[1]), Y(j, g.n[1], g.h[1], g.bc[2], g.bc[3]),
      Z(k, g.n[2], g.h[2], g.bc[4], g.bc[5]);
  const int nx = g.act[0] ? X.count() : 1, ny = g.act[1] ? Y.count() : 1, nz = g.act[2] ? Z.count() : 1;
  for (int c = 0; c < nz; ++c)
    for (int b = 0; b < ny; ++b)
      for (int a = c + b == 0 ? 1 : 0; a < nx; ++a) {
        const int x = X.at(i, a), y = Y.at(j, b), z = Z.at(k, c);
        const long long e = cell_at(g, x, y, z);
        P[e] = w[0];
        P[g.vs + e] = bc_sign(x, g.n[0], g.bc[0], g.bc[1]) * w[1];
        P[2 * g.vs + e] = bc_sign(y, g.n[1], g.bc[2], g.bc[3]) * w[2];
        P[3 * g.vs + e] = bc_sign(z, g.n[2], g.bc[4], g.bc[5]) * w[3];
        P[4 * g.vs + e] = w[4];
      }
}

// Writing the divergence contribution D = (G+ - G-)/dx of one cell, in two
// halves so that a marching sweep can issue the loads of the cell's update
// (accumulated R, stage states) before the face arithmetic and store after
// it: EmitIn holds the loaded values. MODE_WRITE / MODE_ACC store R = -D or
// R - D; the RK modes store Uout = a Un + b (Uk + dt R) instead of R.
struct EmitIn {
  double r[5], un[5], uk[5];
};

// Cell c + off (off in bytes; a lane's offset from a wavefront-uniform c, or 0).
// A stage whose weight a of U^n is zero (TVD-RK3 stage 1, where U^(k) is
// U^n) does not load U^n.
template <int MODE>
__device__ __forceinline__ void emit_fetch(const StageIO& io, long long vs, long long c, unsigned off, EmitIn& in) {
  const bool with_un = io.a != 0.0;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const long long e = v * vs + c;
    if (MODE == MODE_ACC || MODE == MODE_ACC_RK) in.r[v] = ld_at(io.R + e, off);
    if (mode_rk(MODE)) {
      in.un[v] = with_un ? ld_at(io.Un + e, off) : 0.0;
      in.uk[v] = ld_at(io.Uk + e, off);
    }
  }
}

// (i, j, k): the cell's coordinates, for its halo images.
// IMG: also store the primitives' halo images.
template <int MODE, bool PN = false, bool IMG = false>
__device__ __forceinline__ void emit_put(const StageIO& io, const Geom& g, long long c, unsigned off, const double* D,
                                         const EmitIn& in, double dt, double& smax, int& bad, int i, int j, int k) {
  double uo[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const long long e = v * g.vs + c;
    if (MODE == MODE_WRITE || MODE == MODE_ACC) {
      st_at(io.R + e, off, MODE == MODE_WRITE ? -D[v] : in.r[v] - D[v]);
    } else {
      const double r = MODE == MODE_WRITE_RK ? -D[v] : in.r[v] - D[v];
      uo[v] = io.a * in.un[v] + io.b * (in.uk[v] + dt * r);
      st_at(io.Uout + e, off, uo[v]);
    }
  }
  if constexpr (PN && mode_rk(MODE)) {
    double w[6];
    const double ir = cons_to_prim(g, uo, w);
#pragma unroll
    for (int v = 0; v < 5; ++v) st_at(io.Pn + v * g.vs + c, off, w[v]);
    if constexpr (IMG) store_images(io.Pn, g, i, j, k, w);
    if (io.what & PRIM_CFL) smax = fmax(smax, cfl_rate(g, w, ir));
    if (io.what & PRIM_HEALTH) bad |= health_bits(uo, w[4]);
  }
}

// End of a sweep that stored next-stage primitives: the block's CFL rate
// maximum into its slot, the health bits into the control block. Every thread
// of the block calls it. With io.next set the sweep ends a step: the last
// block to publish its maximum advances t by the step just taken, forms the
// next step's size and clears the slots, so that a run of steps needs no
// launch between them. The slots and the block counter are touched by atomics
// only, each block's counter increment after its maximum has returned, so the
// last block sees every maximum without a cache write-back per block.
__device__ __forceinline__ void finish_prims(const StageIO& io, double smax, int bad) {
  if (bad) atomicOr(&io.ctl->status, bad);
  if (!(io.what & PRIM_CFL)) return;
  const unsigned block = blockIdx.y * gridDim.x + blockIdx.x;
  smax = block_max(smax);
  __shared__ int last;
  if (threadIdx.x == 0) {
    unsigned long long old = 0;
    if (smax > 0.0)
      old = atomicMax(reinterpret_cast<unsigned long long*>(io.partial) + (block & (kCflSlots - 1)),
                      (unsigned long long)__double_as_longlong(smax));
    if (io.next) {
      asm volatile("s_waitcnt vmcnt(0)" : "+v"(old) : : "memory");
      last = atomicAdd(&io.ctl->done, 1u) == gridDim.x * gridDim.y - 1;
    }
  }
  if (!io.next) return;
  __syncthreads();
  if (!last) return;
  double m = 0.0;
  for (int i = threadIdx.x; i < kCflSlots; i += blockDim.x)
    m = fmax(m, __longlong_as_double((long long)atomicExch(reinterpret_cast<unsigned long long*>(io.partial) + i, 0ull)));
  m = block_max(m);
  if (threadIdx.x == 0) {
    if (io.t != nullptr) *io.t = *io.t + io.ctl->dt;
    io.ctl->dt = step_size(io.cfl, m, 0.0, io.t, io.t_end);
    atomicExch(&io.ctl->done, 0u);
  }
}

// Value of x in the lane below (lane - 1) across the whole wavefront, by one
// DPP move per 32-bit half (wavefront shift right by one lane, a VALU
// operation instead of an LDS permute); lane 0 receives 0 (by the bound
// control, so that no register has to be cleared beforehand).
__device__ __forceinline__ int dpp_shr1(int x) { return __builtin_amdgcn_update_dpp(x, x, 0x138, 0xf, 0xf, true); }
__device__ __forceinline__ int dpp_shl1(int x) { return __builtin_amdgcn_update_dpp(x, x, 0x130, 0xf, 0xf, true); }
__device__ __forceinline__ double lane_shr1(double x) {
  return __hiloint2double(dpp_shr1(__double2hiint(x)), dpp_shr1(__double2loint(x)));
}

// Value of x in the lane above (lane + 1), wavefront shift left by one lane;
// lane 63 receives 0.
__device__ __forceinline__ double lane_shl1(double x) {
  return __hiloint2double(dpp_shl1(__double2hiint(x)), dpp_shl1(__double2loint(x)));
}

// x sweep: every interior row holds kXCtx context slots followed by its nx+1
// faces, and the slots of all rows are numbered row-major; slot s of a row is
// face f = s - kXCtx, lying between cells f-1 and f. A wavefront takes 64
// consecutive slots, one per lane. The lane of slot s computes the tangential
// velocity derivatives of cell f+1, and face f takes those of cells f-2..f+1
// from itself and the three lanes below it (context slots only supply the
// first faces of their row); the left-face flux of a cell comes from the lane
// below. The first kXCtx+1 slots of a wavefront overlap its predecessor and
// only seed these shuffles. One slot per lane keeps the kernel at three
// wavefronts per SIMD.
constexpr int kXCtx = 3;
constexpr int kXFaces = 64 - (kXCtx + 1);  // faces a wavefront emits

// Interior row `row` (a line of cells along x) of an x sweep in band-major
// order: bands of kXBand consecutive y rows, within a band z outer and y
// inner. The blocks one XCD runs at a time then cover a few planes of a
// narrow band, so the y and z neighbours the tangential stencils read are
// mostly still in that XCD's L2. At 256^3 bands of 32 rows measured 1 %
// faster than 16 or 64 (8: 2 % slower), with the WENO5 x sweep.
constexpr int kXBand = 32;

__device__ __forceinline__ void x_row(const Geom& g, int row, int& j, int& k) {
  const int full = g.n[1] / kXBand;
  const int band_rows = kXBand * g.n[2];
  int band = row / band_rows, h = kXBand;
  if (band >= full) {
    band = full;
    h = g.n[1] - full * kXBand;
  }
  const int r = row - band * band_rows;
  k = r / h;
  j = band * kXBand + (r - k * h);
}

template <int MODE, bool PN, int PHYS>
__device__ __forceinline__ void sweep_x_body_face(const double* __restrict__ P, const StageIO& io, const Geom& g,
                                              int bx) {
  // slot numbering fits in 32 bits (checked when the solver is created)
  const int lane = threadIdx.x & 63;
  const int wave = (bx * kBlock + (int)threadIdx.x) >> 6;
  const int S = g.n[0] + 1 + kXCtx;
  const int total = S * g.n[1] * g.n[2];
  const int first = wave * kXFaces;
  double smax = 0.0;
  int bad = 0;
  if (first < total) {  // uniform per wavefront
    const double dt = mode_rk(MODE) ? stage_dt(io) : 0.0;
    const int gs = first - (kXCtx + 1) + lane;
    const bool inrange = gs >= 0 && gs < total;
    int f = 0, j = 0, k = 0;
    if (inrange) {
      const int row = gs / S;
      f = gs - row * S - kXCtx;
      x_row(g, row, j, k);
    }
    const bool valid = inrange && f >= 0 && gs >= first - 1;  // lanes whose face flux is used
    // Every lane loads a window inside the padded block (context slots and
    // lanes past the end take face 0 of their row) and computes a flux, so the
    // window loads, the derivative loads and the shuffles need no branch and
    // are in flight together.
    const int fl = f < 0 ? 0 : f;
    const long long c0 = cell_at(g, fl - 3, j, k);
    double q[6][5];
#pragma unroll
    for (int m = 0; m < 6; ++m) load_prims(P, g.vs, c0 + m, q[m]);
    double d[4] = {0.0, 0.0, 0.0, 0.0};  // tangential sums and T~ of cell f+1
    const long long c1 = cell_at(g, f + 1, j, k);
    if (with_viscous<PHYS>(g)) {
      double x[4][4];
      tangential_load<0>(g, P, c1, x);
      __builtin_amdgcn_sched_barrier(0);
      tangential_combine3<0>(g, x, d);
    }
    if (with_heat<PHYS>(g)) d[3] = div_nr(P[4 * g.vs + c1], P[c1]);
    // face values of the derivatives from cells f-2..f+1 (lanes - 3 .. lane)
    double tf[3], T[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double t2 = lane_shr1(d[v]);
      const double t1 = lane_shr1(t2);
      const double t0 = lane_shr1(t1);
      if (v < 3) {
        tf[v] = rc4(t0, t1, t2, d[v]);
      } else {
        T[0] = t0;
        T[1] = t1;
        T[2] = t2;
        T[3] = d[v];
      }
    }
    double G[5];
    roe_face_flux<0, PHYS>(g, q, T, tf, G);
    double Gm[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Gm[v] = lane_shr1(G[v]);
    if (valid && gs >= first && f >= 1) {
      double D[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) D[v] = (G[v] - Gm[v]) * g.idx[0];
      const long long ce = cell_at(g, f - 1, j, k);
      EmitIn ein;
      emit_fetch<MODE>(io, g.vs, ce, 0, ein);
      emit_put<MODE, PN>(io, g, ce, 0, D, ein, dt, smax, bad, f - 1, j, k);
    }
  }
  if (PN) finish_prims(io, smax, bad);
}

// The same for the cell-centred schemes: the lane of face f reconstructs at
// both faces of cell f (window cells f-2 .. f+2, one smoothness evaluation
// for the two faces) and takes the left state of face f from the lane below,
// which reconstructed cell f-1.
template <int MODE, bool PN, int SCH, int PHYS, bool IMG>
__device__ __forceinline__ void sweep_x_body_pair(const double* __restrict__ P, const StageIO& io, const Geom& g,
                                                  int bx) {
  const int lane = threadIdx.x & 63;
  const int wave = (bx * kBlock + (int)threadIdx.x) >> 6;
  const int S = g.n[0] + 1 + kXCtx;
  const int total = S * g.n[1] * g.n[2];
  const int first = wave * kXFaces;
  double smax = 0.0;
  int bad = 0;
  if (first < total) {  // uniform per wavefront
    const double dt = mode_rk(MODE) ? stage_dt(io) : 0.0;
    const int gs = first - (kXCtx + 1) + lane;
    const bool inrange = gs >= 0 && gs < total;
    int f = 0, j = 0, k = 0;
    if (inrange) {
      const int row = gs / S;
      f = gs - row * S - kXCtx;
      x_row(g, row, j, k);
    }
    const bool valid = inrange && f >= 0 && gs >= first - 1;  // lanes whose face flux is used
    // every lane loads a window inside the padded block and computes a flux:
    // the context slots before a row's first face reconstruct cell -1 (the
    // left state of face 0 comes from the slot below it), lanes past the end
    // take face 0 of the first row
    const int fl = f < -1 ? -1 : f;
    const long long c0 = cell_at(g, fl - 2, j, k);  // cells f-2 .. f+2
    double q[5][5];
#pragma unroll
    for (int m = 0; m < 5; ++m) load_prims(P, g.vs, c0 + m, q[m]);
    double d[3] = {0.0, 0.0, 0.0};
    if (with_viscous<PHYS>(g)) {
      double x[4][4];
      tangential_load<0>(g, P, cell_at(g, f + 1, j, k), x);
      __builtin_amdgcn_sched_barrier(0);
      tangential_combine3<0>(g, x, d);
    }
    // T~ = p/rho of cells f-2 .. f+1 (heat flux only), from the window
    double T[4] = {0.0, 0.0, 0.0, 0.0};
    if (with_heat<PHYS>(g)) {
#pragma unroll
      for (int m = 0; m < 4; ++m) T[m] = div_nr(q[m][4], q[m][0]);
    }
    // face values of the derivatives from cells f-2..f+1 (lanes - 3 .. lane)
    double tf[3];
#pragma unroll
    for (int v = 0; v < 3; ++v) {
      const double t2 = lane_shr1(d[v]);
      const double t1 = lane_shr1(t2);
      const double t0 = lane_shr1(t1);
      tf[v] = rc4(t0, t1, t2, d[v]);
    }
    double WL[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, WR[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if (with_inviscid<PHYS>(g)) {
      double qr[5];
      recon_pair<SCH>(q, qr, WR);
#pragma unroll
      for (int v = 0; v < 5; ++v) WL[v] = lane_shr1(qr[v]);
      check_face_states(g, valid, WL, WR, q[1], q[2], bad);
    }
    double alpha = 0.0;
    if constexpr (SCH == SCH_W3_NN) alpha = g.nna[c0 + 1];  // alpha of face f (left cell f-1)
    double G[5];
    face_flux_states<0, SCH, PHYS>(g, WL, WR, q, T, tf, alpha, G);
    double Gm[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) Gm[v] = lane_shr1(G[v]);
    if (valid && gs >= first && f >= 1) {
      double D[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) D[v] = (G[v] - Gm[v]) * g.idx[0];
      const long long ce = cell_at(g, f - 1, j, k);
      EmitIn ein;
      emit_fetch<MODE>(io, g.vs, ce, 0, ein);
      emit_put<MODE, PN, IMG>(io, g, ce, 0, D, ein, dt, smax, bad, f - 1, j, k);
    }
  }
  if (PN) finish_prims(io, smax, bad);
  else if (bad && io.ctl) atomicOr(&io.ctl->status, bad);
}

template <int MODE, bool PN = false, int SCH = SCH_JS, int PHYS = PHYS_ANY, bool IMG = false>
__device__ __forceinline__ void sweep_x_body(const double* __restrict__ P, const StageIO& io, const Geom& g,
                                             int bx) {
  if constexpr (SCH == SCH_ROE) sweep_x_body_face<MODE, PN, PHYS>(P, io, g, bx);
  else sweep_x_body_pair<MODE, PN, SCH, PHYS, IMG>(P, io, g, bx);
}

// Blocks are taken in XCD-major order, so that the neighbouring rows and
// planes whose velocities the derivative stencils read are being processed in
// the same XCD and stay in its L2.
// Three wavefronts per SIMD; two for the Roe splitting with run-time flux terms,
// which spills 150 B a lane at three (convective and viscous 128^3, with the
// marches below at one wavefront: two steps 3069 -> 2294 us). With all flux terms
// it spills 20 B at three, which is still faster than two without (2001 against
// 2085 us).
template <int MODE, bool PN, int SCH, int PHYS, bool IMG>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(SCH == SCH_ROE && PHYS == PHYS_ANY ? 2 : 3))) k_sweep_x(const double* __restrict__ P, StageIO io, Geom g) {
  if (step_disabled(io.dtp)) return;
  sweep_x_body<MODE, PN, SCH, PHYS, IMG>(P, io, g, xcd_major_block(blockIdx.x, gridDim.x));
}

// Blocks of an x sweep.
__host__ __device__ __forceinline__ int sweep_x_blocks(const Geom& g) {
  const long long slots = (long long)(g.n[0] + 1 + kXCtx) * g.n[1] * g.n[2];
  const long long waves = (slots + kXFaces - 1) / kXFaces;
  return (int)((waves + 3) / 4);
}

// y / z sweep: one lane per (x, other) column segment of Geom::seg cells
// along the axis; lanes run along x so every load is coalesced. The segment's
// first face is computed only to seed the left flux.
constexpr int kSeg = 32;

// The four values a central difference at cell c takes along the axis of
// stride st, and the difference (times 12 dx).
struct Diff4 {
  double x[4];
  __device__ __forceinline__ void load(const double* q, long long st, unsigned off) {
    x[0] = ld_at(q - 2 * st, off);
    x[1] = ld_at(q - st, off);
    x[2] = ld_at(q + st, off);
    x[3] = ld_at(q + 2 * st, off);
  }
  __device__ __forceinline__ double diff() const { return fma(8.0, x[2] - x[1], x[0] - x[3]); }
};

// y / z sweep body of one lane. Lanes beyond the grid (a partial last block)
// march a valid column too but store nothing, so that every lane reaches the
// block-wide CFL reduction of a sweep that stores next-stage primitives.
// Cell-centred schemes carry the left state of the next face, reconstructed
// with the right state of the current face from the cell between them (one
// smoothness evaluation for the two faces), so their window holds five cells,
// f-1 .. f+3 for face f+1/2, and the segment starts with the reconstruction of
// cell s0-1, for the left state of its first face. The Roe splitting's face
// takes the six cells f-2 .. f+3 (qm is cell f-2).
template <int AX, int MODE, bool PN = false, int SCH = SCH_JS, int PHYS = PHYS_ANY>
__device__ __forceinline__ void sweep_march_body(const double* __restrict__ P, const StageIO& io,
                                                      const Geom& g, int bx, int by) {
  constexpr int OT = AX == 1 ? 2 : 1;  // the other transverse axis
  constexpr int T1 = (AX + 1) % 3, T2 = (AX + 2) % 3;
  const int i = bx * 64 + (int)(threadIdx.x & 63);
  const int sl = g.seg;
  const int nseg = (g.n[AX] + sl - 1) / sl;
  const int col = uniform(by * (kBlock >> 6) + wave_in_block());
  const bool live = col < g.n[OT] * nseg;  // uniform
  const bool in = live && i < g.n[0];
  if (!PN && !live) return;
  double smax = 0.0;
  int bad = 0;
  const int colc = live ? col : 0;
  const int o = uniform(colc / nseg);
  const int s0 = (colc - o * nseg) * sl;
  const int s1 = min(s0 + sl, g.n[AX]);
  const long long st = g.s[AX];
  int q3[3];
  q3[0] = 0;
  q3[OT] = o;
  q3[AX] = s0 - 3;
  const long long c = cell_at(g, q3[0], q3[1], q3[2]);  // uniform: cell s0-3 of the column at x = 0
  const unsigned off = (unsigned)(i < g.n[0] ? i : g.n[0] - 1) * 8u;
  const bool vis = with_viscous<PHYS>(g), heat = with_heat<PHYS>(g);
  const long long sT1 = g.act[T1] ? g.s[T1] : 0, sT2 = g.act[T2] ? g.s[T2] : 0;
  const double w1 = g.act[T1] ? g.idx[T1] * (1.0 / 12.0) : 0.0, w2 = g.act[T2] ? g.idx[T2] * (1.0 / 12.0) : 0.0;
  constexpr bool kRoe = SCH == SCH_ROE;
  double q[5][5];   // window: cells f-1 .. f+3 for face f+1/2
  double qm[5];     // Roe splitting: cell f-2
  double WLc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};  // left state of face f+1/2
  {
    double s[5][5];  // cells s0-3 .. s0+1
#pragma unroll
    for (int m = 0; m < 5; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) s[m][v] = ld_at(P + v * g.vs + c + m * st, off);
#pragma unroll
    for (int v = 0; v < 5; ++v) q[4][v] = ld_at(P + v * g.vs + c + 5 * st, off);
    if constexpr (kRoe) {
#pragma unroll
      for (int v = 0; v < 5; ++v) qm[v] = s[0][v];
    } else if (with_inviscid<PHYS>(g)) {
      double unused[5];
      recon_pair<SCH>(s, WLc, unused);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) q[m][v] = s[m + 1][v];
  }
  const long long c1 = c + st;  // window cell 0: cell f-1 for the first face f = s0-1
  // T~ and the tangential sums (sub_dissipative_q) of cells f-1 .. f+2
  double T[4] = {0.0, 0.0, 0.0, 0.0}, tg[4][3];
  // the entering cell's tangential stencil: u_D and u_T1 along T1, u_D and u_T2 along T2
  Diff4 d[4];
  auto tang_load = [&](long long cc) {
    d[0].load(P + (1 + AX) * g.vs + cc, sT1, off);
    d[1].load(P + (1 + T1) * g.vs + cc, sT1, off);
    d[2].load(P + (1 + AX) * g.vs + cc, sT2, off);
    d[3].load(P + (1 + T2) * g.vs + cc, sT2, off);
  };
  auto tang_sum = [&](double* t) {
    t[0] = d[0].diff() * w1;
    t[1] = d[2].diff() * w2;
    t[2] = fma(d[1].diff(), w1, d[3].diff() * w2);
  };
#pragma unroll
  for (int m = 0; m < 4; ++m) {
#pragma unroll
    for (int v = 0; v < 3; ++v) tg[m][v] = 0.0;
    if (vis) {
      tang_load(c1 + m * st);
      tang_sum(tg[m]);
    }
    if (heat) T[m] = div_nr(q[m][4], q[m][0]);
  }
  double Gm[5];
  const double dt = mode_rk(MODE) ? stage_dt(io) : 0.0;
  for (int f = s0 - 1; f < s1; ++f) {
    // issue the loads of the cell entering the window at the next face, and
    // of its tangential stencil, before this face's arithmetic, so that their
    // latency overlaps it
    // (after the segment's last face the loaded cell is not used; it is the
    // window's last one then, inside the padded block)
    const long long c = c1 + uniform(f - (s0 - 1)) * st;  // window cell 0
    const long long ce = f + 1 < s1 ? c + 5 * st : c + 4 * st;
    double nq[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) nq[v] = ld_at(P + v * g.vs + ce, off);
    // ... and those of the cell update at this face (the segment's first face
    // has none: the row is in the padded block and its values are not used).
    // The Roe splitting has no registers to hold either across its face.
    EmitIn ein;
    if constexpr (!kRoe) {
      if (vis) tang_load(c + 4 * st);
      emit_fetch<MODE>(io, g.vs, c + st, off, ein);  // window cell 1 is cell f
    }
    __builtin_amdgcn_sched_barrier(0);
    double alpha = 0.0;
    if constexpr (SCH == SCH_W3_NN) alpha = ld_at(g.nna + AX * g.vs + c + st, off);  // face f+1/2, left cell f
    double WR[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, qr[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    if constexpr (!kRoe) {
      if (with_inviscid<PHYS>(g)) {
        recon_pair<SCH>(q, qr, WR);  // cell f+1: left state of face f+3/2, right state of f+1/2
        check_face_states(g, true, WLc, WR, q[1], q[2], bad);
      }
    }
    double tf[3] = {0.0, 0.0, 0.0};
    if (vis) {
#pragma unroll
      for (int v = 0; v < 3; ++v) tf[v] = rc4(tg[0][v], tg[1][v], tg[2][v], tg[3][v]);
    }
    double G[5];
    if constexpr (kRoe) {
      double q6[6][5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        q6[0][v] = qm[v];
#pragma unroll
        for (int m = 0; m < 5; ++m) q6[1 + m][v] = q[m][v];
      }
      roe_face_flux<AX, PHYS>(g, q6, T, tf, G);
    } else {
      face_flux_states<AX, SCH, PHYS>(g, WLc, WR, q, T, tf, alpha, G);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) pin(G[v]);
    if (f >= s0 && in) {
      double D[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) D[v] = (G[v] - Gm[v]) * g.idx[AX];
      if constexpr (kRoe) emit_fetch<MODE>(io, g.vs, c + st, off, ein);
      emit_put<MODE, PN>(io, g, c + st, off, D, ein, dt, smax, bad, i, AX == 1 ? f : o, AX == 1 ? o : f);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      Gm[v] = G[v];
      WLc[v] = qr[v];
    }
    if constexpr (kRoe)
      if (vis) tang_load(c + 4 * st);
    // shift the window by one cell along the axis
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      T[m] = T[m + 1];
#pragma unroll
      for (int v = 0; v < 3; ++v) tg[m][v] = tg[m + 1][v];
    }
    if (heat) T[3] = div_nr(q[4][4], q[4][0]);  // cell f+3
    if (vis) tang_sum(tg[3]);
    if constexpr (kRoe) {
#pragma unroll
      for (int v = 0; v < 5; ++v) qm[v] = q[0][v];
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) q[m][v] = q[m + 1][v];
#pragma unroll
    for (int v = 0; v < 5; ++v) q[4][v] = nq[v];
  }
  if (PN) finish_prims(io, smax, bad);
  else if (bad && io.ctl) atomicOr(&io.ctl->status, bad);
}

// Two wavefronts per SIMD; one for the Roe splitting with run-time flux terms,
// which spills 68 to 148 B a lane at two.
template <int AX, int MODE, bool PN, int SCH, int PHYS>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(SCH == SCH_ROE && PHYS == PHYS_ANY ? 1 : 2)))
k_sweep_march(const double* __restrict__ P, StageIO io, Geom g) {
  if (step_disabled(io.dtp)) return;
  // XCD-major block order (see k_sweep_x): consecutive column groups, hence
  // neighbouring planes of the transverse derivatives, share an XCD
  const int logical = xcd_major_block(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int by = logical / gridDim.x;
  sweep_march_body<AX, MODE, PN, SCH, PHYS>(P, io, g, logical - by * gridDim.x, by);
}

// Marching sweep along AX that also forms the x faces of the rows it passes
// (cell-centred schemes): the stage's last sweep wherever x and another axis
// are active. A wavefront holds 64 consecutive x of a row; while it marches,
// the x face of lane l (between lanes l-1 and l) takes its stencil from the
// window rows of the neighbouring lanes (DPP shifts), so one pass over P
// serves both axes and the x divergence never goes through memory. The x part
// treats the row at the window's centre (f+1 at face f+1/2), whose
// derivatives along AX are in the window already; a row's x divergence is
// carried to the next face with the flux of the face between them. The first
// three lanes and the last three of a wavefront only supply stencils: it
// emits kMxNew cells. Rows of different transverse index o follow each other
// in the lanes (slots -3 .. n+2 of every row) unless strips of kMxNew cells of
// one row take fewer wavefronts (Geom::xs).
// Bounds: FP64 VALU and the latency of the march's loads at two wavefronts
// per SIMD; without this fusion the x sweep re-read P, R and both stage
// states at the rate of a plain copy (4.9 TB/s at 256^3) while the marches,
// at 2.6 TB/s, waited on latency.
constexpr int kMxCtx = 3, kMxNew = 64 - 2 * kMxCtx;

template <int AX, int MODE, bool PN, int SCH, int PHYS, bool IMG = false, bool BEFORE_FLUX = false>
__device__ __forceinline__ void sweep_mx_body(const double* __restrict__ P, const StageIO& io, const Geom& g,
                                              int block) {
  constexpr int OT = 3 - AX;  // the transverse axis of the rows
  constexpr int T1 = (AX + 1) % 3;
  const int lane = threadIdx.x & 63;
  const int sl = g.segx;
  const int nseg = (g.n[AX] + sl - 1) / sl;
  const int item = uniform(block * (kBlock >> 6) + wave_in_block());
  const int seg = uniform(item / g.xg);
  const int gw = item - seg * g.xg;
  const bool live = seg < nseg;  // uniform
  if (!PN && !live) return;
  double smax = 0.0;
  int bad = 0;
  if (live) {
    int o, x, ob;
    bool inrow;
    if (g.xs) {
      const int k = (g.n[0] + kMxNew - 1) / kMxNew;
      ob = o = uniform(gw / k);
      x = (gw - o * k) * kMxNew + lane - kMxCtx;
      inrow = x < g.n[0];
    } else {
      const int S = g.n[0] + 2 * kMxCtx;
      const int slot = gw * kMxNew + lane - kMxCtx;
      const int sc = min(max(slot, 0), S * g.n[OT] - 1);
      o = sc / S;
      x = sc - o * S - kMxCtx;
      inrow = slot == sc && x >= 0 && x < g.n[0];
      ob = uniform(o);
    }
    const bool emit = inrow && lane >= kMxCtx && lane < 64 - kMxCtx;
    const bool xface = lane >= kMxCtx && lane <= 64 - kMxCtx && x >= 0 && x <= g.n[0];  // lane's x face is used
    const unsigned off = (unsigned)((o - ob) * g.s[OT] + min(max(x, -kMxCtx), g.n[0] + kMxCtx - 1) + g.h[0]) * 8u;
    const int s0 = seg * sl;
    const int s1 = min(s0 + sl, g.n[AX]);
    const long long st = g.s[AX], sO = g.act[OT] ? g.s[OT] : 0;
    const double wA = g.idx[AX] * (1.0 / 12.0), wO = g.act[OT] ? g.idx[OT] * (1.0 / 12.0) : 0.0,
                 w0 = g.idx[0] * (1.0 / 12.0);
    const bool vis = with_viscous<PHYS>(g), heat = with_heat<PHYS>(g);
    // uniform base of row s0-2 (window cell 0 of the first face) at padded x = 0
    const long long c1 = (long long)(ob + g.h[OT]) * g.s[OT] + (long long)(s0 - 2 + g.h[AX]) * st;
    double q[5][5];  // window: rows f-1 .. f+3 for face f+1/2
    double WLc[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    {
      double s[5][5];  // rows s0-3 .. s0+1
#pragma unroll
      for (int m = 0; m < 5; ++m)
#pragma unroll
        for (int v = 0; v < 5; ++v) s[m][v] = ld_at(P + v * g.vs + c1 + (m - 1) * st, off);
#pragma unroll
      for (int v = 0; v < 5; ++v) q[4][v] = ld_at(P + v * g.vs + c1 + 4 * st, off);
      if (with_inviscid<PHYS>(g)) {
        double unused[5];
        recon_pair<SCH>(s, WLc, unused);
      }
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int v = 0; v < 5; ++v) q[m][v] = s[m + 1][v];
    }
    // Rows f-1 .. f+2: T~ and the tangential derivatives of the AX faces -
    // along OT and x of u_AX, and du_OT/dOT + du_x/dx; du_OT/dOT and du_x/dOT
    // on their own for the x part of the rows from the centre on.
    double T[4] = {0.0, 0.0, 0.0, 0.0}, tO[4], tX[4], tS[4], rO[4], rX[4];
    Diff4 d[3];
    auto o_load = [&](long long cc) {
      d[0].load(P + (1 + AX) * g.vs + cc, sO, off);
      d[1].load(P + (1 + OT) * g.vs + cc, sO, off);
      d[2].load(P + g.vs + cc, sO, off);
    };
    auto x_diff = [&](double u) {
      const double b = lane_shr1(u), e = lane_shl1(u);
      return fma(8.0, e - b, lane_shr1(b) - lane_shl1(e)) * w0;
    };
    auto tang = [&](int m, const double* row) {
      tO[m] = d[0].diff() * wO;
      tX[m] = x_diff(row[1 + AX]);
      rO[m] = d[1].diff() * wO;
      rX[m] = d[2].diff() * wO;
      tS[m] = rO[m] + x_diff(row[1]);
    };
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      tO[m] = tX[m] = tS[m] = rO[m] = rX[m] = 0.0;
      if (vis) {
        o_load(c1 + m * st);
        tang(m, q[m]);
      }
      if (heat) T[m] = div_nr(q[m][4], q[m][0]);
    }
    double Gm[5], Dx[5];  // flux of face f-1/2 and x divergence of row f
    const double dt = mode_rk(MODE) ? stage_dt(io) : 0.0;
    for (int f = s0 - 1; f < s1; ++f) {
      const long long c = c1 + uniform(f - (s0 - 1)) * st;  // row f-1
      // the entering row (after the segment's last face a row already held,
      // inside the padded block)
      const long long ce = f + 1 < s1 ? c + 5 * st : c + 4 * st;
      double nq[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) nq[v] = ld_at(P + v * g.vs + ce, off);
      if (vis) o_load(c + 4 * st);
      // the update's loads before the face's arithmetic, as the stencils', where
      // they are ten values (2D 1024^2: 4 steps 818 -> 805 us). The fifteen of
      // MODE_ACC_RK are loaded where they are used: held across the face they
      // cost the third Euler wavefront and 24 B of spills with viscous fluxes,
      // HIT 256^3 (2 steps) 11386 against 10618 us, TGV 64^3 182 against 178 us.
      // BEFORE_FLUX issues them between the reconstruction and the flux, which
      // suits the viscous single-grid sweep without images (10616 and 175 us), not
      // the one with them (rollout at 40^3 8.21 against 8.03 ms), nor the Euler
      // one (two wavefronts instead of three)
      EmitIn ein;  // row f (the segment's first face uses none: row -1 may be in the halo)
      if constexpr (MODE != MODE_ACC_RK) emit_fetch<MODE>(io, g.vs, c + st, off, ein);
      __builtin_amdgcn_sched_barrier(0);
      double G[5], nWL[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
      {
        double alpha = 0.0;
        if constexpr (SCH == SCH_W3_NN) alpha = ld_at(g.nna + AX * g.vs + c + st, off);  // face f+1/2, left cell f
        double WR[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        if (with_inviscid<PHYS>(g)) {
          recon_pair<SCH>(q, nWL, WR);  // row f+1: left state of face f+3/2, right state of f+1/2
          check_face_states(g, emit, WLc, WR, q[1], q[2], bad);
        }
        double tf[3] = {0.0, 0.0, 0.0};
        if (vis) {
          const double a = rc4(tO[0], tO[1], tO[2], tO[3]), b = rc4(tX[0], tX[1], tX[2], tX[3]);
          tf[0] = T1 == 0 ? b : a;
          tf[1] = T1 == 0 ? a : b;
          tf[2] = rc4(tS[0], tS[1], tS[2], tS[3]);
        }
        if constexpr (MODE == MODE_ACC_RK && BEFORE_FLUX) {
          emit_fetch<MODE>(io, g.vs, c + st, off, ein);
          __builtin_amdgcn_sched_barrier(0);
        }
        face_flux_states<AX, SCH, PHYS>(g, WLc, WR, q, T, tf, alpha, G);
#pragma unroll
        for (int v = 0; v < 5; ++v) pin(G[v]);
      }
      // row f is complete with this face
      if (f >= s0 && emit) {
        if constexpr (MODE == MODE_ACC_RK && !BEFORE_FLUX) emit_fetch<MODE>(io, g.vs, c + st, off, ein);
        double D[5];
#pragma unroll
        for (int v = 0; v < 5; ++v) D[v] = fma(G[v] - Gm[v], g.idx[AX], Dx[v]);
        emit_put<MODE, PN, IMG>(io, g, c + st, off, D, ein, dt, smax, bad, x, AX == 1 ? f : o, AX == 1 ? o : f);
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        Gm[v] = G[v];
        WLc[v] = nWL[v];
      }
      // x faces of row f+1 (not after the segment's last face)
      if (f + 1 < s1) {
        double WL[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, WR[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        double xq[4][5];  // cells x-2 .. x+1 of the lane's left face
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          xq[2][v] = q[2][v];
          xq[1][v] = lane_shr1(q[2][v]);
          xq[0][v] = lane_shr1(xq[1][v]);
          xq[3][v] = lane_shl1(q[2][v]);
          if (with_inviscid<PHYS>(g)) {
            double r;
            const double e = lane_shl1(xq[3][v]);
            if constexpr (sch_weno3(SCH)) weno3_pair(xq[1][v], xq[2][v], xq[3][v], r, WR[v]);
            else if constexpr (SCH == SCH_Z) weno5z_pair(xq[0][v], xq[1][v], xq[2][v], xq[3][v], e, r, WR[v]);
            else weno5_pair(xq[0][v], xq[1][v], xq[2][v], xq[3][v], e, r, WR[v]);
            WL[v] = lane_shr1(r);
            pin(WL[v]);
            pin(WR[v]);
          }
        }
        if (with_inviscid<PHYS>(g)) check_face_states(g, xface, WL, WR, xq[1], xq[2], bad);
        double tf[3] = {0.0, 0.0, 0.0}, xT[4] = {0.0, 0.0, 0.0, 0.0};
        if (vis) {
          // du_x/dy, du_x/dz, du_y/dy + du_z/dz at the row; their face values
          auto a_diff = [&](int v) { return fma(8.0, q[3][v] - q[1][v], q[0][v] - q[4][v]) * wA; };
          const double xA = a_diff(1), t[3] = {AX == 1 ? xA : rX[2], AX == 1 ? rX[2] : xA, a_diff(1 + AX) + rO[2]};
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const double b = lane_shr1(t[k]);
            tf[k] = rc4(lane_shr1(b), b, t[k], lane_shl1(t[k]));
          }
        }
        if (heat) {
          xT[2] = T[2];
          xT[1] = lane_shr1(T[2]);
          xT[0] = lane_shr1(xT[1]);
          xT[3] = lane_shl1(T[2]);
        }
        double alpha = 0.0, Gx[5];
        if constexpr (SCH == SCH_W3_NN) alpha = ld_at(g.nna + c + 2 * st - 1, off);  // face x, left cell x-1
        face_flux_states<0, SCH, PHYS>(g, WL, WR, xq, xT, tf, alpha, Gx);
#pragma unroll
        for (int v = 0; v < 5; ++v) Dx[v] = (lane_shl1(Gx[v]) - Gx[v]) * g.idx[0];
      }
      // shift the window by one row
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        T[m] = T[m + 1];
        tO[m] = tO[m + 1];
        tX[m] = tX[m + 1];
        tS[m] = tS[m + 1];
        rO[m] = rO[m + 1];
        rX[m] = rX[m + 1];
      }
      if (heat) T[3] = div_nr(q[4][4], q[4][0]);
      if (vis) tang(3, q[4]);
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int v = 0; v < 5; ++v) q[m][v] = q[m + 1][v];
#pragma unroll
      for (int v = 0; v < 5; ++v) q[4][v] = nq[v];
    }
  }
  if (PN) finish_prims(io, smax, bad);
  else if (bad && io.ctl) atomicOr(&io.ctl->status, bad);
}

template <int AX, int MODE, bool PN, int SCH, int PHYS, bool IMG>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
k_sweep_mx(const double* __restrict__ P, StageIO io, Geom g) {
  if (step_disabled(io.dtp)) return;
  sweep_mx_body<AX, MODE, PN, SCH, PHYS, IMG, PHYS == PHYS_NS && !IMG>(P, io, g, xcd_major_block(blockIdx.x, gridDim.x));
}

// Blocks of a march with x faces along AX.
__host__ __device__ __forceinline__ int sweep_mx_blocks(const Geom& g, int ax) {
  const long long items = (long long)g.xg * ((g.n[ax] + g.segx - 1) / g.segx);
  return (int)((items + 3) / 4);
}

// Launch shape of a marching sweep along AX (x blocks, y blocks).
template <int AX>
__host__ __device__ __forceinline__ void sweep_march_blocks(const Geom& g, int& gx, int& gy) {
  constexpr int OT = AX == 1 ? 2 : 1;
  const int nseg = (g.n[AX] + g.seg - 1) / g.seg;
  gx = (g.n[0] + 63) / 64;
  gy = (int)(((long long)g.n[OT] * nseg + 3) / 4);
}

// Order of the sweeps where a stage has one per active axis (the Roe splitting,
// grids with one active axis or without x): y, z, x. The last stores the new
// state and the next primitives.
constexpr int kSweepAxes[3] = {1, 2, 0};

// Zero a buffer (graph-safe replacement for a memset node), 16 bytes a store
// where the buffer is aligned to them. Launched with at most kZeroBlocks
// blocks: bound by the writes then; with a block per 256 values the dispatch
// of the blocks ruled (the 128^3 reverse pass 3.50 -> 3.47 ms).
constexpr int kZeroBlocks = 2048;
__global__ void __launch_bounds__(kBlock) k_zero(double* x, long long n) {
  const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x, step = (long long)gridDim.x * blockDim.x;
  if (((size_t)x & 15) == 0) {
    double2* y = reinterpret_cast<double2*>(x);
    const long long n2 = n >> 1;
    for (long long e = t; e < n2; e += step) y[e] = make_double2(0.0, 0.0);
    if ((n & 1) && t == 0) x[n - 1] = 0.0;
  } else {
    for (long long e = t; e < n; e += step) x[e] = 0.0;
  }
}

}  // namespace cfd
