// How the marches of a grid are cut: lanes, segment lengths and whether the last
// sweep stores halo images. Host code.
#pragma once
#include <algorithm>
#include <cmath>
#include <vector>

#include "kernels_fwd.hpp"

namespace cfd {

// The Roe splitting projects face by face; the others reconstruct per cell.
inline bool face_by_face(const Geom& g) { return g.roe; }

// Whether the last sweep of a stage stores the halo images of the primitives it
// writes (cell-centred schemes with an x axis, up to kImagesMaxCells padded
// cells; else a pass of its own copies them). The pass is a launch of 4 to 5 us per
// stage, the images cost the sweep registers and scattered stores: without ->
// with them the implosion at 128^2 500 -> 412 us (20 steps), KH 331^2 583 ->
// 528 us, a TGV step at 32^3 95 -> 87 us, but at 64^3 171 -> 180 us, KH 600^2
// 556 -> 579 us and HIT 256^3 11.2 -> 11.6 ms.
constexpr long long kImagesMaxCells = 1LL << 18;
inline bool stores_images(const Geom& g) { return !face_by_face(g) && g.act[0] && g.vs <= kImagesMaxCells; }

// Lanes of a march with x faces: wavefronts per march segment, either strips
// of kMxNew cells of one row each, or all rows' slots one after another (rows
// shorter than a strip share wavefronts), whichever takes fewer; strips too
// where the byte offsets between the rows of one wavefront would not fit in
// 32 bits.
inline void choose_mx_lanes(Geom& g) {
  const int ot = g.act[1] ? 2 : 1;
  const long long S = g.n[0] + 2 * kMxCtx, rows = g.n[ot];
  const long long strips = (g.n[0] + kMxNew - 1) / kMxNew * rows, flat = (S * rows + kMxNew - 1) / kMxNew;
  const double span = 8.0 * ((64.0 / S + 2.0) * (double)g.s[ot] + g.N[0]);
  g.xs = strips <= flat || span >= 4.0e9;
  g.xg = (int)(g.xs ? strips : flat);
}

// Time of `waves` wavefronts over the chip's 1024 SIMDs, `res` of them resident
// on one at a time, in units of one wavefront's pure issue time: measured, a
// SIMD with w wavefronts of a march takes w + 0.6 (one alone 1.6: nothing
// hides its latencies), so that 331^2 marches with x faces in segments of 2,
// 3, 4 and 8 rows (one wavefront per SIMD or less) run 11, 14, 17 and 28 us.
inline double waves_time(double waves, int res) {
  const double w = waves / 1024.0, full = std::floor(w / res);
  if (full >= 3) return w * (res + 0.6) / res + 0.3;
  const double rem = std::ceil(w - full * res);
  return full * (res + 0.6) + (rem > 0 ? rem + 0.6 : 0.0);
}

// Segment length along an axis of n cells that makes `groups(1 segment)`
// wavefronts finish first: long segments seldom recompute their seed (worth
// `seed` cells), short ones give the SIMDs more wavefronts. `face` is the work
// per cell next to the first face's, `res` the resident wavefronts per SIMD.
inline int best_segment(int n, double groups, double face, double seed, int res) {
  int best = 1;
  double cost = 0.0;
  for (int s = 1; s <= std::min(n, 256); ++s) {
    const double c = (face * s + 1.0 + seed) * waves_time(groups * ((n + s - 1) / s), res);
    if (s == 1 || c < cost) {
      cost = c;
      best = s;
    }
  }
  return best;
}

// Wavefronts per SIMD that the registers of a grid's marches leave room for
// (tests/test_segments_cpu.py holds them against the built kernels).
// The march of one axis: the z march of a 3D Euler step keeps to 128 registers,
// the others to 256; the Roe splitting with run-time flux terms takes more. On
// Euler grids without x, where the marches run with run-time flux terms at two,
// the lengths for four are the faster ones (300 x 300 in y and z, 4 steps: 2859
// against 3172 us).
inline int march_waves(const Geom& g) {
  const bool euler = g.inviscid && !g.viscous && !g.heat, ns = g.inviscid && g.viscous && g.heat;
  if (g.roe) return euler || ns ? 2 : 1;
  return euler ? 4 : 2;
}
// The march with x faces: three for the Euler equations, but two where it holds
// both states across its face and stores images (2D grids; WENO3-JS with HLLC
// stays within 168 registers).
inline int mx_waves(const Geom& g, bool images) {
  if (!(g.inviscid && !g.viscous && !g.heat)) return 2;
  const bool flat = !(g.act[0] && g.act[1] && g.act[2]);
  return flat && images && !(g.weno3 && !g.rusanov && !g.nn) ? 2 : 3;
}

// March segments of a single-grid solver. Against the fixed rule of 8 to 128
// cells by powers of two (at least 1024 wavefronts): the implosion at 128^2
// 1208 -> 590 us per 20 steps, KH 331^2 1079 -> 571 us and 1024^2 1130 -> 814 us
// per 10 and 4 steps, a TGV step at 32^3 210 -> 97 us and at 128^3 1018 -> 822 us,
// HIT 256^3 12.04 -> 11.02 ms per two steps. The serving batch chooses its
// own (batch_segment): it fills the chip with many grids.
inline void choose_segment(Geom& g, bool images) {
  // a cell-centred scheme marches y alone only on grids without x: there, and for
  // the Roe splitting, one length serves both axes
  const bool y_alone = face_by_face(g) || !g.act[0];
  int seg = 0;
  for (int ax = 1; ax < 3; ++ax) {
    if (!g.act[ax] || (ax == 1 && !y_alone)) continue;
    const double groups = (double)((g.n[0] + 63) / 64) * g.n[3 - ax];
    const int s = best_segment(g.n[ax], groups, 1.0, g.roe ? 4.0 : 3.0, march_waves(g));
    seg = seg ? std::min(seg, s) : s;
  }
  g.seg = seg ? seg : 1;
  const int mx = g.act[1] ? 1 : 2;
  g.segx = best_segment(g.n[mx], (double)g.xg, 2.0, 1.5, mx_waves(g, images));
}

constexpr unsigned kPersistentBlocks = 2048;  // workgroups of a batch phase: 8 per CU on 256 CUs

// March segment lengths of a serving batch's resident grids, one for the z
// marches and one for the marches with x faces: the longest power of two from 64
// down with which the phase still holds kPersistentBlocks blocks over all of them
// (long segments seldom recompute their seeds), and 2 where none does. Each face
// flux is computed the same way with any segment length, so the results do
// not depend on it.
inline void batch_segment(std::vector<Geom>& grids, int& seg, int& segx) {
  bool march_ok = false, mx_ok = false;
  seg = segx = 2;
  for (int len = 64; len >= 2 && !(march_ok && mx_ok); len /= 2) {
    long long march = 0, mx = 0;
    for (Geom& g : grids) {
      g.seg = g.segx = len;
      int gx = 0, gy = 0;
      if (g.act[2]) sweep_march_blocks<2>(g, gx, gy);
      march += (long long)gx * gy;
      if (g.act[0] && (g.act[1] || g.act[2])) mx += sweep_mx_blocks(g, g.act[1] ? 1 : 2);
    }
    if (!march_ok && march >= kPersistentBlocks) {
      march_ok = true;
      seg = len;
    }
    if (!mx_ok && mx >= kPersistentBlocks) {
      mx_ok = true;
      segx = len;
    }
  }
}

}  // namespace cfd
