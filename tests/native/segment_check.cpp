// Prints how the marches of the grids given on the command line are cut
// (segments.hpp; host code, no GPU). Arguments: "batch" or "solo", then per grid
// nx ny nz scheme physics, with scheme one of js z w3 jsrus w3rus nn roe and
// physics one of e (convective), ns (all terms), v (convective and viscous).
// solo: a line per grid "seg segx march_waves mx_waves"; batch: one line "seg segx".
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../paper_2203_13760_amd/csrc/segments.hpp"

using namespace cfd;

int main(int argc, char** argv) {
  std::vector<Geom> grids;
  for (int a = 2; a + 4 < argc; a += 5) {
    Geom g;
    std::memset(&g, 0, sizeof(g));
    for (int d = 0; d < 3; ++d) {
      g.n[d] = std::atoi(argv[a + d]);
      g.act[d] = g.n[d] > 1;
      g.h[d] = g.act[d] ? 3 : 0;
      g.N[d] = g.n[d] + 2 * g.h[d];
    }
    g.s[0] = 1;
    g.s[1] = g.N[0];
    g.s[2] = (long long)g.N[0] * g.N[1];
    g.vs = g.s[2] * g.N[2];
    const std::string scheme = argv[a + 3], phys = argv[a + 4];
    g.inviscid = 1;
    g.viscous = phys != "e";
    g.heat = phys == "ns";
    g.wenoz = scheme == "z";
    g.roe = scheme == "roe";
    g.nn = scheme == "nn";
    g.weno3 = scheme == "w3" || scheme == "w3rus" || g.nn;
    g.rusanov = scheme == "jsrus" || scheme == "w3rus";
    choose_mx_lanes(g);
    grids.push_back(g);
  }
  if (std::strcmp(argv[1], "batch") == 0) {
    int seg, segx;
    batch_segment(grids, seg, segx);
    std::printf("%d %d\n", seg, segx);
    return 0;
  }
  for (Geom& g : grids) {
    choose_segment(g, stores_images(g));
    std::printf("%d %d %d %d\n", g.seg, g.segx, march_waves(g), mx_waves(g, stores_images(g)));
  }
  return 0;
}
