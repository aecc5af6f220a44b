// Walks the matrix-core stencil's sweep cursor over every position of a lattice, as the waves of its
// blocks do (from the start of each wave's range), and compares site and neighbours with the brick order
// and the neighbours found from coordinates.  Arguments: X Y Z T by bz bt nsub (by = 0: the default brick).
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1405_4524_amd/csrc/runtime.h"

using namespace a2a;

int main(int argc, char** argv) {
  if (argc != 9) return 2;
  a2a_geom gm{};
  for (int i = 0; i < 4; ++i) gm.dims[i] = std::atoi(argv[1 + i]);
  gm.t_bc = -1;
  Geo g{};
  if (geom_to_geo(&gm, &g)) return 3;
  if (std::atoi(argv[5])) {
    g.by = (unsigned char)std::atoi(argv[5]);
    g.bz = (unsigned char)std::atoi(argv[6]);
    g.bt = (unsigned char)std::atoi(argv[7]);
  }
  const int nsub = std::atoi(argv[8]), spw = 64 / nsub, nblk = (g.hv + 255) / 256;
  std::vector<int> seen(g.hv, 0);
  for (int b = 0; b < nblk * nsub; ++b)
    for (int w = 0; w < 4; ++w) {
      const int s0 = b / nsub * 256 + w * 64 + b % nsub * spw;
      const int cnt = s0 < g.hv ? (g.hv - s0 < spw ? g.hv - s0 : spw) : 0;
      if (cnt <= 0) continue;
      SweepCursor cu;
      cu.init(g, s0);
      for (int k = 0; k < cnt; ++k) {
        if (k) cu.next(g);
        for (int par = 0; par < 2; ++par) {
          int nb[8], c[4];
          const int site = cursor_neighbours(g, cu, par, nb);
          if (site != brick_site<true>(g, s0 + k)) return std::printf("site %d of %d\n", s0 + k, g.hv), 1;
          cb_coords(g, site, par, c);
          for (int d = 0; d < 8; ++d)
            if (nb[d] != neighbor(g, c, d / 2, d % 2 ? -1 : 1)) return std::printf("neighbour %d of %d\n", d, site), 1;
          if (par) seen[site]++;
        }
      }
    }
  for (int s = 0; s < g.hv; ++s)
    if (seen[s] != 1) return std::printf("site %d seen %d times\n", s, seen[s]), 1;
  std::printf("ok\n");
  return 0;
}
