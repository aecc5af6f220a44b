// Walks the matrix-core stencil's pair cursor over every position of a lattice, as the waves of its blocks
// do (from the start of each wave's range), and compares what each site takes as its neighbours (the x and
// y inputs kept from pair to pair included) with the neighbours found from coordinates.  Arguments: X Y Z T by bz bt nsub (by = 0: the default brick).
#include <cstdio>
#include <cstdlib>
#include <cstring>
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
      if (s0 % 2 || cnt % 2) return std::printf("odd range at %d\n", s0), 1;
      for (int par = 0; par < 2; ++par) {
        PairCursor cu;
        cu.init(g, s0 / 2);
        int P[2] = {-1, -1}, Q[2] = {-1, -1};  // inputs at the pair's x_h and: behind it (P), ahead of it (Q)
        bool fresh = true;
        for (int k = 0; k < cnt / 2; ++k) {
          if (k) fresh = cu.next(g);
          PairCursor at;  // carries equal divisions
          at.init(g, s0 / 2 + k);
          if (std::memcmp(&at, &cu, sizeof(at))) return std::printf("pair %d of %d\n", s0 / 2 + k, g.hv / 2), 1;
          const int i = cu.X0 + cu.rx;
          auto wrap = [&](int j) { return j < 0 ? j + g.Xh : j >= g.Xh ? j - g.Xh : j; };
          int nb[2][5], up[2], row[2], site[2];
          for (int r = 0; r < 2; ++r) site[r] = pair_site(g, cu, par, r, nb[r], &up[r], &row[r]);
          P[1] = fresh ? row[0] + wrap(i - 1) : P[0];
          P[0] = row[0] + i;
          Q[0] = fresh ? row[1] + i : Q[1];
          Q[1] = row[1] + wrap(i + 1);
          for (int r = 0; r < 2; ++r) {
            int c[4];
            cb_coords(g, site[r], par, c);
            const int own_up = r ? P[0] : Q[0];  // the y neighbour in the pair's other row
            const int got[8] = {r ? Q[1] : P[0], r ? Q[0] : P[1], up[r] ? nb[r][0] : own_up,
                                up[r] ? own_up : nb[r][0], nb[r][1], nb[r][2], nb[r][3], nb[r][4]};
            for (int d = 0; d < 8; ++d)
              if (got[d] != neighbor(g, c, d / 2, d % 2 ? -1 : 1)) return std::printf("neighbour %d of %d\n", d, site[r]), 1;
            seen[site[r]] += par;
          }
        }
      }
    }
  for (int s = 0; s < g.hv; ++s)
    if (seen[s] != 1) return std::printf("site %d seen %d times\n", s, seen[s]), 1;
  std::printf("ok\n");
  return 0;
}
