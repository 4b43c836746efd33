// Host check of the box passes' shapes: for extents of every remainder, the
// box fits the buffers that the kernels hold it in (sized for 16 x 8 x 4 cells:
// its frames of 2 and of 1 cells, half of the latter, and the coarse cells of
// the trilinear correction), has even extents and at most 512 cells, and the
// boxes counted for a level cover it, each found by its index.  Exits with the number of mismatches.
#include <algorithm>
#include <cstdio>

#include "fld.h"
#include "fld_engine.h"

using namespace fld;

int main() {
  const int ext[] = {4, 6, 8, 10, 12, 14, 16, 18, 20, 24, 30, 32, 34, 64, 66, 130, 258, 1024, 4096};
  int bad = 0, cases = 0;
  fld_params p;
  fld_default_params(&p, 3e10, 1.0);
  p.fused_tile_z = 0;
  for (int nx : ext)
    for (int ny : ext)
      for (int nz : ext) {
        const long long cells = (long long)nx * ny * nz;
        if (cells >= 1LL << 31) continue;
        int tx, ty, tz;
        box_shape(nx, ny, nz, tx, ty, tz);
        auto up = [](int a, int b) { return (a + b - 1) / b; };
        bool ok = tx % 2 == 0 && ty % 2 == 0 && tz % 2 == 0 && tx * ty * tz <= 512 &&
                  tx <= std::min(nx, 16) && ty <= ny && tz <= nz && std::max(ty, tz) <= 16 &&
                  (tx + 4) * (ty + 4) * (tz + 4) <= 20 * 12 * 8 &&
                  (tx + 2) / 2 * (ty + 2) * (tz + 2) <= 9 * 10 * 6 &&
                  (tx / 2 + 4) * (ty / 2 + 4) * (tz / 2 + 4) <= 12 * 8 * 6;
        // the index of a box to its place by multiplication, wherever the
        // record says that this is exact
        BoxRec r;
        const bool exact = box_rec(nx, ny, nz, r);
        const long long n = (long long)up(nx, tx) * up(ny, ty) * up(nz, tz);
        ok = ok && (int)r.nbx == up(nx, tx) && (int)r.nby == up(ny, ty);
        auto div = [](unsigned u, unsigned m) {
          return m ? (unsigned)(((unsigned long long)u * m) >> 32) : u;
        };
        ok = ok && r.ext == (unsigned)(tx | ty << 8 | tz << 16) && (exact || cells >= 3LL << 19);
        for (long long u = 0; exact && u < n; u += 1 + n / 5000) {
          for (long long v : {u, std::min(n, (u / r.nbx + 1) * r.nbx) - 1}) {
            const unsigned row = div((unsigned)v, r.mx);
            ok = ok && row == v / r.nbx && div(row, r.my) == row / r.nby;
          }
        }
        if (cells < (3LL << 19)) {
          fld_grid g{};
          g.nx = nx;
          g.ny = ny;
          g.nz = nz;
          g.dx = g.dy = g.dz = 1.0;
          const Hier h = make_hier(g, p);
          ok = ok && h.box[0] && h.ftiles[0] == up(nx, tx) * up(ny, ty) * up(nz, tz);
        }
        if (!ok) printf("%d x %d x %d: box %d x %d x %d MISMATCH\n", nx, ny, nz, tx, ty, tz);
        bad += !ok;
        ++cases;
      }
  printf("%d cases, %d mismatches\n", cases, bad);
  return bad > 255 ? 255 : bad;
}
