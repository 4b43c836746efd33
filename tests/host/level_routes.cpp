// Host check of the route that each level of a hierarchy takes: box by box or
// marching tiles (the line at 1.5 x 2^20 cells, fused_levels, fused_tile_z) and
// their counts, remainders included, the first level of the tail in the fused
// and in the per-sweep cycles, and whether the finest SpMV runs on the fused
// tiles.  Exits with the number of mismatches.
#include <cstdio>
#include <functional>
#include <vector>

#include "fld.h"
#include "fld_engine.h"

using namespace fld;

int main() {
  struct Case {
    int nx, ny, nz;
    std::function<void(fld_params &)> set;
    int levels, tail, tail_sweeps, nbox;  // levels 0 .. nbox - 1 march, box from there
    std::vector<int> ftiles;              // of the levels above the tail
    bool spf;
  };
  const auto none = [](fld_params &) {};
  const Case cases[] = {
      // 16 x 8 x 4 boxes, then 8 x 4 x 4 where 256 are not reached
      {64, 64, 64, none, 5, 3, 2, 0, {4 * 8 * 16, 4 * 8 * 8, 2 * 4 * 4}, false},
      {36, 20, 12, none, 2, 1, 1, 0, {5 * 5 * 3}, false},
      {12, 20, 36, none, 2, 1, 1, 0, {2 * 5 * 9}, false},
      // either side of 1.5 x 2^20 cells
      {116, 116, 116, none, 3, 2, 2, 0, {8 * 15 * 29, 4 * 8 * 15}, false},
      {118, 118, 118, none, 2, 1, 1, 1, {2 * 8 * 59}, false},
      {256, 256, 256, none, 7, 5, 4, 2,
       {4 * 16 * 8, 2 * 8 * 32, 4 * 8 * 16, 4 * 8 * 8, 2 * 4 * 4}, false},
      // marching tiles asked for
      {64, 64, 64, [](fld_params &p) { p.fused_levels = 1; }, 5, 3, 2, 1,
       {1 * 4 * 32, 4 * 8 * 8, 2 * 4 * 4}, false},
      {64, 64, 64, [](fld_params &p) { p.fused_levels = 9; }, 5, 3, 2, 9,
       {1 * 4 * 32, 1 * 2 * 8, 1 * 1 * 4}, false},
      {64, 64, 64, [](fld_params &p) { p.fused_tile_z = 8; }, 5, 3, 2, 1,
       {1 * 4 * 8, 4 * 8 * 8, 2 * 4 * 4}, false},
      // the fused-tile SpMV takes 2048 tiles
      {96, 194, 320, [](fld_params &p) { p.fused_tile_z = 4; }, 2, 1, 1, 1, {2 * 13 * 80}, true},
      {320, 194, 96, [](fld_params &p) { p.fused_tile_z = 4; }, 2, 1, 1, 1, {5 * 13 * 24}, false},
      // tails: 512 cells, none, levels of up to 4096 in the per-sweep cycles
      {32, 32, 64, none, 4, 3, 2, 0, {2 * 4 * 16 * 2, 2 * 4 * 8, 1 * 2 * 4}, false},
      {32, 32, 32, [](fld_params &p) { p.tail_cells = 0; }, 4, 3, 3, 0,
       {4 * 8 * 8, 2 * 4 * 4, 1 * 2 * 2}, false},
      {32, 32, 32, [](fld_params &p) { p.tail_cells = 4096; }, 4, 1, 1, 0, {4 * 8 * 8}, false},
      {32, 32, 32, [](fld_params &p) { p.smoother = FLD_SMOOTH_JACOBI; }, 4, 3, 3, 0,
       {4 * 8 * 8, 2 * 4 * 4, 1 * 2 * 2}, false},
      // one level
      {4, 6, 10, none, 1, 1, 1, 0, {1 * 2 * 3}, false},
  };
  int bad = 0;
  for (const Case &c : cases) {
    fld_params p;
    fld_default_params(&p, 3e10, 1.0);
    c.set(p);
    fld_grid g{};
    g.nx = c.nx;
    g.ny = c.ny;
    g.nz = c.nz;
    g.dx = g.dy = g.dz = 1.0;
    const Hier h = make_hier(g, p);
    bool ok = h.levels == c.levels && h.tail == c.tail && h.tail_sweeps == c.tail_sweeps &&
              spmv_on_fused(h) == c.spf;
    printf("%d x %d x %d: levels %d tail %d %d spf %d:", c.nx, c.ny, c.nz, h.levels, h.tail,
           h.tail_sweeps, spmv_on_fused(h));
    for (int l = 0; l < h.levels; ++l) {
      const bool smoothed = l < (int)c.ftiles.size();
      printf(" %s%d", h.box[l] ? "box " : "", h.ftiles[l]);
      ok = ok && h.ftiles[l] == (smoothed ? c.ftiles[l] : 0);
      ok = ok && h.box[l] == (smoothed && l >= c.nbox);
    }
    printf(" %s\n", ok ? "ok" : "MISMATCH");
    bad += !ok;
  }
  printf("%d mismatches\n", bad);
  return bad;
}
