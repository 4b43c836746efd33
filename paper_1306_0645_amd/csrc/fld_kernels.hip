// HIP kernels (gfx950 / CDNA4) of the implicit grey FLD step.
//
// What is computed (Norman et al., arXiv:1306.0645):
//  - assembly: the flux limiter on every face from E^n (Sec. 2) and the
//    theta-method system (I - theta dt L) dE = dt (L E^n + eta) in
//    residual-correction form (Sec. 3.3);
//  - the multigrid V-cycle preconditioner with red/black Gauss-Seidel
//    smoothing (Table 1);
//  - the preconditioned conjugate-gradient recurrences (Table 1).
//
// All of this is memory-bound stencil and vector work (well under 1 flop per
// byte), so no kernel uses MFMA.  Every kernel processes a list of tiles;
// one 256-thread block (4 wave64) handles one tile: each thread owns one
// (x, y) column of the tile and walks its tz planes, so x-consecutive lanes
// read x-consecutive cells (coalesced).  Blocks are remapped so that each of
// the 8 XCDs gets a contiguous run of tiles and neighbouring tiles share an L2.
// Reductions are deterministic: wave sums by DPP row scans, a fixed LDS order,
// one partial per tile, then a per-problem finalize kernel that sums the
// partials in tile order.

#include "fld_device.h"
#include "fld_profile.h"

#include <math.h>

#include <type_traits>
#include <vector>

namespace fld {

// ---------------------------------------------------------------------------
// assembly (Sec. 2 limiter, Sec. 3.3 theta-method)
// ---------------------------------------------------------------------------

// D on the face between cells 1 and 2: arithmetic-mean E, harmonic-mean
// kappa, R from the face-normal difference (floored at R_min, and R_min when
// the face mean is not positive), capped at D_max.  Comparisons are written
// so that NaN inputs propagate.
__device__ __forceinline__ double face_D(double e1, double e2, double k1,
                                         double k2, double ih, double c,
                                         double dmax, double rmin) {
  const double ebar = 0.5 * (e1 + e2);
  const double ks = k1 + k2;
  const double kb = (ks != 0.0) ? 2.0 * k1 * k2 / ks : 0.0;
  double R = (ebar > 0.0) ? fabs(e2 - e1) * ih / ebar : rmin;
  R = (R < rmin) ? rmin : R;
  const double D = c / sqrt(9.0 * kb * kb + R * R);
  return (D > dmax) ? dmax : D;
}

// exclusive prefix sums of a and b over the block's threads (thread order)
// and their totals
__device__ __forceinline__ void block_scan2(int a, int b, int *sh, int &ea, int &eb,
                                            int &ta, int &tb) {
  constexpr int NW = kBlock / 64;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int ia = a, ib = b;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int ua = __shfl_up(ia, d, 64), ub = __shfl_up(ib, d, 64);
    if (lane >= d) {
      ia += ua;
      ib += ub;
    }
  }
  if (lane == 63) {
    sh[w] = ia;
    sh[NW + w] = ib;
  }
  __syncthreads();
  int oa = 0, ob = 0;
  ta = 0;
  tb = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if (i < w) {
      oa += sh[i];
      ob += sh[NW + i];
    }
    ta += sh[i];
    tb += sh[NW + i];
  }
  ea = oa + ia - a;
  eb = ob + ib - b;
}

// index of the q-th cell of tile t's box (x fastest)
__device__ __forceinline__ int box_cell(const Tile &t, int q, int nx, int ny) {
  const int txy = t.tx * t.ty, lz = q / txy, rm = q - lz * txy, ly = rm / t.tx;
  return ((t.z0 + lz) * ny + t.y0 + ly) * nx + t.x0 + (rm - ly * t.tx);
}

// the tile's listed cells (bits: the listed planes of the thread's column, m0
// and m1 of them of colour 0 and 1) into llist and lcnt
__device__ __forceinline__ void list_cells(const Tile &t, const Col &col, int tid,
                                           const ProbDev &P, int nx, int ny,
                                           unsigned long long bits, int m0, int m1) {
  __shared__ int sh[2 * (kBlock / 64)];
  int e0, e1, n0, n1;
  block_scan2(m0, m1, sh, e0, e1, n0, n1);
  while (bits) {
    const int b = __ffsll((long long)bits) - 1;
    bits &= bits - 1;
    const int k = t.z0 + b;
    const int q = ((col.i + col.j + k) & 1) ? n0 + e1++ : e0++;
    P.llist[box_cell(t, q, nx, ny)] = (k * ny + col.j) * nx + col.i;
  }
  if (threadIdx.x == 0) {
    P.lcnt[2 * (tid - P.t0)] = n0;
    P.lcnt[2 * (tid - P.t0) + 1] = n1;
  }
}

// edge faces of an assembly tile: kEdgeZ planes at a time, of at most 64
// columns (or, in a tile 4 wide, 64 rows)
constexpr int kEdgeZ = 8, kEdge = kEdgeZ * 64;

// One thread per (x, y) column of the tile, walking z: E and kappa of the
// column at k-1, k, k+1 stay in registers and the -z face of plane k is the +z
// face computed at plane k-1.  A limiter costs some 60 instructions (three
// divisions and a root), so the -x and -y faces are not evaluated again but
// taken, through LDS, from the threads whose + faces they are; the tile's own
// -x and -y edges are evaluated for 8 planes at a time: 3.5 limiters a cell in
// a tile of 64 x 4 x 8 instead of 5.  The cells of the local sweeps are listed
// here too (local; see k_local), where their faces are at hand.  Measured at
// 256^3, mixed, warm: 545 + 116 us with five limiters a cell and the lists in a
// pass of their own, 494 us together.
template <bool NT>
__global__ __launch_bounds__(kBlock) void k_assemble(Tables T, TileList L0,
                                                     double c_light, double theta,
                                                     double dmax, double rmin,
                                                     int mixed, int local,
                                                     double coupling) {
  int tid;
  const Tile t = get_tile(L0, tid);
  const Scal &sc = T.sc[t.prob];
  if (!asm_due(sc)) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const StepDev S = T.sd[t.prob];
  const Col col = tile_col(t);
  const double tdt = theta * S.dt;
  const double ix2 = S.idx * S.idx, iy2 = S.idy * S.idy, iz2 = S.idz * S.idz;
  const double *__restrict__ E = S.E;
  const double *__restrict__ K = S.kappa;
  const double *__restrict__ eta = S.eta;
  double *__restrict__ Tx = L.Tx;
  double *__restrict__ Ty = L.Ty;
  double *__restrict__ Tz = L.Tz;
  double *__restrict__ Dg = L.diag;
  double *__restrict__ bv = P.b;
  double *__restrict__ rv = rcur(P, sc);
  double *__restrict__ xv = P.x;
  // warm start from two history buffers that nothing writes here, so their
  // values at a neighbour are read on the fly (the thread holds all 6 faces):
  // extrapolated guess x0 = w1 dE(n) + w2 dE(n-1): r = b - A x0 comes out of
  // this pass; Galerkin guess: this pass sums (h_i, A h_j) and (h_i, b) for
  // the new operator, and k_warm_x forms x0 and r once c is known
  const bool warm = S.warm > 0.0, gal = S.warm > 1.0;
  const double w1 = S.w1, w2 = S.w2;
  const double *__restrict__ h1 = S.h1;
  const double *__restrict__ h2 = S.h2;
  auto guess = [&](int g) { return h2 ? w1 * h1[g] + w2 * h2[g] : w1 * h1[g]; };
  double bb = 0.0, rr = 0.0, g11 = 0.0, g12 = 0.0, g22 = 0.0, gb1 = 0.0,
         gb2 = 0.0;
  const int nx = L.nx, ny = L.ny, nz = L.nz, plane = nx * ny;
  __shared__ double sx[2][kBlock], sy[2][kBlock];  // Dxp, Dyp of a plane
  __shared__ double ex[kEdge], ey[kEdge];          // edge faces [plane][row], [plane][column]
  // -x faces of column x0 and -y faces of row y0 of the tile on planes
  // z0 + l0 .. z0 + l0 + n - 1
  auto edges = [&](int l0, int n) {
    for (int q = threadIdx.x; q < n * (t.ty + t.tx); q += kBlock) {
      const bool isx = q < n * t.ty;
      const int u = isx ? q : q - n * t.ty, w = isx ? t.ty : t.tx;
      const int lz = u / w, lw = u - lz * w;
      const int i = isx ? t.x0 : t.x0 + lw, j = isx ? t.y0 + lw : t.y0;
      const int c = (t.z0 + l0 + lz) * plane + j * nx + i;
      const int m = isx ? (i == 0 ? c + nx - 1 : c - 1) : (j == 0 ? c + (ny - 1) * nx : c - nx);
      const double D = face_D(E[m], E[c], K[m], K[c], isx ? S.idx : S.idy, c_light, dmax, rmin);
      if (isx) ex[u] = D;
      else ey[u] = D;
    }
  };
  unsigned long long bits = 0;  // listed planes of the column: bit k - z0
  int m0 = 0, m1 = 0;           // listed cells of colour 0, 1
  const int lx = col.i - t.x0, ly = col.j - t.y0;
  {
    // (threads beyond the tile's rows follow row 0 up to the barriers)
    const int i = col.i, j = col.on ? col.j : t.y0;
    const int dxm = (i == 0) ? nx - 1 : -1, dxp = (i == nx - 1) ? 1 - nx : 1;
    const int dym = (j == 0) ? (ny - 1) * nx : -nx;
    const int dyp = (j == ny - 1) ? -(ny - 1) * nx : nx;
    int cc = t.z0 * plane + j * nx + i;
    const int cm = (t.z0 == 0) ? cc + (nz - 1) * plane : cc - plane;
    double Em = E[cm], Km = K[cm];
    double Ec = E[cc], Kc = K[cc];
    double Dzm = face_D(Em, Ec, Km, Kc, S.idz, c_light, dmax, rmin);
    double gm = 0.0, gc = 0.0;  // guess (Galerkin: dE(n)) at planes k - 1, k
    double um = 0.0, uc = 0.0;  // Galerkin: dE(n-1) at planes k - 1, k
    if (gal) {
      gm = h1[cm];
      gc = h1[cc];
      if (h2) {
        um = h2[cm];
        uc = h2[cc];
      }
    } else if (warm) {
      gm = guess(cm);
      gc = guess(cc);
    }
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const int lz = k - t.z0, le = lz % kEdgeZ;
      if (le == 0) {
        if (lz) __syncthreads();  // the last planes' edge faces are read
        edges(lz, min(kEdgeZ, t.tz - lz));
      }
      const int cp = (k == nz - 1) ? cc - (nz - 1) * plane : cc + plane;
      const double Ep = E[cp], Kp = K[cp];
      const double Exp = E[cc + dxp], Exm = E[cc + dxm];
      const double Eyp = E[cc + dyp], Eym = E[cc + dym];
      const double Dxp = face_D(Ec, Exp, Kc, K[cc + dxp], S.idx, c_light, dmax, rmin);
      const double Dyp = face_D(Ec, Eyp, Kc, K[cc + dyp], S.idy, c_light, dmax, rmin);
      const double Dzp = face_D(Ec, Ep, Kc, Kp, S.idz, c_light, dmax, rmin);
      const int sl = lz & 1;
      sx[sl][threadIdx.x] = Dxp;
      sy[sl][threadIdx.x] = Dyp;
      // (two slots: a plane's reads and the writes of the plane after the next
      // are a barrier apart)
      __syncthreads();
      if (!col.on) {
        cc = cp;
        continue;
      }
      const double Dxm = lx > 0 ? sx[sl][threadIdx.x - 1] : ex[le * t.ty + ly];
      const double Dym = ly > 0 ? sy[sl][threadIdx.x - t.tx] : ey[le * t.tx + lx];
      const double mu = S.adot_a + c_light * Kc;
      const double faces =
          (Dxp + Dxm) * ix2 + (Dyp + Dym) * iy2 + (Dzp + Dzm) * iz2;
      const double diag = 1.0 + tdt * (mu + faces);
      const double LE = (Dxp * (Exp - Ec) - Dxm * (Ec - Exm)) * ix2 +
                        (Dyp * (Eyp - Ec) - Dym * (Ec - Eym)) * iy2 +
                        (Dzp * (Ep - Ec) - Dzm * (Ec - Em)) * iz2 - mu * Ec;
      const double b = S.dt * (LE + stream_in<NT>(&eta[cc]));
      const double tx = tdt * Dxp * ix2, ty = tdt * Dyp * iy2, tz = tdt * Dzp * iz2;
      const double txm = tdt * Dxm * ix2, tym = tdt * Dym * iy2, tzm = tdt * Dzm * iz2;
      if (local && tx + txm + ty + tym + tz + tzm > coupling * diag) {
        bits |= 1ull << lz;
        if ((i + j + k) & 1) ++m1;
        else ++m0;
      }
      stream_out<NT>(&Tx[cc], tx);
      stream_out<NT>(&Ty[cc], ty);
      stream_out<NT>(&Tz[cc], tz);
      stream_out<NT>(&Dg[cc], diag);
      if (mixed) {
        stream_out<NT>(&L.Tx32[cc], (float)tx);
        stream_out<NT>(&L.Ty32[cc], (float)ty);
        stream_out<NT>(&L.Tz32[cc], (float)tz);
        stream_out<NT>(&L.diag32[cc], (float)diag);
      }
      stream_out<NT>(&bv[cc], b);
      bb += b * b;
      if (gal) {
        // A h at the cell for h = dE(n) and dE(n-1); x and r are k_warm_x's
        const double gp = h1[cp];
        const double a1 = diag * gc - (tx * h1[cc + dxp] + txm * h1[cc + dxm] +
                                       ty * h1[cc + dyp] + tym * h1[cc + dym] +
                                       tz * gp + tzm * gm);
        g11 += gc * a1;
        gb1 += gc * b;
        gm = gc;
        gc = gp;
        if (h2) {
          const double up = h2[cp];
          const double a2 = diag * uc - (tx * h2[cc + dxp] + txm * h2[cc + dxm] +
                                         ty * h2[cc + dyp] + tym * h2[cc + dym] +
                                         tz * up + tzm * um);
          g12 += uc * a1;  // (dE(n-1), A dE(n)): A is symmetric
          g22 += uc * a2;
          gb2 += uc * b;
          um = uc;
          uc = up;
        }
      } else if (warm) {
        const double gp = guess(cp);
        const double off = tx * guess(cc + dxp) + txm * guess(cc + dxm) +
                           ty * guess(cc + dyp) + tym * guess(cc + dym) +
                           tz * gp + tzm * gm;
        const double r = b - (diag * gc - off);
        stream_out<NT>(&xv[cc], gc);
        stream_out<NT>(&rv[cc], r);
        rr += r * r;
        gm = gc;
        gc = gp;
      } else {
        stream_out<NT>(&xv[cc], 0.0);
        stream_out<NT>(&rv[cc], b);
      }
      Em = Ec;
      Km = Kc;
      Ec = Ep;
      Kc = Kp;
      Dzm = Dzp;
      cc = cp;
    }
  }
  const double sums[kAsmSums] = {bb, rr, g11, g12, g22, gb1, gb2};
  write_sums(T.gpart, tid, sums);
  if (local) list_cells(t, col, tid, P, nx, ny, bits, m0, m1);
}

// Coarse operator of level lc from level lc-1 (one thread per coarse cell).
// The coarse "mass" (diagonal minus faces) is the sum of the 8 children's.
// Coarse faces, op = 0: coarse_scale times the sum of the 4 fine faces they
// cover.  op = 1: each of the 4 fine rows that cross the coarse face joins
// the two coarse centres through three fine faces in series, half of the
// inner face of each coarse cell and the whole face between them, so the row
// conducts 1 / (0.5 / T_in + 1 / T_mid + 0.5 / T_in'); the coarse face is
// 2 coarse_scale times the sum over the rows (for a uniform medium both rules
// give coarse_scale times the 4 fine faces).  Either way a coarse face is the
// same sum of the same terms for both cells it joins, so the coarse operator
// is exactly symmetric.
__device__ __forceinline__ double series3(double a, double b, double c) {
  return 1.0 / (0.5 / a + 1.0 / b + 0.5 / c);
}

__global__ __launch_bounds__(kBlock) void k_coarsen(Tables T, TileList LC,
                                                    int lc, double scale,
                                                    int mixed, int op) {
  const Tile t = get_tile(LC);
  const Scal &sc = T.sc[t.prob];
  if (!asm_due(sc)) return;
  const LevelDev F = T.lv[(lc - 1) * T.nprob + t.prob];
  const LevelDev C = T.lv[lc * T.nprob + t.prob];
  const ProbDev &P = T.pd[t.prob];
  // the coarsest level, where its solve streams the operator: the reciprocal
  // diagonal too, behind that solve's x
  const bool inv = lc == P.levels - 1 && C.n > kTailSmall && C.n <= kTailBig;
  const Col col = tile_col(t);
  if (!col.on) return;
  const int fx = F.nx, fy = F.ny, fz = F.nz;
  for (int K = t.z0; K < t.z0 + t.tz; ++K) {
    const int I = col.i, J = col.j;
    double mass = 0.0, txp = 0.0, txm = 0.0, typ = 0.0, tym = 0.0,
           tzp = 0.0, tzm = 0.0;
#pragma unroll
    for (int cz = 0; cz < 2; ++cz)
#pragma unroll
      for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
          const Nb n = nbrs(2 * I + cx, 2 * J + cy, 2 * K + cz, fx, fy, fz);
          const double fxp = F.Tx[n.c], fxm = F.Tx[n.xm];
          const double fyp = F.Ty[n.c], fym = F.Ty[n.ym];
          const double fzp = F.Tz[n.c], fzm = F.Tz[n.zm];
          mass += F.diag[n.c] - (fxp + fxm + fyp + fym + fzp + fzm);
          if (op == 0) {
            if (cx == 1) txp += fxp; else txm += fxm;
            if (cy == 1) typ += fyp; else tym += fym;
            if (cz == 1) tzp += fzp; else tzm += fzm;
          } else {
            // a child on the + side: its -face (inner), its +face (the
            // coarse face) and the neighbour's +face; on the - side: the
            // -face of the cell two below, its own -face and +face
            if (cx == 1) {
              txp += series3(fxm, fxp, F.Tx[n.xp]);
            } else {
              const int i2 = 2 * I >= 2 ? 2 * I - 2 : 2 * I - 2 + fx;
              txm += series3(F.Tx[n.c - 2 * I + i2], fxm, fxp);
            }
            if (cy == 1) {
              typ += series3(fym, fyp, F.Ty[n.yp]);
            } else {
              const int j2 = 2 * J >= 2 ? 2 * J - 2 : 2 * J - 2 + fy;
              tym += series3(F.Ty[n.c + (j2 - 2 * J) * fx], fym, fyp);
            }
            if (cz == 1) {
              tzp += series3(fzm, fzp, F.Tz[n.zp]);
            } else {
              const int k2 = 2 * K >= 2 ? 2 * K - 2 : 2 * K - 2 + fz;
              tzm += series3(F.Tz[n.c + (long long)(k2 - 2 * K) * fx * fy], fzm, fzp);
            }
          }
        }
    const double s2 = op == 0 ? scale : 2.0 * scale;
    txp *= s2; txm *= s2; typ *= s2; tym *= s2; tzp *= s2; tzm *= s2;
    const double diag = mass + txp + txm + typ + tym + tzp + tzm;
    const int o = (K * C.ny + J) * C.nx + I;
    C.Tx[o] = txp;
    C.Ty[o] = typ;
    C.Tz[o] = tzp;
    C.diag[o] = diag;
    if (inv) P.cs[C.n + o] = 1.0 / diag;
    if (mixed) {
      C.Tx32[o] = (float)txp;
      C.Ty32[o] = (float)typ;
      C.Tz32[o] = (float)tzp;
      C.diag32[o] = (float)diag;
    }
  }
}

// ---------------------------------------------------------------------------
// V-cycle kernels (any sweep count; one cell per lane, colour test per cell)
// ---------------------------------------------------------------------------

// First pre-smoothing sweep from x = 0: red cells x = f/d, then black cells
// from those red values (computed on the fly, so one pass suffices).
template <typename R, bool L0>
__global__ __launch_bounds__(kBlock) void k_pre0(Tables T, TileList TL, int l) {
  const Tile t = get_tile(TL);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[l * T.nprob + t.prob];
  const ProbDev P = T.pd[t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, L0>(L, P, sc);
  R *x = (R *)L.x;
  const Col col = tile_col(t);
  if (!col.on) return;
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    const Nb n = nbrs(col.i, col.j, k, L.nx, L.ny, L.nz);
    R v;
    if (((col.i + col.j + k) & 1) == 0) {
      v = f(n.c) * recip(C.d[n.c]);
    } else {
      auto red = [&](int q) { return f(q) * recip(C.d[q]); };
      v = (f(n.c) + offsum(C, n, red)) * recip(C.d[n.c]);
    }
    x[n.c] = v;
  }
}

// One half-sweep of red/black Gauss-Seidel on the cells of one colour
// (colour 0 = red = even i+j+k), in place.
template <typename R, bool L0>
__global__ __launch_bounds__(kBlock) void k_half(Tables T, TileList TL, int l,
                                                 int colour) {
  const Tile t = get_tile(TL);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[l * T.nprob + t.prob];
  const ProbDev P = T.pd[t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, L0>(L, P, sc);
  R *x = (R *)L.x;
  const Col col = tile_col(t);
  if (!col.on) return;
  auto xv = [&](int q) { return x[q]; };
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    if (((col.i + col.j + k) & 1) != colour) continue;
    const Nb n = nbrs(col.i, col.j, k, L.nx, L.ny, L.nz);
    x[n.c] = (f(n.c) + offsum(C, n, xv)) * recip(C.d[n.c]);
  }
}

// Black half-sweep fused with the coarse-grid correction: the red
// neighbours are read as x + e(parent).  (The black cells' own corrected
// value is overwritten by the sweep, so it is never formed.)
template <typename R, bool L0>
__global__ __launch_bounds__(kBlock) void k_prolong_black(Tables T, TileList TL,
                                                          int l, int trilinear) {
  const Tile t = get_tile(TL);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[l * T.nprob + t.prob];
  const ProbDev P = T.pd[t.prob];
  const bool has_coarse = l + 1 < P.levels;
  const LevelDev Cl = T.lv[min(l + 1, kMaxLevels - 1) * T.nprob + t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, L0>(L, P, sc);
  R *x = (R *)L.x;
  const R *e = (const R *)Cl.x;
  const int cnx = Cl.nx, cny = Cl.ny, cnz = Cl.nz;
  const bool tri = trilinear != 0;
  const Col col = tile_col(t);
  if (!col.on) return;
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    if (((col.i + col.j + k) & 1) != 1) continue;
    const int i = col.i, j = col.j;
    const Nb n = nbrs(i, j, k, nx, ny, nz);
    R s;
    if (has_coarse) {
      const int im = i == 0 ? nx - 1 : i - 1, ip = i == nx - 1 ? 0 : i + 1;
      const int jm = j == 0 ? ny - 1 : j - 1, jp = j == ny - 1 ? 0 : j + 1;
      const int km = k == 0 ? nz - 1 : k - 1, kp = k == nz - 1 ? 0 : k + 1;
      auto par = [&](int a, int b2, int c2) {
        return coarse_corr(e, a, b2, c2, cnx, cny, cnz, tri);
      };
      s = C.tx[n.c] * (x[n.xp] + par(ip, j, k)) +
          C.tx[n.xm] * (x[n.xm] + par(im, j, k)) +
          C.ty[n.c] * (x[n.yp] + par(i, jp, k)) +
          C.ty[n.ym] * (x[n.ym] + par(i, jm, k)) +
          C.tz[n.c] * (x[n.zp] + par(i, j, kp)) +
          C.tz[n.zm] * (x[n.zm] + par(i, j, km));
    } else {
      auto xv = [&](int q) { return x[q]; };
      s = offsum(C, n, xv);
    }
    x[n.c] = (f(n.c) + s) * recip(C.d[n.c]);
  }
}

// Last red half-sweep on the finest level, producing z = s * x (FP64 form: in
// place; mixed form: x itself as z32, z = zscale z32) and the partial sums r.z
// and (flexible PCG, except at a (re)start) r.z_old.
template <typename R>
__global__ __launch_bounds__(kBlock) void k_half_out(Tables T, TileList TL,
                                                     int flexible) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, true>(L, P, sc);
  R *x = (R *)L.x;
  const double s = sc.s, zs_old = sc.zscale;
  const bool rd_old = flexible && !sc.restart;
  const Col col = tile_col(t);
  double rz = 0.0, rzo = 0.0;
  if (col.on) {
    auto xv = [&](int q) { return x[q]; };
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const Nb n = nbrs(col.i, col.j, k, L.nx, L.ny, L.nz);
      R v;
      const bool red = ((col.i + col.j + k) & 1) == 0;
      if (red) v = (f(n.c) + offsum(C, n, xv)) * recip(C.d[n.c]);
      else v = x[n.c];
      const double rv = f.r[n.c];
      const double zv = (double)v * s;
      if constexpr (sizeof(R) == 8) {
        // FP64: the finest iterate is z itself
        if (red) x[n.c] = (R)zv;
      } else {
        if (rd_old) rzo += rv * ((double)P.z32[n.c] * zs_old);
        P.z32[n.c] = v;
      }
      rz += rv * zv;
    }
  }
  write_partials(T, tid, rz, rzo);
}

// Residual f - A x on the fine level summed over the 8 children of each
// coarse cell: the coarse right-hand side (restriction = transpose of the
// piecewise-constant prolongation).  One thread per coarse cell.
template <typename R, bool L0>
__global__ __launch_bounds__(kBlock) void k_resid_restrict(Tables T,
                                                           TileList LC, int lc) {
  const Tile t = get_tile(LC);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev F = T.lv[(lc - 1) * T.nprob + t.prob];
  const LevelDev Cv = T.lv[lc * T.nprob + t.prob];
  const ProbDev P = T.pd[t.prob];
  const Coef<R> C = coefs<R>(F);
  const auto f = fsrc<R, L0>(F, P, sc);
  const R *x = (const R *)F.x;
  R *fc = (R *)Cv.f;
  const Col col = tile_col(t);
  if (!col.on) return;
  auto xv = [&](int q) { return x[q]; };
  for (int K = t.z0; K < t.z0 + t.tz; ++K) {
    const int I = col.i;
    R acc = 0;
#pragma unroll
    for (int cz = 0; cz < 2; ++cz)
#pragma unroll
      for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) {
          const Nb n = nbrs(2 * I + cx, 2 * col.j + cy, 2 * K + cz, F.nx,
                            F.ny, F.nz);
          acc += f(n.c) - (C.d[n.c] * x[n.c] - offsum(C, n, xv));
        }
    fc[(K * Cv.ny + col.j) * Cv.nx + I] = acc;
  }
}

// ---------------------------------------------------------------------------
// Weighted Jacobi smoother (the alternative to red/black Gauss-Seidel):
//   x_new = x + w (f - A x) / d,  w = 6/7,
// which updates every cell from the old iterate, so it ping-pongs between
// LevelDev::x and LevelDev::x2.  Symmetric in both sweeps, so the FP64
// V-cycle stays a symmetric preconditioner.
// ---------------------------------------------------------------------------

constexpr double kJacobiW = 6.0 / 7.0;

template <typename R, bool L0>
__global__ __launch_bounds__(kBlock) void k_jacobi(Tables T, TileList TL, int l,
                                                   int mode, int in_x2,
                                                   int flexible) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[l * T.nprob + t.prob];
  const ProbDev P = T.pd[t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, L0>(L, P, sc);
  const R w = (R)kJacobiW;
  const R *xin = (const R *)(in_x2 ? L.x2 : L.x);
  R *xout = (R *)(in_x2 ? L.x : L.x2);
  const Col col = tile_col(t);
  double rz = 0.0, rzo = 0.0;
  if (col.on) {
    auto xv = [&](int q) { return xin[q]; };
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const Nb n = nbrs(col.i, col.j, k, L.nx, L.ny, L.nz);
      R v;
      if (mode == 0) {
        v = w * f(n.c) * recip(C.d[n.c]);
      } else {
        const R xc = xin[n.c];
        v = xc + w * (f(n.c) - (C.d[n.c] * xc - offsum(C, n, xv))) * recip(C.d[n.c]);
      }
      if constexpr (L0) {
        if (mode == 2) {
          // z = s x (FP64 form: into z; mixed form: x itself into z32)
          const double zv = (double)v * sc.s;
          const double rv = f.r[n.c];
          if constexpr (sizeof(R) == 8) {
            if (flexible) rzo += rv * P.z[n.c];
            P.z[n.c] = zv;
          } else {
            if (flexible && !sc.restart) rzo += rv * ((double)P.z32[n.c] * sc.zscale);
            P.z32[n.c] = v;
          }
          rz += rv * zv;
          continue;
        }
      }
      xout[n.c] = v;
    }
  }
  if constexpr (L0) {
    if (mode == 2) write_partials(T, tid, rz, rzo);
  }
}

// out = x + P e over every cell of level l (P from coarse_corr); out is x
// itself or x2
template <typename R>
__global__ __launch_bounds__(kBlock) void k_prolong_add(Tables T, TileList TL,
                                                        int l, int trilinear,
                                                        int to_x2) {
  const Tile t = get_tile(TL);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[l * T.nprob + t.prob];
  const ProbDev P = T.pd[t.prob];
  const bool has_coarse = l + 1 < P.levels;  // one-level problem: a copy
  const LevelDev Cl = T.lv[min(l + 1, kMaxLevels - 1) * T.nprob + t.prob];
  const R *e = (const R *)Cl.x;
  const R *x = (const R *)L.x;
  R *out = (R *)(to_x2 ? L.x2 : L.x);
  const Col col = tile_col(t);
  if (!col.on) return;
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    const int c = (k * L.ny + col.j) * L.nx + col.i;
    const R ec = has_coarse ? coarse_corr(e, col.i, col.j, k, Cl.nx, Cl.ny,
                                          Cl.nz, trilinear != 0)
                            : (R)0;
    out[c] = x[c] + ec;
  }
}

// ---------------------------------------------------------------------------
// Krylov kernels (FP64, finest level; two x-consecutive cells per thread)
// ---------------------------------------------------------------------------

// p = z + beta p_old (formed at the cell and its neighbours on the fly),
// q = A p, partial p . q.  p is double-buffered so neighbours read the old
// direction while the new one is written.  Each thread walks its column in z
// keeping p at planes k-1, k, k+1 and the -z face in registers.
// Krylov storage modes (KM): KM_FP64: z and p FP64.  KM_MIX32 (mixed form):
// z, p_old and p FP32 at a scale each (zs for z and p, ps for p_old); p is
// rounded to FP32 before it is used, so q, the dot and the later x update all
// see the direction that is stored.  KM_MIX64 (mixed form with an FP64
// direction): z FP32 at the scale zs (the V-cycle's output as it is), p_old
// and p FP64.
//
// The iterations of the fused cycle store the direction every other time:
//   F_SKIP:  p_k = z_k + beta_k base; neither p nor x is written;
//   F_STORE: p_k again from z_k (kept in the other z buffer) and the base,
//            p_{k+1} = z_{k+1} + beta_{k+1} p_k is stored as the next base,
//            and x += alpha_{k-1} base + alpha_k p_k, both updates at once.
// p_k comes out of the same fused multiply-adds both times, so q, x and the
// stored directions are bit for bit those of an iteration that stores every
// direction and updates x each time, for 52 and 80 B a cell instead of 76
// and 76 (FP64 direction; FP32: 48 and 72 instead of 68 and 68; in the FP64
// form 56 and 88 instead of 64 and, in k_update, 24 of its 48).  Bound by
// these bytes: 640^3, FP64 direction, 4252 -> 3712 us a launch (4.67 TB/s of
// them).  F_PLAIN (the other iterations): p is stored every time, x updated
// in k_update.
enum : int { KM_FP64 = 0, KM_MIX32 = 1, KM_MIX64 = 2 };
enum : int { F_PLAIN = 0, F_SKIP = 1, F_STORE = 2 };

template <int KM>
using ZT = std::conditional_t<KM == KM_FP64, double, float>;
template <int KM>
using DirT = std::conditional_t<KM == KM_MIX32, float, double>;

// what the directions are formed from; BASE: a base exists (beta != 0)
template <int F, bool BASE, int KM>
struct DirSrc {
  using D = DirT<KM>;
  const ZT<KM> *__restrict__ z;    // this iteration's z
  const ZT<KM> *__restrict__ z1;   // F_STORE: the z before
  const D *__restrict__ po;        // base (p_old)
  double zs, zs1, ps;              // scales of z, z1 and (KM_MIX32) the base
  double c, c1;                    // the direction's coefficient of the one before
  double a, a1;                    // F_STORE: x += a1 base + a mid
  // loads at a cell, then the direction there; F_STORE: mid is p_k
  struct In {
    ZT<KM> z, z1;
    D po;
  };
  __device__ __forceinline__ In load(int g) const {
    In v;
    v.z = z[g];
    v.z1 = F == F_STORE ? z1[g] : (ZT<KM>)0;
    v.po = BASE ? po[g] : (D)0;
    return v;
  }
  __device__ __forceinline__ static D one(ZT<KM> zv, double s, double cf, D prev) {
    if constexpr (KM == KM_MIX32) return (float)__builtin_fma(cf, (double)prev, (double)zv);
    else if constexpr (KM == KM_MIX64) return __builtin_fma(cf, prev, s * (double)zv);
    else return __builtin_fma(cf, prev, zv);
  }
  __device__ __forceinline__ static D first(ZT<KM> zv, double s) {
    if constexpr (KM == KM_MIX64) return s * (double)zv;
    else return zv;
  }
  __device__ __forceinline__ D make(const In &v, D &mid) const {
    if constexpr (F == F_STORE) {
      mid = BASE ? one(v.z1, zs1, c1, v.po) : first(v.z1, zs1);
      return one(v.z, zs, c, mid);
    } else {
      mid = (D)0;
      return BASE ? one(v.z, zs, c, v.po) : first(v.z, zs);
    }
  }
  __device__ __forceinline__ D raw(int g) const {
    D mid;
    return make(load(g), mid);
  }
  __device__ __forceinline__ double val(D v) const {
    if constexpr (KM == KM_MIX32) return zs * (double)v;
    else return v;
  }
  // x with the two pending updates
  __device__ __forceinline__ double advance(double x, D base, D mid) const {
    if constexpr (KM == KM_MIX32) {
      if (BASE) x = __builtin_fma(a1, ps * (double)base, x);
      return __builtin_fma(a, zs1 * (double)mid, x);
    } else {
      if (BASE) x = __builtin_fma(a1, base, x);
      return __builtin_fma(a, mid, x);
    }
  }
};

template <int F, bool BASE, int KM>
__device__ __forceinline__ DirSrc<F, BASE, KM> dir_src(const ProbDev &P, const Scal &sc) {
  DirSrc<F, BASE, KM> S;
  S.z = zcur<ZT<KM>>(P, sc);
  S.z1 = znext<ZT<KM>>(P, sc);
  if constexpr (KM == KM_MIX32) S.po = sc.pbuf ? P.pf1 : P.pf0;
  else S.po = sc.pbuf ? P.p1 : P.p0;
  S.zs = sc.zscale;
  S.zs1 = sc.zscale1;
  S.ps = sc.pscale;
  S.c = sc.beta;
  S.c1 = sc.beta1;
  if constexpr (KM == KM_MIX32) {
    // the previous direction's share, in z's scale
    S.c = F == F_STORE ? sc.beta * sc.zscale1 / sc.zscale : sc.beta * sc.pscale / sc.zscale;
    S.c1 = sc.beta1 * sc.pscale / sc.zscale1;
  }
  S.a = sc.alpha;
  S.a1 = sc.alpha1;
  return S;
}

template <int KM>
__device__ __forceinline__ DirT<KM> *dir_next(const ProbDev &P, const Scal &sc) {
  if constexpr (KM == KM_MIX32) return sc.pbuf ? P.pf0 : P.pf1;
  else return sc.pbuf ? P.p0 : P.p1;
}

template <bool NT, int F, bool BASE, int KM>
__device__ __forceinline__ double spmv_column(
    const Tile &t, const Col &col, int nx, int ny, int nz, const DirSrc<F, BASE, KM> &S,
    DirT<KM> *__restrict__ pn, double *__restrict__ q, const double *__restrict__ Tx,
    const double *__restrict__ Ty, const double *__restrict__ Tz,
    const double *__restrict__ Dg, double *__restrict__ x) {
  using D = DirT<KM>;
  const int plane = nx * ny, i = col.i, j = col.j;
  const int dxm = (i == 0) ? nx - 1 : -1, dxp = (i == nx - 1) ? 1 - nx : 1;
  const int dym = (j == 0) ? (ny - 1) * nx : -nx;
  const int dyp = (j == ny - 1) ? -(ny - 1) * nx : nx;
  int c = t.z0 * plane + j * nx + i;
  const int cm0 = (t.z0 == 0) ? c + (nz - 1) * plane : c - plane;
  const auto ic = S.load(c);
  D m_c, m_p;            // F_STORE: p_k at planes k, k + 1, and the base there
  D r_m = S.raw(cm0), r_c = S.make(ic, m_c), b_c = ic.po;
  double tz_m = Tz[cm0];
  double acc = 0.0;
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    const int cp = (k == nz - 1) ? c - (nz - 1) * plane : c + plane;
    const auto ip = S.load(cp);
    const D r_p = S.make(ip, m_p);
    const double s = Tx[c] * S.val(S.raw(c + dxp)) + Tx[c + dxm] * S.val(S.raw(c + dxm)) +
                     Ty[c] * S.val(S.raw(c + dyp)) + Ty[c + dym] * S.val(S.raw(c + dym)) +
                     Tz[c] * S.val(r_p) + tz_m * S.val(r_m);
    const double p_c = S.val(r_c);
    const double qq = stream_in<NT>(&Dg[c]) * p_c - s;
    if constexpr (F == F_STORE) stream_out<NT>(&x[c], S.advance(stream_in<NT>(&x[c]), b_c, m_c));
    if constexpr (F != F_SKIP) stream_out<NT>(&pn[c], r_c);
    stream_out<NT>(&q[c], qq);
    acc += p_c * qq;
    tz_m = Tz[c];
    r_m = r_c;
    r_c = r_p;
    m_c = m_p;
    b_c = ip.po;
    c = cp;
  }
  return acc;
}

template <bool LAZY, int KM, bool NT>
__global__ __launch_bounds__(kBlock) void k_spmv_p(Tables T, TileList TL) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const Col col = tile_col(t);
  double pq = 0.0;
  if (col.on) {
    auto run = [&](auto S) {
      return spmv_column<NT>(t, col, L.nx, L.ny, L.nz, S, dir_next<KM>(P, sc), P.q, L.Tx, L.Ty,
                             L.Tz, L.diag, P.x);
    };
    if constexpr (LAZY) {
      if (sc.lag) {
        if (sc.hasb) pq = run(dir_src<F_STORE, true, KM>(P, sc));
        else pq = run(dir_src<F_STORE, false, KM>(P, sc));
      } else {
        if (sc.hasb) pq = run(dir_src<F_SKIP, true, KM>(P, sc));
        else pq = run(dir_src<F_SKIP, false, KM>(P, sc));
      }
    } else {
      if (sc.beta != 0.0) pq = run(dir_src<F_PLAIN, true, KM>(P, sc));
      else pq = run(dir_src<F_PLAIN, false, KM>(P, sc));
    }
  }
  write_partials(T, tid, pq, 0.0);
}

// The fused iteration's SpMV on the fused tiles (64 x 16 cells, tz planes):
// each thread takes kSpRows consecutive rows of one column and walks z, so
// the y neighbours inside its rows come from registers and only the rows
// just below and above are loaded (2 of 16 rows, against 2 of 4 for the
// 64 x 4 tiles), as are the z neighbours (2 planes per tile).  The x
// neighbours come from the adjacent lanes (a wave is one 64-cell row
// segment); only the lanes at the tile's x edges load theirs.  Nothing is
// read twice: a plane's direction and z were loaded one plane earlier and
// are held, where reading them again a plane later would miss the L2, which
// holds less than one plane of all the resident tiles.  Per cell the
// arithmetic is spmv_column's, term by term, so q and p are the same.
// (Always streaming: 2048 such tiles are beyond the caches.)
constexpr int kSpRows = 4;

template <int F, bool BASE, int KM>
__device__ __forceinline__ double spmv_rows(
    const Tile &t, int lx, int i, int j0, int nr, int nx, int ny, int nz,
    const DirSrc<F, BASE, KM> &S, DirT<KM> *__restrict__ pn, double *__restrict__ q,
    const double *__restrict__ Tx, const double *__restrict__ Ty,
    const double *__restrict__ Tz, const double *__restrict__ Dg, double *__restrict__ x) {
  using D = DirT<KM>;
  const int plane = nx * ny;
  const int dxm = (i == 0) ? nx - 1 : -1, dxp = (i == nx - 1) ? 1 - nx : 1;
  const bool ledge = lx == 0, redge = lx == t.tx - 1;
  const int rlo = (j0 == 0 ? ny - 1 : j0 - 1) * nx;        // the row below
  const int rhi = (j0 + nr == ny ? 0 : j0 + nr) * nx;      // the row above
  const int km0 = t.z0 == 0 ? nz - 1 : t.z0 - 1;
  D pm[kSpRows], pc[kSpRows];  // p at k - 1, k
  D oc[kSpRows], mc[kSpRows];  // base and (F_STORE) p_k at k
  double tzm[kSpRows];
#pragma unroll
  for (int r = 0; r < kSpRows; ++r) {
    if (r < nr) {
      const int o = (j0 + r) * nx + i, c = t.z0 * plane + o;
      pm[r] = S.raw(km0 * plane + o);
      const auto in = S.load(c);
      oc[r] = in.po;
      pc[r] = S.make(in, mc[r]);
      tzm[r] = Tz[km0 * plane + o];
    }
  }
  double acc = 0.0;
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    const int kp = (k == nz - 1) ? 0 : k + 1;
    const int b = k * plane + i;
    D pp[kSpRows], op[kSpRows], mp[kSpRows];
#pragma unroll
    for (int r = 0; r < kSpRows; ++r) {
      if (r < nr) {
        const auto in = S.load(kp * plane + (j0 + r) * nx + i);
        op[r] = in.po;
        pp[r] = S.make(in, mp[r]);
      }
    }
    const D plo = S.raw(b + rlo), phi = S.raw(b + rhi);
    double tyd = Ty[b + rlo];  // the -y face of the next row
#pragma unroll
    for (int r = 0; r < kSpRows; ++r) {
      if (r < nr) {
        const int c = b + (j0 + r) * nx;
        D xl = __shfl_up(pc[r], 1, 64), xr = __shfl_down(pc[r], 1, 64);
        if (ledge) xl = S.raw(c + dxm);
        if (redge) xr = S.raw(c + dxp);
        const D dn = r == 0 ? plo : pc[r > 0 ? r - 1 : 0];
        const D up = r + 1 == nr ? phi : pc[r + 1 < kSpRows ? r + 1 : r];
        const double tyc = Ty[c];
        const double sm = Tx[c] * S.val(xr) + Tx[c + dxm] * S.val(xl) + tyc * S.val(up) +
                          tyd * S.val(dn) + Tz[c] * S.val(pp[r]) + tzm[r] * S.val(pm[r]);
        const double p_c = S.val(pc[r]);
        const double qq = stream_in<true>(&Dg[c]) * p_c - sm;
        if constexpr (F == F_STORE) stream_out<true>(&x[c], S.advance(stream_in<true>(&x[c]), oc[r], mc[r]));
        if constexpr (F != F_SKIP) stream_out<true>(&pn[c], pc[r]);
        stream_out<true>(&q[c], qq);
        acc += p_c * qq;
        tzm[r] = Tz[c];
        tyd = tyc;
      }
    }
#pragma unroll
    for (int r = 0; r < kSpRows; ++r) {
      if (r < nr) {
        pm[r] = pc[r];
        pc[r] = pp[r];
        oc[r] = op[r];
        mc[r] = mp[r];
      }
    }
  }
  return acc;
}

template <int KM>
__global__ __launch_bounds__(kBlock) void k_spmv_f(Tables T, TileList TL) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const int lx = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int nr = min(kSpRows, t.ty - kSpRows * g);
  double pq = 0.0;
  if (lx < t.tx && nr > 0) {
    const int i = t.x0 + lx, j0 = t.y0 + kSpRows * g;
    auto run = [&](auto S) {
      return spmv_rows(t, lx, i, j0, nr, L.nx, L.ny, L.nz, S, dir_next<KM>(P, sc), P.q, L.Tx,
                       L.Ty, L.Tz, L.diag, P.x);
    };
    if (sc.lag) {
      if (sc.hasb) pq = run(dir_src<F_STORE, true, KM>(P, sc));
      else pq = run(dir_src<F_STORE, false, KM>(P, sc));
    } else {
      if (sc.hasb) pq = run(dir_src<F_SKIP, true, KM>(P, sc));
      else pq = run(dir_src<F_SKIP, false, KM>(P, sc));
    }
  }
  write_partials(T, tid, pq, 0.0);
}

// out = s z32 right after a mixed-form cycle (s: the scale it ran at)
__global__ __launch_bounds__(kBlock) void k_z_out(Tables T, TileList TL, int fused,
                                                  double *__restrict__ out) {
  const Tile t = get_tile(TL);
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const Scal &sc = T.sc[t.prob];
  const double zs = sc.s;
  const float *z = fused ? znext(P, sc) : zcur(P, sc);
  const Col col = tile_col(t);
  if (!col.on) return;
  const int plane = L.nx * L.ny;
  int c = t.z0 * plane + col.j * L.nx + col.i;
  for (int k = 0; k < t.tz; ++k, c += plane) out[c] = (double)z[c] * zs;
}

// the newest direction p at cell c (after FIN_PQ has swapped the buffers)
template <int KM>
__device__ __forceinline__ double newest_p(const ProbDev &P, const Scal &sc, int c) {
  if constexpr (KM == KM_MIX32) return sc.pscale * (double)(sc.pbuf ? P.pf1 : P.pf0)[c];
  else return (sc.pbuf ? P.p1 : P.p0)[c];
}

// the pending update of x for problems that stopped iterating in the fused
// iteration: alpha1 base + alpha (z + beta base) where the newest direction
// was not stored, alpha base where it was
template <int KM>
__global__ __launch_bounds__(kBlock) void k_xfix(Tables T, TileList TL) {
  const Tile t = get_tile(TL);
  const Scal &sc = T.sc[t.prob];
  if (!sc.xlag || sc.phase == PH_ITER) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const Col col = tile_col(t);
  if (!col.on) return;
  const int plane = L.nx * L.ny;
  int c = t.z0 * plane + col.j * L.nx + col.i;
  if (!sc.lag) {
    for (int k = 0; k < t.tz; ++k, c += plane)
      P.x[c] = __builtin_fma(sc.alpha, newest_p<KM>(P, sc, c), P.x[c]);
    return;
  }
  auto run = [&](auto S) {
    S.zs1 = sc.zscale;  // the unstored direction is the newest
    for (int k = 0; k < t.tz; ++k, c += plane) {
      const auto in = S.load(c);
      DirT<KM> mid;
      const DirT<KM> p = S.make(in, mid);
      P.x[c] = S.advance(P.x[c], in.po, p);
    }
  };
  if (sc.hasb) run(dir_src<F_SKIP, true, KM>(P, sc));
  else run(dir_src<F_SKIP, false, KM>(P, sc));
}

// r -= alpha q, partial ||r||^2, and (X) x += alpha p
template <int KM, bool X, bool NT>
__global__ __launch_bounds__(kBlock) void k_update(Tables T, TileList TL) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const double alpha = sc.alpha;
  const double *__restrict__ q = P.q;
  double *__restrict__ x = P.x;
  double *__restrict__ r = rcur(P, sc);
  const Col col = tile_col(t);
  double rr = 0.0;
  if (col.on) {
    const int plane = L.nx * L.ny;
    int c = t.z0 * plane + col.j * L.nx + col.i;
    for (int k = 0; k < t.tz; ++k, c += plane) {
      if constexpr (X) stream_out<NT>(&x[c], stream_in<NT>(&x[c]) + alpha * newest_p<KM>(P, sc, c));
      const double rn = r[c] - alpha * stream_in<NT>(&q[c]);
      stream_out<NT>(&r[c], rn);
      rr += rn * rn;
    }
  }
  write_partials(T, tid, rr, 0.0);
}

// true residual r = b - A x in FP64 (problems whose recursive residual met
// the tolerance), partial ||r||^2
// (bound by its loads, of which the caches serve most: a plane's x and Tz are
// carried to the next one, and the stores cannot alias the loads.  256^3
// mixed, a pass of three steps: 15.71 -> 15.65 ms; 4 groups of 128^3 7.77 ->
// 7.72)
template <bool NT>
__global__ __launch_bounds__(kBlock) void k_true_resid(Tables T, TileList TL) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (sc.phase != PH_VERIFY) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const double *__restrict__ x = P.x;
  const double *__restrict__ Tx = L.Tx;
  const double *__restrict__ Ty = L.Ty;
  const double *__restrict__ Tz = L.Tz;
  double *__restrict__ rv = rcur(P, sc);
  const Col col = tile_col(t);
  double rr = 0.0;
  if (col.on) {
    const int nx = L.nx, ny = L.ny, nz = L.nz, plane = nx * ny;
    const int i = col.i, j = col.j;
    const int dxm = (i == 0) ? nx - 1 : -1, dxp = (i == nx - 1) ? 1 - nx : 1;
    const int dym = (j == 0) ? (ny - 1) * nx : -nx;
    const int dyp = (j == ny - 1) ? -(ny - 1) * nx : nx;
    int c = t.z0 * plane + j * nx + i;
    const int cm0 = (t.z0 == 0) ? c + (nz - 1) * plane : c - plane;
    double x_m = x[cm0], x_c = x[c], tz_m = Tz[cm0];
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const int cp = (k == nz - 1) ? c - (nz - 1) * plane : c + plane;
      const double x_p = x[cp], tz_c = Tz[c];
      const double off = Tx[c] * x[c + dxp] + Tx[c + dxm] * x[c + dxm] + Ty[c] * x[c + dyp] +
                         Ty[c + dym] * x[c + dym] + tz_c * x_p + tz_m * x_m;
      const double r = stream_in<NT>(&P.b[c]) - (stream_in<NT>(&L.diag[c]) * x_c - off);
      stream_out<NT>(&rv[c], r);
      rr += r * r;
      tz_m = tz_c;
      x_m = x_c;
      x_c = x_p;
      c = cp;
    }
  }
  write_partials(T, tid, rr, 0.0);
}

// Galerkin warm guess, once FIN_BB has solved for c: x0 = c1 dE(n) + c2
// dE(n-1), formed at the cell and its neighbours on the fly, and r = b - A x0
// with the assembled FP64 operator; partial ||r||^2 for FIN_WARM.
template <bool NT>
__global__ __launch_bounds__(kBlock) void k_warm_x(Tables T, TileList TL) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  const StepDev S = T.sd[t.prob];
  if (!warm_due(sc) || !(S.warm > 1.0) || sc.phase != PH_ITER || sc.cold) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const double c1 = sc.c1, c2 = sc.c2;
  const double *__restrict__ h1 = S.h1;
  const double *__restrict__ h2 = S.h2;
  auto g = [&](int q) { return h2 ? c1 * h1[q] + c2 * h2[q] : c1 * h1[q]; };
  const double *__restrict__ Tx = L.Tx;
  const double *__restrict__ Ty = L.Ty;
  const double *__restrict__ Tz = L.Tz;
  double *__restrict__ rv = rcur(P, sc);
  const Col col = tile_col(t);
  double rr = 0.0;
  if (col.on) {
    const int nx = L.nx, ny = L.ny, nz = L.nz, plane = nx * ny;
    const int i = col.i, j = col.j;
    const int dxm = (i == 0) ? nx - 1 : -1, dxp = (i == nx - 1) ? 1 - nx : 1;
    const int dym = (j == 0) ? (ny - 1) * nx : -nx;
    const int dyp = (j == ny - 1) ? -(ny - 1) * nx : nx;
    int c = t.z0 * plane + j * nx + i;
    const int cm0 = (t.z0 == 0) ? c + (nz - 1) * plane : c - plane;
    double x_m = g(cm0), x_c = g(c), tz_m = Tz[cm0];
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const int cp = (k == nz - 1) ? c - (nz - 1) * plane : c + plane;
      const double x_p = g(cp);
      const double off = Tx[c] * g(c + dxp) + Tx[c + dxm] * g(c + dxm) +
                         Ty[c] * g(c + dyp) + Ty[c + dym] * g(c + dym) +
                         Tz[c] * x_p + tz_m * x_m;
      const double r = stream_in<NT>(&P.b[c]) - (stream_in<NT>(&L.diag[c]) * x_c - off);
      stream_out<NT>(&P.x[c], x_c);
      stream_out<NT>(&rv[c], r);
      rr += r * r;
      tz_m = Tz[c];
      x_m = x_c;
      x_c = x_p;
      c = cp;
    }
  }
  write_partials(T, tid, rr, 0.0);
}

// Local smoothing.  Where a cell's coupling to its neighbours dominates its
// diagonal (an ionized bubble: little absorption, D near D_max, so the cell
// is almost a pure diffusion cell), one red/black sweep leaves the error that
// is smooth inside the bubble nearly untouched and the coarse levels, whose
// cells mix bubble and neutral children, do not represent it; extra sweeps
// restricted to those cells act on it at a small fraction of a full sweep's
// cost.  k_assemble marks them from the FP64 finest operator and lists them
// per tile and colour (list_cells); k_local runs one half-sweep of colour
// `colour` over a tile's listed cells, in place in the cycle's FP32 output
// z32, with the cycle's scaled right-hand side and FP32 coefficients, and
// records the change of r.z that the update makes (r the FP64 residual the
// cycle ran on, z = s z32).
//
// The list of a tile lives in llist at the tile's own cells: entry q (the
// colour-0 cells first, then the colour-1 cells, each in thread and plane
// order) is stored at the q-th cell of the tile's box in x, y, z order, so
// tiles never overlap and one wave reads 64 consecutive entries.  lcnt[2u],
// lcnt[2u + 1]: the counts per colour of the problem's finest tile u (held
// with the problem: a server rebuilds its tables between the assembly and
// the sweeps).  Within one colour the updates are independent (a cell of
// that colour reads only cells of the other), so k_local gives every listed
// cell a thread of its own.

__global__ __launch_bounds__(kBlock) void k_local(Tables T, TileList TL, int colour) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (!sc.active) return;
  const ProbDev P = T.pd[t.prob];
  // the counts come from the assembly; bounded by the tile's box all the same, so
  // that no read of the list can leave the tile's own cells
  const int u = tid - P.t0, box = t.tx * t.ty * t.tz;
  const int first = colour ? min(max(P.lcnt[2 * u], 0), box) : 0;
  const int cnt = min(max(P.lcnt[2 * u + colour], 0), box - first);
  if (cnt == 0) {
    if (threadIdx.x == 0) T.lpart[2 * tid + colour] = 0.0;
    return;
  }
  const LevelDev L = T.lv[t.prob];
  const Coef<float> C = coefs<float>(L);
  const double *r = rcur(P, sc);
  const double inv_s = sc.inv_s, s = sc.s;
  float *z = znext(P, sc);
  const int plane = L.nx * L.ny;
  double dz = 0.0;
  for (int q = threadIdx.x; q < cnt; q += kBlock) {
    const int c = P.llist[box_cell(t, first + q, L.nx, L.ny)];
    if ((unsigned)c >= (unsigned)(plane * L.nz)) continue;  // not a cell
    const int k = c / plane, rm = c - k * plane, j = rm / L.nx;
    const Nb n = nbrs(rm - j * L.nx, j, k, L.nx, L.ny, L.nz);
    const float f = (float)(r[n.c] * inv_s);
    const float sum = C.tx[n.c] * z[n.xp] + C.tx[n.xm] * z[n.xm] +
                      C.ty[n.c] * z[n.yp] + C.ty[n.ym] * z[n.ym] +
                      C.tz[n.c] * z[n.zp] + C.tz[n.zm] * z[n.zm];
    const float xn = (f + sum) * recip(C.d[n.c]);
    const float xo = z[n.c];
    z[n.c] = xn;
    dz += r[n.c] * (s * ((double)xn - (double)xo));
  }
  __shared__ double sh[kBlock / 64];
  const double w = wave_total(dz);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = w;
  __syncthreads();
  if (threadIdx.x == 0) {
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < kBlock / 64; ++i) v += sh[i];
    T.lpart[2 * tid + colour] = v;
  }
}

// Warm-started problems whose guess was dropped (by FIN_BB or FIN_WARM: it
// did not reduce the residual): x = 0, r = b.  And b = 0: the solution is 0
// whatever the guess.
__global__ __launch_bounds__(kBlock) void k_warm_revert(Tables T, TileList TL) {
  const Tile t = get_tile(TL);
  const Scal &sc = T.sc[t.prob];
  if (!warm_due(sc) || !(T.sd[t.prob].warm > 0.0)) return;
  const bool zero_b = sc.phase == PH_DONE && sc.status == ST_OK;
  if (!zero_b && !(sc.phase == PH_ITER && sc.cold)) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  double *rv = rcur(P, sc);
  const Col col = tile_col(t);
  if (!col.on) return;
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    const int c0 = (k * L.ny + col.j) * L.nx + col.i;
    P.x[c0] = 0.0;
    rv[c0] = P.b[c0];
  }
}

// out = A u (single problem, inspection entry point)
__global__ __launch_bounds__(kBlock) void k_apply(Tables T, TileList TL,
                                                  const double *u, double *out) {
  const Tile t = get_tile(TL);
  const LevelDev L = T.lv[t.prob];
  const Coef<double> C = coefs<double>(L);
  const Col col = tile_col(t);
  if (!col.on) return;
  auto uv = [&](int q) { return u[q]; };
  for (int k = t.z0; k < t.z0 + t.tz; ++k) {
    const Nb n = nbrs(col.i, col.j, k, L.nx, L.ny, L.nz);
    out[n.c] = C.d[n.c] * u[n.c] - offsum(C, n, uv);
  }
}

// load an external residual (preconditioner entry point): r = given, ||r||^2
__global__ __launch_bounds__(kBlock) void k_set_r(Tables T, TileList TL,
                                                  const double *rin) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  double *rv = rcur(P, sc);
  const Col col = tile_col(t);
  double rr = 0.0;
  if (col.on) {
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const int c0 = (k * L.ny + col.j) * L.nx + col.i;
      const double r = rin[c0];
      rv[c0] = r;
      rr += r * r;
    }
  }
  write_partials(T, tid, rr, 0.0);
}

// E_out = E + dE with the relative-change sum (dE / max(|E_out|, floor))^2
// and ||dE||^2; copy_only: E_out = dE (solve entry point).
// in_solve: launched right after the verification; acts only on problems it
// just decided (done, ok, not yet committed)
__device__ __forceinline__ bool commit_now(const Scal &sc) {
  return sc.live && sc.phase == PH_DONE && sc.status == ST_OK && !sc.committed;
}

template <bool NT>
__global__ __launch_bounds__(kBlock) void k_update_E(Tables T, TileList TL,
                                                     double floor,
                                                     int copy_only, int in_solve) {
  int tid;
  const Tile t = get_tile(TL, tid);
  const Scal &sc = T.sc[t.prob];
  if (in_solve ? !commit_now(sc) : !sc.live) return;
  const LevelDev L = T.lv[t.prob];
  const ProbDev P = T.pd[t.prob];
  const StepDev S = T.sd[t.prob];
  const Col col = tile_col(t);
  double ch = 0.0, dd = 0.0;
  if (col.on) {
    for (int k = t.z0; k < t.z0 + t.tz; ++k) {
      const int c0 = (k * L.ny + col.j) * L.nx + col.i;
      const int c = c0;
      const double d = P.x[c];
      dd += d * d;
      if (copy_only) {
        stream_out<NT>(&S.Eout[c], d);
      } else {
        const double en = stream_in<NT>(&S.E[c]) + d;
        stream_out<NT>(&S.Eout[c], en);
        double w = fabs(en);
        w = (w < floor) ? floor : w;
        if (w > 0.0) {
          const double q = d / w;
          ch += q * q;
        }
      }
    }
  }
  write_partials(T, tid, ch, dd);
}

// ---------------------------------------------------------------------------
// per-problem finalize: sum the tile partials in tile order, update scalars
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool finite(double v) { return isfinite(v); }

__device__ __forceinline__ void set_scale(Scal &sc, int n, int mixed) {
  double s = 1.0;
  if (mixed) {
    s = sqrt(sc.rr / (double)n);
    if (!(s > 0.0) || !finite(s)) s = 1.0;
  }
  sc.s = s;
  sc.inv_s = 1.0 / s;
}

__device__ __forceinline__ void fail(Scal &sc, int status) {
  sc.status = status;
  sc.phase = PH_DONE;
  sc.active = 0;
}

// FIN_BB: the assembly's sums (in tile order), the start of the solve and,
// for a warm start, the guess: the extrapolated one is kept if it reduces
// the residual; the Galerkin one gets its coefficients here (k_warm_x then
// forms it and FIN_WARM applies the same test)
__global__ __launch_bounds__(kFinBlock) void k_fin_bb(Tables T, int mixed) {
  const int p = blockIdx.x;
  Scal &sc = T.sc[p];
  if (!asm_due(sc)) return;
  const ProbDev &P = T.pd[p];
  double a[kAsmSums];
#pragma unroll
  for (int i = 0; i < kAsmSums; ++i) a[i] = 0.0;
  for (int t = P.t0 + (int)threadIdx.x; t < P.t1; t += kFinBlock) {
#pragma unroll
    for (int i = 0; i < kAsmSums; ++i) a[i] += T.gpart[kAsmSums * t + i];
  }
  constexpr int NW = kFinBlock / 64;
  __shared__ double sh[kAsmSums][NW];
#pragma unroll
  for (int i = 0; i < kAsmSums; ++i) {
    const double w = wave_total(a[i]);
    if ((threadIdx.x & 63) == 0) sh[i][threadIdx.x >> 6] = w;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
#pragma unroll
  for (int i = 0; i < kAsmSums; ++i) a[i] = row_total(sh[i][threadIdx.x & (NW - 1)]);
  if (threadIdx.x != 0) return;
  const double bb = a[AS_BB];
  sc.bb = bb;
  sc.rr = bb;
  sc.rr_true = bb;
  sc.iter = 0;
  sc.restart = 1;
  sc.restarts = 0;
  sc.pbuf = 0;
  sc.has_dir = sc.xlag = sc.snew = 0;
  sc.lag = sc.hasb = sc.zbuf = 0;
  sc.fresh = 1;
  sc.committed = 0;
  sc.status = ST_OK;
  sc.phase = PH_ITER;
  sc.active = 1;
  sc.cold = 0;
  const double warm = T.sd[p].warm;
  if (!finite(bb)) {
    fail(sc, ST_ENONFINITE);
  } else if (bb == 0.0) {
    sc.phase = PH_DONE;
    sc.active = 0;
  } else if (warm > 1.0) {
    // (h_i, A h_j) c = (h_i, b): the A-norm-closest point of span{h} to the
    // solution; one vector when the pair is (nearly) dependent or absent
    const double g11 = a[AS_G11], g12 = a[AS_G12], g22 = a[AS_G22];
    const double b1 = a[AS_B1], b2 = a[AS_B2];
    const double det = g11 * g22 - g12 * g12;
    double c1 = 0.0, c2 = 0.0;
    bool ok = g11 > 0.0 && finite(g11) && finite(b1);
    if (ok && T.sd[p].h2 && g22 > 0.0 && det > 1e-10 * g11 * g22 &&
        finite(g12) && finite(g22) && finite(b2)) {
      c1 = (b1 * g22 - b2 * g12) / det;
      c2 = (b2 * g11 - b1 * g12) / det;
    } else if (ok) {
      c1 = b1 / g11;
    }
    ok = ok && finite(c1) && finite(c2);
    sc.c1 = c1;
    sc.c2 = c2;
    sc.cold = !ok;
  } else if (warm > 0.0) {
    // PCG from the warm guess (same ||b||), or from 0 (k_warm_revert)
    // if the guess does not reduce the residual
    const double rr = a[AS_RR];
    sc.cold = !(rr < bb);
    if (!sc.cold) sc.rr = rr;
    if (!finite(rr)) fail(sc, ST_ENONFINITE);
  }
  set_scale(sc, P.n, mixed);
  if (sc.ctl) sc.stage = 2;  // device-controlled: the warm start is next
}

__global__ __launch_bounds__(kFinBlock) void k_fin(Tables T, int which, int mixed,
                                                  int alt) {
  const int p = blockIdx.x;
  Scal &sc = T.sc[p];
  const ProbDev P = T.pd[p];
  // partials of the fused tiles: the fused cycle's r.z, the down pass's
  // ||r||^2 and the fused iteration's SpMV
  const bool fz = (alt && which == FIN_RZ) || (alt && which == FIN_PQ && P.spf) ||
                  which == FIN_RR2;
  const int t0 = fz ? P.f0 : P.t0;
  const int t1 = (which == FIN_XFIX) ? t0 : (fz ? P.f1 : P.t1);
  // state changes that need no sums ride along (a launch each would cost as
  // much as the sums): in a device-controlled unit the warm start is behind
  // the first cycle, and x is up to date once the true residual is formed
  if (which == FIN_RZ && threadIdx.x == 0 && sc.ctl && sc.stage == 2) sc.stage = 0;
  if (which == FIN_TRUE && alt && threadIdx.x == 0 && sc.xlag && sc.phase != PH_ITER)
    sc.xlag = sc.lag = sc.hasb = 0;
  bool part;
  switch (which) {
    case FIN_STEP: part = alt ? commit_now(sc) : sc.live != 0; break;
    case FIN_TRUE: part = sc.phase == PH_VERIFY; break;
    case FIN_SETR: part = true; break;
    case FIN_RR2: part = sc.active && sc.has_dir; break;
    case FIN_XFIX: part = sc.xlag && sc.phase != PH_ITER; break;
    case FIN_WARM:
      part = warm_due(sc) && T.sd[p].warm > 1.0 && sc.phase == PH_ITER && !sc.cold;
      break;
    default: part = sc.active != 0; break;
  }
  if (!part) return;
  // independent loads in flight: 4 per thread per round, summed in order
  double a0 = 0.0, a1 = 0.0;
  if (which == FIN_RZ && alt == 2) {
    // r.z changes of the local sweeps (black, red), per finest tile
    for (int t = P.t0 + (int)threadIdx.x; t < P.t1; t += kFinBlock)
      a0 += T.lpart[2 * t] + T.lpart[2 * t + 1];
  }
  int t = t0 + (int)threadIdx.x;
  for (; t + 3 * kFinBlock < t1; t += 4 * kFinBlock) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      v[2 * u] = T.part[2 * (t + u * kFinBlock)];
      v[2 * u + 1] = T.part[2 * (t + u * kFinBlock) + 1];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a0 += v[2 * u];
      a1 += v[2 * u + 1];
    }
  }
  for (; t < t1; t += kFinBlock) {
    a0 += T.part[2 * t];
    a1 += T.part[2 * t + 1];
  }
  constexpr int NW = kFinBlock / 64;
  __shared__ double sh[2][NW];
  a0 = wave_total(a0);
  a1 = wave_total(a1);
  const int lane = threadIdx.x & 63;
  if (lane == 0) {
    sh[0][threadIdx.x >> 6] = a0;
    sh[1][threadIdx.x >> 6] = a1;
  }
  __syncthreads();
  if (threadIdx.x >= 64) return;
  a0 = row_total(sh[0][lane & (NW - 1)]);
  a1 = row_total(sh[1][lane & (NW - 1)]);
  if (threadIdx.x != 0) return;
  switch (which) {
    case FIN_RZ: {
      sc.rho = a0;
      sc.rzo = a1;
      sc.fresh = 0;  // (the finest down pass is done)
      // (a failed solve keeps the z and the scale that its pending update of
      // x is formed from)
      if (!finite(a0) || !finite(a1)) { fail(sc, ST_ENONFINITE); break; }
      if (!(a0 > 0.0)) { fail(sc, ST_ENOCONV); break; }
      sc.zscale1 = sc.zscale;
      sc.zscale = sc.s;  // the scale z was just formed with
      if (alt) sc.zbuf ^= 1;  // the fused cycle wrote the other buffer
      double beta = 0.0;
      if (!sc.restart) beta = mixed ? (a0 - a1) / sc.rho_old : a0 / sc.rho_old;
      sc.beta1 = sc.beta;
      sc.beta = beta;
      sc.restart = 0;
      sc.rho_old = a0;
      break;
    }
    case FIN_PQ:
      sc.pq = a0;
      // (fused iteration: the SpMV that stores also brings x up to date)
      if (alt && sc.lag) sc.xlag = 0;
      if (!finite(a0)) { fail(sc, ST_ENONFINITE); break; }
      if (!(a0 > 0.0)) { fail(sc, ST_ENOCONV); break; }
      sc.alpha1 = sc.alpha;
      sc.alpha = sc.rho / a0;
      if (alt && !sc.lag) {
        sc.lag = 1;
      } else {
        sc.pscale = sc.zscale;  // the direction just stored has z's scale
        sc.pbuf ^= 1;
        sc.lag = 0;
        sc.hasb = alt;
      }
      if (alt) {
        // fused iteration: r -= alpha q happens in the next down pass, x +=
        // alpha p in a later SpMV; the V-cycle scale changes between cycles
        sc.has_dir = 1;
        sc.xlag = 1;
        if (sc.snew) {
          sc.s = sc.s_next;
          sc.inv_s = 1.0 / sc.s_next;
          sc.snew = 0;
        }
      }
      break;
    case FIN_RR2:
      sc.rr = a0;
      sc.iter += 1;
      sc.rbuf ^= 1;  // the down pass wrote r - alpha q to the other buffer
      if (!finite(a0)) { fail(sc, ST_ENONFINITE); break; }
      if (a0 <= sc.tol2 * sc.bb) {
        sc.phase = PH_VERIFY;
        sc.active = 0;
      } else if (sc.iter >= sc.max_iter) {
        fail(sc, ST_ENOCONV);
      }
      {
        // scale of the next V-cycle (this one already uses the current s)
        const double s0 = sc.s, i0 = sc.inv_s;
        set_scale(sc, P.n, mixed);
        sc.s_next = sc.s;
        sc.s = s0;
        sc.inv_s = i0;
        sc.snew = 1;
      }
      break;
    case FIN_XFIX:
      sc.xlag = sc.lag = sc.hasb = 0;
      break;
    case FIN_WARM:
      // keep the projected guess only if it reduces the residual (else
      // k_warm_revert starts from 0)
      sc.cold = !(a0 < sc.bb);
      if (!finite(a0)) { fail(sc, ST_ENONFINITE); break; }
      if (!sc.cold) {
        sc.rr = a0;
        set_scale(sc, P.n, mixed);
      }
      break;
    case FIN_RR:
      sc.rr = a0;
      sc.iter += 1;
      if (!finite(a0)) { fail(sc, ST_ENONFINITE); break; }
      if (a0 <= sc.tol2 * sc.bb) {
        sc.phase = PH_VERIFY;
        sc.active = 0;
      } else if (sc.iter >= sc.max_iter) {
        fail(sc, ST_ENOCONV);
      }
      set_scale(sc, P.n, mixed);
      break;
    case FIN_TRUE:
      sc.rr_true = a0;
      sc.rr = a0;
      if (!finite(a0)) { fail(sc, ST_ENONFINITE); break; }
      if (a0 <= sc.tol2 * sc.bb) {
        sc.status = ST_OK;
        sc.phase = PH_DONE;
        sc.active = 0;
      } else if (sc.iter < sc.max_iter) {
        sc.phase = PH_ITER;
        sc.active = 1;
        sc.restart = 1;
        sc.restarts += 1;
        sc.has_dir = sc.snew = 0;
        sc.lag = sc.hasb = 0;
        sc.fresh = 1;
        set_scale(sc, P.n, mixed);
      } else {
        fail(sc, ST_ENOCONV);
      }
      break;
    case FIN_STEP:
      sc.change2 = a0;
      sc.dEdE = a1;
      sc.committed = 1;
      break;
    case FIN_SETR:
      sc.rr = a0;
      sc.active = 1;
      sc.phase = PH_ITER;
      sc.has_dir = sc.xlag = sc.snew = sc.fresh = 0;
      sc.lag = sc.hasb = sc.zbuf = 0;
      set_scale(sc, P.n, mixed);
      break;
  }
}

// ---------------------------------------------------------------------------
// per-kernel timing hook (include/fld_profile.h)
// ---------------------------------------------------------------------------

static const char *kKernelNames[K_NUM] = {
    "assemble", "coarsen", "fin", "pre0_fine", "pre0_coarse", "half_fine",
    "half_coarse", "half_out", "resid_restrict_fine", "resid_restrict_coarse",
    "prolong_black_fine", "prolong_black_coarse", "coarse_solve", "spmv_p",
    "update", "true_resid", "apply", "set_r", "update_E", "vdown_fine",
    "vdown_coarse", "vup_fine", "vup_coarse", "chem_h", "ionized_sum",
    "warm_revert", "jacobi0_fine", "jacobi_fine", "jacobi_out",
    "jacobi_coarse", "prolong_add_fine", "prolong_add_coarse", "spmv_px",
    "xfix", "warm_x", "local", "control", "copy_E", "update_r"};

namespace prof {
struct Rec {
  hipEvent_t a, b;
  int k;
};
static int sel = -1;
static std::vector<Rec> recs;
static std::vector<hipEvent_t> pool;

static hipEvent_t get() {
  if (!pool.empty()) {
    hipEvent_t e = pool.back();
    pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

static bool on(int k, hipStream_t s) {
  if (!(sel == k || sel == -2)) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone)
    return false;
  return true;
}

}  // namespace prof

ProfScope::ProfScope(int k_, hipStream_t s_) : k(k_), s(s_), a(nullptr) {
  if (prof::on(k, s)) {
    a = prof::get();
    if (a) hipEventRecord(a, s);
  }
}

ProfScope::~ProfScope() {
  if (!a) return;
  hipEvent_t b = prof::get();
  if (!b) return;
  hipEventRecord(b, s);
  prof::recs.push_back({a, b, k});
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------

#define LAUNCH FLD_LAUNCH

void launch_assemble(const Tables &T, TileList L0, double c, double theta,
                     double dmax, double rmin, int mixed, int local,
                     double coupling, hipStream_t s) {
  if (!L0.nblocks) return;
  with_stream(T, [&](auto nt) {
    LAUNCH(K_ASSEMBLE, k_assemble<nt()>, L0.nblocks, kBlock, s, T, L0, c, theta, dmax, rmin, mixed, local, coupling);
  });
}

void launch_coarsen(const Tables &T, TileList LC, int lc, double scale,
                    int mixed, int op, hipStream_t s) {
  if (LC.nblocks) LAUNCH(K_COARSEN, k_coarsen, LC.nblocks, kBlock, s, T, LC, lc, scale, mixed, op);
}

void launch_fin(const Tables &T, int which, int mixed, hipStream_t s, int alt) {
  if (!T.nprob) return;
  if (which == FIN_BB) LAUNCH(K_FIN, k_fin_bb, T.nprob, kFinBlock, s, T, mixed);
  else LAUNCH(K_FIN, k_fin, T.nprob, kFinBlock, s, T, which, mixed, alt);
}

void launch_pre0(const Tables &T, TileList L, int l, int prec, hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l == 0 ? K_PRE0_F : K_PRE0_C;
  if (prec) {
    if (l == 0) LAUNCH(id, (k_pre0<float, true>), L.nblocks, kBlock, s, T, L, l);
    else LAUNCH(id, (k_pre0<float, false>), L.nblocks, kBlock, s, T, L, l);
  } else {
    if (l == 0) LAUNCH(id, (k_pre0<double, true>), L.nblocks, kBlock, s, T, L, l);
    else LAUNCH(id, (k_pre0<double, false>), L.nblocks, kBlock, s, T, L, l);
  }
}

void launch_half(const Tables &T, TileList L, int l, int colour, int prec,
                 hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l == 0 ? K_HALF_F : K_HALF_C;
  if (prec) {
    if (l == 0) LAUNCH(id, (k_half<float, true>), L.nblocks, kBlock, s, T, L, l, colour);
    else LAUNCH(id, (k_half<float, false>), L.nblocks, kBlock, s, T, L, l, colour);
  } else {
    if (l == 0) LAUNCH(id, (k_half<double, true>), L.nblocks, kBlock, s, T, L, l, colour);
    else LAUNCH(id, (k_half<double, false>), L.nblocks, kBlock, s, T, L, l, colour);
  }
}

void launch_half_out(const Tables &T, TileList L0, int prec, int flexible,
                     hipStream_t s) {
  if (!L0.nblocks) return;
  if (prec) LAUNCH(K_HALF_OUT, (k_half_out<float>), L0.nblocks, kBlock, s, T, L0, flexible);
  else LAUNCH(K_HALF_OUT, (k_half_out<double>), L0.nblocks, kBlock, s, T, L0, flexible);
}

void launch_resid_restrict(const Tables &T, TileList LC, int lc, int prec,
                           hipStream_t s) {
  if (!LC.nblocks) return;
  const int id = lc == 1 ? K_RESTRICT_F : K_RESTRICT_C;
  if (prec) {
    if (lc == 1) LAUNCH(id, (k_resid_restrict<float, true>), LC.nblocks, kBlock, s, T, LC, lc);
    else LAUNCH(id, (k_resid_restrict<float, false>), LC.nblocks, kBlock, s, T, LC, lc);
  } else {
    if (lc == 1) LAUNCH(id, (k_resid_restrict<double, true>), LC.nblocks, kBlock, s, T, LC, lc);
    else LAUNCH(id, (k_resid_restrict<double, false>), LC.nblocks, kBlock, s, T, LC, lc);
  }
}

void launch_prolong_black(const Tables &T, TileList L, int l, int prec,
                          int trilinear, hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l == 0 ? K_PROLONG_F : K_PROLONG_C;
  if (prec) {
    if (l == 0) LAUNCH(id, (k_prolong_black<float, true>), L.nblocks, kBlock, s, T, L, l, trilinear);
    else LAUNCH(id, (k_prolong_black<float, false>), L.nblocks, kBlock, s, T, L, l, trilinear);
  } else {
    if (l == 0) LAUNCH(id, (k_prolong_black<double, true>), L.nblocks, kBlock, s, T, L, l, trilinear);
    else LAUNCH(id, (k_prolong_black<double, false>), L.nblocks, kBlock, s, T, L, l, trilinear);
  }
}

void launch_spmv_f(const Tables &T, TileList F0, int km, hipStream_t s) {
  if (!F0.nblocks) return;
  if (km == KM_MIX64) LAUNCH(K_SPMV_PX, k_spmv_f<KM_MIX64>, F0.nblocks, kBlock, s, T, F0);
  else LAUNCH(K_SPMV_PX, k_spmv_f<KM_MIX32>, F0.nblocks, kBlock, s, T, F0);
}

void launch_spmv_p(const Tables &T, TileList L0, int lazy, int km, hipStream_t s) {
  if (!L0.nblocks) return;
  with_stream(T, [&](auto nt) {
    if (lazy && km == KM_FP64) LAUNCH(K_SPMV_PX, (k_spmv_p<true, KM_FP64, nt()>), L0.nblocks, kBlock, s, T, L0);
    else if (lazy && km == KM_MIX64) LAUNCH(K_SPMV_PX, (k_spmv_p<true, KM_MIX64, nt()>), L0.nblocks, kBlock, s, T, L0);
    else if (lazy) LAUNCH(K_SPMV_PX, (k_spmv_p<true, KM_MIX32, nt()>), L0.nblocks, kBlock, s, T, L0);
    else if (km == KM_MIX64) LAUNCH(K_SPMV_P, (k_spmv_p<false, KM_MIX64, nt()>), L0.nblocks, kBlock, s, T, L0);
    else if (km == KM_MIX32) LAUNCH(K_SPMV_P, (k_spmv_p<false, KM_MIX32, nt()>), L0.nblocks, kBlock, s, T, L0);
    else LAUNCH(K_SPMV_P, (k_spmv_p<false, KM_FP64, nt()>), L0.nblocks, kBlock, s, T, L0);
  });
}

void launch_z_out(const Tables &T, TileList L0, int fused, double *out, hipStream_t s) {
  if (L0.nblocks) LAUNCH(K_APPLY, k_z_out, L0.nblocks, kBlock, s, T, L0, fused, out);
}

void launch_xfix(const Tables &T, TileList L0, int km, hipStream_t s) {
  if (!L0.nblocks) return;
  if (km == KM_MIX32) LAUNCH(K_XFIX, k_xfix<KM_MIX32>, L0.nblocks, kBlock, s, T, L0);
  else if (km == KM_MIX64) LAUNCH(K_XFIX, k_xfix<KM_MIX64>, L0.nblocks, kBlock, s, T, L0);
  else LAUNCH(K_XFIX, k_xfix<KM_FP64>, L0.nblocks, kBlock, s, T, L0);
}

void launch_update(const Tables &T, TileList L0, int km, int r_only, hipStream_t s) {
  if (!L0.nblocks) return;
  with_stream(T, [&](auto nt) {
    if (r_only) LAUNCH(K_UPDATE_R, (k_update<KM_FP64, false, nt()>), L0.nblocks, kBlock, s, T, L0);
    else if (km == KM_MIX32) LAUNCH(K_UPDATE, (k_update<KM_MIX32, true, nt()>), L0.nblocks, kBlock, s, T, L0);
    else if (km == KM_MIX64) LAUNCH(K_UPDATE, (k_update<KM_MIX64, true, nt()>), L0.nblocks, kBlock, s, T, L0);
    else LAUNCH(K_UPDATE, (k_update<KM_FP64, true, nt()>), L0.nblocks, kBlock, s, T, L0);
  });
}

void launch_true_resid(const Tables &T, TileList L0, hipStream_t s) {
  if (!L0.nblocks) return;
  with_stream(T, [&](auto nt) {
    LAUNCH(K_TRUE_RESID, k_true_resid<nt()>, L0.nblocks, kBlock, s, T, L0);
  });
}


void launch_local(const Tables &T, TileList L0, int colour, hipStream_t s) {
  if (L0.nblocks) LAUNCH(K_LOCAL, k_local, L0.nblocks, kBlock, s, T, L0, colour);
}

void launch_warm_x(const Tables &T, TileList L0, hipStream_t s) {
  if (!L0.nblocks) return;
  with_stream(T, [&](auto nt) {
    LAUNCH(K_WARM_X, k_warm_x<nt()>, L0.nblocks, kBlock, s, T, L0);
  });
}

void launch_apply(const Tables &T, TileList L0, const double *u, double *out,
                  hipStream_t s) {
  if (L0.nblocks) LAUNCH(K_APPLY, k_apply, L0.nblocks, kBlock, s, T, L0, u, out);
}

void launch_set_r(const Tables &T, TileList L0, const double *r, int prec,
                  hipStream_t s) {
  (void)prec;
  if (L0.nblocks) LAUNCH(K_SET_R, k_set_r, L0.nblocks, kBlock, s, T, L0, r);
}


void launch_jacobi(const Tables &T, TileList L, int l, int prec, int mode,
                   int in_x2, int flexible, hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l ? K_JACOBI_C : mode == 0 ? K_JACOBI0_F : mode == 1 ? K_JACOBI_F : K_JACOBI_OUT;
  if (prec) {
    if (l == 0) LAUNCH(id, (k_jacobi<float, true>), L.nblocks, kBlock, s, T, L, l, mode, in_x2, flexible);
    else LAUNCH(id, (k_jacobi<float, false>), L.nblocks, kBlock, s, T, L, l, mode, in_x2, flexible);
  } else {
    if (l == 0) LAUNCH(id, (k_jacobi<double, true>), L.nblocks, kBlock, s, T, L, l, mode, in_x2, flexible);
    else LAUNCH(id, (k_jacobi<double, false>), L.nblocks, kBlock, s, T, L, l, mode, in_x2, flexible);
  }
}

void launch_prolong_add(const Tables &T, TileList L, int l, int prec,
                        int trilinear, int to_x2, hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l ? K_PROLONG_ADD_C : K_PROLONG_ADD_F;
  if (prec) LAUNCH(id, k_prolong_add<float>, L.nblocks, kBlock, s, T, L, l, trilinear, to_x2);
  else LAUNCH(id, k_prolong_add<double>, L.nblocks, kBlock, s, T, L, l, trilinear, to_x2);
}

void launch_warm_revert(const Tables &T, TileList L0, hipStream_t s) {
  if (L0.nblocks) LAUNCH(K_WARM_REVERT, k_warm_revert, L0.nblocks, kBlock, s, T, L0);
}

void launch_update_E(const Tables &T, TileList L0, double floor, int copy_only,
                     hipStream_t s, int in_solve) {
  if (!L0.nblocks) return;
  with_stream(T, [&](auto nt) {
    LAUNCH(K_UPDATE_E, k_update_E<nt()>, L0.nblocks, kBlock, s, T, L0, floor, copy_only,
           in_solve);
  });
}

}  // namespace fld

extern "C" {

int32_t fld_profile_num_kernels(void) { return fld::K_NUM; }

const char *fld_profile_kernel_name(int32_t k) {
  return (k >= 0 && k < fld::K_NUM) ? fld::kKernelNames[k] : nullptr;
}

int32_t fld_profile_select(int32_t k) {
  if (k < -2 || k >= fld::K_NUM) return -1;
  for (auto &r : fld::prof::recs) {
    hipEventSynchronize(r.b);
    fld::prof::pool.push_back(r.a);
    fld::prof::pool.push_back(r.b);
  }
  fld::prof::recs.clear();
  fld::prof::sel = k;
  return 0;
}

int32_t fld_profile_read(int32_t k, double *total_ms, int64_t *launches) {
  if (k < 0 || k >= fld::K_NUM) return -1;
  double tot = 0.0;
  int64_t cnt = 0;
  for (auto &r : fld::prof::recs) {
    if (r.k != k) continue;
    if (hipEventSynchronize(r.b) != hipSuccess) return -1;
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, r.a, r.b) != hipSuccess) return -1;
    tot += ms;
    ++cnt;
  }
  if (total_ms) *total_ms = tot;
  if (launches) *launches = cnt;
  return 0;
}

}  // extern "C"
