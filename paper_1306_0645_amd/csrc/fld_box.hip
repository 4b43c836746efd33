// One-sweep V-cycle passes for levels that do not fill the GPU: a block does
// a small box of the level (up to 512 cells, 16 x 8 x 4 where the level is not
// thin) at once instead of marching through planes.
//
// The algebra is that of the marching passes (x = 0 on entry, one red/black
// sweep before and one black/red sweep after the coarse-grid correction):
//   down: y = f / d on the box + 2 cells, the black values x_b on the box + 1,
//         the red residuals sum_nb T x_b, summed over the 8 children into the
//         coarse right-hand side (the finest level of the fused PCG iteration
//         forms r - alpha q on the way and writes it for the box's own cells);
//   up:   v = y (+ e at red cells) on the box + 2, the new black values on
//         the box + 1, the new red values, every cell written (the finest
//         level: z and the r.z sums).
// Such a level is bound by latency, not by bytes: a march pays a memory
// latency and two barriers per plane, and a kernel per half-sweep pays a
// launch for each of the four half-sweeps.  Here every load of a thread (the
// haloed right-hand side and diagonal, the coefficients of its black cells
// and of its red cells) is issued before the first barrier, so a pass costs
// one round of memory latency, two barriers and one launch; the halo is read
// again by the neighbouring boxes (3.75 times the cells for a full box) from
// the caches.  The box is no larger, so that the loads in flight leave room
// for three blocks and more per CU (a batch of 23 problems of 32^3 to 128^3,
// FP64: 6157 us a step, 6515 with 16 x 8 x 8, 6182 with 8 x 8 x 4).
#include "fld_device.h"

namespace fld {

constexpr int kBX = kBoxX, kBY = kBoxY, kBZ = kBoxZ;               // the widest box (box_shape:
                                                                  // the others fit its buffers)
constexpr int kYN = (kBX + 4) * (kBY + 4) * (kBZ + 4);             // its + 2 frame
constexpr int kHN = (kBX + 2) / 2 * (kBY + 2) * (kBZ + 2);         // black half of the + 1 frame
constexpr int kYS = (kYN + kBlock - 1) / kBlock, kHS = (kHN + kBlock - 1) / kBlock;
constexpr int kPS = (kBX * kBY * kBZ / 2 + kBlock - 1) / kBlock;    // x-pairs (red cells) per thread
constexpr int kCN = (kBX / 2 + 4) * (kBY / 2 + 4) * (kBZ / 2 + 4); // coarse cells staged (trilinear)
constexpr int kCS = (kCN + kBlock - 1) / kBlock;

// q / d for 0 <= q <= kYN and 1 <= d <= 20 by a multiplication: exact while
// q (m d - 65536) < 65536, m = 65536 / d + 1
struct SmallDiv {
  int d, m;
  __device__ __forceinline__ explicit SmallDiv(int v) : d(v), m(65536 / v + 1) {}
  __device__ __forceinline__ int operator()(int q) const { return (q * m) >> 16; }
};

__device__ __forceinline__ int bwrap(int i, int n) {
  return i < 0 ? i + n : (i >= n ? i - n : i);
}

__device__ __forceinline__ int bmod(int i, int n) {
  const int r = i % n;
  return r < 0 ? r + n : r;
}

// (ex, ey, ez) of entry q of a frame of rows of ax and planes of ay rows
struct Frame {
  SmallDiv ax, ay;
  int n;
  __device__ __forceinline__ Frame(int x, int y, int z) : ax(x), ay(y), n(x * y * z) {}
  __device__ __forceinline__ void at(int q, int &ex, int &ey, int &ez) const {
    const int row = ax(q);
    ex = q - row * ax.d;
    ez = ay(row);
    ey = row - ez * ay.d;
  }
};

// six faces and the diagonal of one cell
template <typename R>
struct Cell7 {
  R xp, xm, yp, ym, zp, zm, d;
};

template <typename R>
__device__ __forceinline__ void load7(Cell7<R> &a, const Coef<R> &C, const Nb &n) {
  a.xp = C.tx[n.c];
  a.xm = C.tx[n.xm];
  a.yp = C.ty[n.c];
  a.ym = C.ty[n.ym];
  a.zp = C.tz[n.c];
  a.zm = C.tz[n.zm];
  a.d = C.d[n.c];
}

// black cell q of the + 1 frame (rows of half cells): frame coordinates; rows
// start at the box's even corner - 1, so cell (ex, ey, ez) of the + 1 frame
// is black where ex + ey + ez is even (the corner (0, 0, 0) has an odd
// coordinate sum).  Cells outside the box in two directions have no red
// neighbour in it: off
__device__ __forceinline__ bool black_cell(const Frame &H, const Tile &t, int q, int &ex,
                                           int &ey, int &ez) {
  int hx;
  H.at(q, hx, ey, ez);
  ex = 2 * hx + ((ey + ez) & 1);
  const int out = (ex == 0 || ex > t.tx) + (ey == 0 || ey > t.ty) + (ez == 0 || ez > t.tz);
  return q < H.n && out <= 1;
}

// x_b = v + (sum_nb T v_nb) / d at offset s of the + 2 frame (rows of ax,
// planes of axy)
template <typename R>
__device__ __forceinline__ R box_black(const Cell7<R> &a, const R *v, int s, int ax, int axy) {
  const R sum = a.xp * v[s + 1] + a.xm * v[s - 1] + a.yp * v[s + ax] + a.ym * v[s - ax] +
                a.zp * v[s + axy] + a.zm * v[s - axy];
  return v[s] + sum * recip(a.d);
}

// sum_nb T x_nb over the black neighbours of the red cell at (ex, ey, ez) of
// the + 1 frame; x holds the black cells of that frame, half rows of hx
template <typename R>
__device__ __forceinline__ R box_red(const Cell7<R> &a, const R *x, int ex, int ey, int ez,
                                     int hx, int hxy) {
  const int row = ez * hxy + ey * hx, h = ex >> 1;
  return a.xp * x[row + ((ex + 1) >> 1)] + a.xm * x[row + ((ex - 1) >> 1)] +
         a.yp * x[row + hx + h] + a.ym * x[row - hx + h] + a.zp * x[row + hxy + h] +
         a.zm * x[row - hxy + h];
}

// u / d for a uniform u (m = 2^32 / d + 1, or 0 for d = 1): scalar operations,
// where the division of two 32-bit numbers takes some 20 dependent ones
__device__ __forceinline__ unsigned box_div(unsigned u, unsigned m) {
  return m ? __umulhi(u, m) : u;
}

// the block's box of level L (unsigned extents of at most 8 bits: the divisions
// by them stay short)
__device__ __forceinline__ Tile get_box(const LevelDev &L, const Range &g) {
  const BoxRec &r = L.box;
  const unsigned u = g.block;
  const unsigned row = box_div(u, r.mx), pl = box_div(row, r.my);
  const unsigned tx = r.ext & 255, ty = r.ext >> 8 & 255, tz = r.ext >> 16 & 255;
  const int x0 = (u - row * r.nbx) * tx, y0 = (row - pl * r.nby) * ty, z0 = pl * tz;
  const int ex = min(tx, (unsigned)(L.nx - x0)), ey = min(ty, (unsigned)(L.ny - y0)),
            ez = min(tz, (unsigned)(L.nz - z0));
  return {g.prob, x0, y0, z0, ex, ey, ez};
}

template <typename R, bool L0>
__global__ __launch_bounds__(kBlock) void k_bdown(Tables T, TileList TL, int l, int sel) {
  using FT = typename FSrc<R, L0>::FT;
  const Range g0 = get_range(TL);
  const Scal &sc = T.sc[g0.prob];
  if (!sc.active) return;
  if ((sel == VD_FRESH && !sc.fresh) || (sel == VD_CONT && sc.fresh)) return;
  const LevelDev L = T.lv[l * T.nprob + g0.prob];
  const ProbDev &P = T.pd[g0.prob];
  const Tile t = get_box(L, g0);
  const bool has_coarse = l + 1 < P.levels;
  const LevelDev &Cv = T.lv[min(l + 1, kMaxLevels - 1) * T.nprob + t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, L0>(L, P, sc);
  const double inv_s = sc.inv_s;
  __shared__ R ys[kYN];
  __shared__ R xs[kHN];
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  constexpr bool kUpd = L0 && sizeof(R) == 4;
  const bool upd = kUpd && sc.has_dir;
  const double alpha = sc.alpha;
  const Frame Y(t.tx + 4, t.ty + 4, t.tz + 4);
  const Frame H((t.tx + 2) >> 1, t.ty + 2, t.tz + 2);
  // every load first: y's sources on the + 2 frame ...
  FT fv[kYS];
  double qv[kUpd ? kYS : 1];
  R dv[kYS];
#pragma unroll
  for (int u = 0; u < kYS; ++u) {
    const int q = threadIdx.x + u * kBlock;
    if (q < Y.n) {
      int ex, ey, ez;
      Y.at(q, ex, ey, ez);
      const int g = (bwrap(t.z0 - 2 + ez, nz) * ny + bwrap(t.y0 - 2 + ey, ny)) * nx +
                    bwrap(t.x0 - 2 + ex, nx);
      fv[u] = f.raw(g);
      dv[u] = C.d[g];
      if constexpr (kUpd) {
        if (upd) qv[u] = P.q[g];
      }
    }
  }
  // ... the coefficients of this thread's black cells ...
  Cell7<R> bc[kHS];
#pragma unroll
  for (int u = 0; u < kHS; ++u) {
    int ex, ey, ez;
    if (black_cell(H, t, threadIdx.x + u * kBlock, ex, ey, ez))
      load7(bc[u], C, nbrs(bwrap(t.x0 - 1 + ex, nx), bwrap(t.y0 - 1 + ey, ny),
                           bwrap(t.z0 - 1 + ez, nz), nx, ny, nz));
  }
  // ... and of its red cells: slot s is red child s & 3 of coarse cell s >> 2
  Cell7<R> rc[kPS];
  const Frame CC(t.tx >> 1, t.ty >> 1, t.tz >> 1);
  const int nred = has_coarse ? 4 * CC.n : 0;
#pragma unroll
  for (int u = 0; u < kPS; ++u) {
    const int s = threadIdx.x + u * kBlock;
    if (s < nred) {
      int I, J, K;
      CC.at(s >> 2, I, J, K);
      const int cy = s & 1, cz = (s >> 1) & 1, cx = cy ^ cz;
      load7(rc[u], C, nbrs(t.x0 + 2 * I + cx, t.y0 + 2 * J + cy, t.z0 + 2 * K + cz, nx, ny, nz));
    }
  }
  double rr = 0.0;
#pragma unroll
  for (int u = 0; u < kYS; ++u) {
    const int q = threadIdx.x + u * kBlock;
    if (q < Y.n) {
      if constexpr (kUpd) {
        if (upd) {
          fv[u] = __builtin_fma(-alpha, qv[u], fv[u]);
          int ex, ey, ez;
          Y.at(q, ex, ey, ez);
          ex -= 2;
          ey -= 2;
          ez -= 2;
          if ((unsigned)ex < (unsigned)t.tx && (unsigned)ey < (unsigned)t.ty &&
              (unsigned)ez < (unsigned)t.tz) {
            rnext(P, sc)[((t.z0 + ez) * ny + t.y0 + ey) * nx + t.x0 + ex] = fv[u];
            rr += fv[u] * fv[u];
          }
        }
      }
      ys[q] = f.scaled(fv[u], inv_s) * recip(dv[u]);
    }
  }
  __syncthreads();
  const int ax = Y.ax.d, axy = Y.ax.d * Y.ay.d, hx = H.ax.d, hxy = H.ax.d * H.ay.d;
#pragma unroll
  for (int u = 0; u < kHS; ++u) {
    const int q = threadIdx.x + u * kBlock;
    int ex, ey, ez;
    if (black_cell(H, t, q, ex, ey, ez))
      xs[q] = box_black(bc[u], ys, (ez + 1) * axy + (ey + 1) * ax + ex + 1, ax, axy);
  }
  __syncthreads();
  R *fc = (R *)Cv.f;
#pragma unroll
  for (int u = 0; u < kPS; ++u) {
    const int s = threadIdx.x + u * kBlock;
    R v = 0;
    int I = 0, J = 0, K = 0;
    if (s < nred) {
      CC.at(s >> 2, I, J, K);
      const int cy = s & 1, cz = (s >> 1) & 1, cx = cy ^ cz;
      v = box_red(rc[u], xs, 2 * I + cx + 1, 2 * J + cy + 1, 2 * K + cz + 1, hx, hxy);
    }
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    if (s < nred && (s & 3) == 0)
      fc[(((t.z0 >> 1) + K) * Cv.ny + (t.y0 >> 1) + J) * Cv.nx + (t.x0 >> 1) + I] = v;
  }
  if constexpr (kUpd) write_partials(T, P.f0 + g0.block, rr, 0.0);
}

template <typename R, bool L0, bool TRI>
__global__ __launch_bounds__(kBlock) void k_bup(Tables T, TileList TL, int l, int flexible) {
  using FT = typename FSrc<R, L0>::FT;
  const Range g0 = get_range(TL);
  const Scal &sc = T.sc[g0.prob];
  if (!sc.active) return;
  const LevelDev L = T.lv[l * T.nprob + g0.prob];
  const ProbDev &P = T.pd[g0.prob];
  const Tile t = get_box(L, g0);
  const bool has_coarse = l + 1 < P.levels;
  const LevelDev Cl = T.lv[min(l + 1, kMaxLevels - 1) * T.nprob + t.prob];
  const Coef<R> C = coefs<R>(L);
  const auto f = fsrc<R, L0>(L, P, sc);
  const double inv_s = sc.inv_s, s_out = sc.s, zs_old = sc.zscale;
  const R *e = (const R *)Cl.x;
  const bool rd_old = flexible && !sc.restart;
  __shared__ R vs[kYN];
  __shared__ R xs[kHN];
  __shared__ R cs[TRI ? kCN : 1];
  const int nx = L.nx, ny = L.ny, nz = L.nz;
  const int cnx = Cl.nx, cny = Cl.ny, cnz = Cl.nz;
  const Frame Y(t.tx + 4, t.ty + 4, t.tz + 4);
  const Frame H((t.tx + 2) >> 1, t.ty + 2, t.tz + 2);
  // trilinear: coarse cells x0 / 2 - 2 .. (x0 + tx) / 2 + 1 (and in y, z), the
  // parents and the interpolation neighbours of the + 2 frame
  const Frame G((t.tx >> 1) + 4, (t.ty >> 1) + 4, (t.tz >> 1) + 4);
  R cv[TRI ? kCS : 1];
  if constexpr (TRI) {
    if (has_coarse) {
#pragma unroll
      for (int u = 0; u < kCS; ++u) {
        const int q = threadIdx.x + u * kBlock;
        if (q < G.n) {
          int ix, iy, iz;
          G.at(q, ix, iy, iz);
          cv[u] = e[(bmod((t.z0 >> 1) - 2 + iz, cnz) * cny + bmod((t.y0 >> 1) - 2 + iy, cny)) *
                        cnx + bmod((t.x0 >> 1) - 2 + ix, cnx)];
        }
      }
    }
  }
  FT fv[kYS];
  R dv[kYS], ev[TRI ? 1 : kYS];
#pragma unroll
  for (int u = 0; u < kYS; ++u) {
    const int q = threadIdx.x + u * kBlock;
    if (q < Y.n) {
      int ex, ey, ez;
      Y.at(q, ex, ey, ez);
      const int gx = bwrap(t.x0 - 2 + ex, nx), gy = bwrap(t.y0 - 2 + ey, ny),
                gz = bwrap(t.z0 - 2 + ez, nz);
      const int g = (gz * ny + gy) * nx + gx;
      fv[u] = f.raw(g);
      dv[u] = C.d[g];
      if constexpr (!TRI)
        ev[u] = has_coarse && ((ex + ey + ez) & 1) == 0
                    ? e[((gz >> 1) * cny + (gy >> 1)) * cnx + (gx >> 1)]
                    : (R)0;
    }
  }
  Cell7<R> bc[kHS];
#pragma unroll
  for (int u = 0; u < kHS; ++u) {
    int ex, ey, ez;
    if (black_cell(H, t, threadIdx.x + u * kBlock, ex, ey, ez))
      load7(bc[u], C, nbrs(bwrap(t.x0 - 1 + ex, nx), bwrap(t.y0 - 1 + ey, ny),
                           bwrap(t.z0 - 1 + ez, nz), nx, ny, nz));
  }
  // outputs: x-pair s of the box, one red and one black cell
  const Frame O(t.tx >> 1, t.ty, t.tz);
  Cell7<R> rc[kPS];
  FT f0[kPS], f1[kPS];
  R z0[kPS], z1[kPS];
#pragma unroll
  for (int u = 0; u < kPS; ++u) {
    const int s = threadIdx.x + u * kBlock;
    z0[u] = z1[u] = 0;
    if (s < O.n) {
      int px, ly, lz;
      O.at(s, px, ly, lz);
      const Nb n = nbrs(t.x0 + 2 * px + ((ly + lz) & 1), t.y0 + ly, t.z0 + lz, nx, ny, nz);
      load7(rc[u], C, n);
      const int g = ((t.z0 + lz) * ny + t.y0 + ly) * nx + t.x0 + 2 * px;
      f0[u] = f.raw(g);
      f1[u] = f.raw(g + 1);
      if constexpr (L0 && sizeof(R) == 4) {
        if (rd_old) {
          z0[u] = zcur(P, sc)[g];
          z1[u] = zcur(P, sc)[g + 1];
        }
      }
    }
  }
  if constexpr (TRI) {
    if (has_coarse) {
#pragma unroll
      for (int u = 0; u < kCS; ++u)
        if (threadIdx.x + u * kBlock < G.n) cs[threadIdx.x + u * kBlock] = cv[u];
    }
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < kYS; ++u) {
    const int q = threadIdx.x + u * kBlock;
    if (q < Y.n) {
      R v = f.scaled(fv[u], inv_s) * recip(dv[u]);
      if constexpr (TRI) {
        int ex, ey, ez;
        Y.at(q, ex, ey, ez);
        if (has_coarse && ((ex + ey + ez) & 1) == 0) {
          // (the weights are combined in the order coarse_corr uses)
          const int gx = G.ax.d, gxy = G.ax.d * G.ay.d;
          const int I = (ex >> 1) + 1, J = (ey >> 1) + 1, K = (ez >> 1) + 1;
          const int I2 = (ex & 1) ? I + 1 : I - 1, J2 = (ey & 1) ? J + 1 : J - 1,
                    K2 = (ez & 1) ? K + 1 : K - 1;
          const R a = (R)0.75, b = (R)0.25;
          auto plane = [&](int k) {
            const R *c0 = cs + k * gxy + J * gx, *c1 = cs + k * gxy + J2 * gx;
            return a * (a * c0[I] + b * c0[I2]) + b * (a * c1[I] + b * c1[I2]);
          };
          v += a * plane(K) + b * plane(K2);
        }
      } else {
        v += ev[u];
      }
      vs[q] = v;
    }
  }
  __syncthreads();
  const int ax = Y.ax.d, axy = Y.ax.d * Y.ay.d, hx = H.ax.d, hxy = H.ax.d * H.ay.d;
#pragma unroll
  for (int u = 0; u < kHS; ++u) {
    const int q = threadIdx.x + u * kBlock;
    int ex, ey, ez;
    if (black_cell(H, t, q, ex, ey, ez))
      xs[q] = box_black(bc[u], vs, (ez + 1) * axy + (ey + 1) * ax + ex + 1, ax, axy);
  }
  __syncthreads();
  double rz = 0.0, rzo = 0.0;
#pragma unroll
  for (int u = 0; u < kPS; ++u) {
    const int s = threadIdx.x + u * kBlock;
    if (s < O.n) {
      int px, ly, lz;
      O.at(s, px, ly, lz);
      const int a = (ly + lz) & 1;  // the red cell of the pair
      const R red = (f.scaled(a ? f1[u] : f0[u], inv_s) +
                     box_red(rc[u], xs, 2 * px + a + 1, ly + 1, lz + 1, hx, hxy)) *
                    recip(rc[u].d);
      const R blk = xs[(lz + 1) * hxy + (ly + 1) * hx + ((2 * px + 2 - a) >> 1)];
      const R v0 = a ? blk : red, v1 = a ? red : blk;
      const int g = ((t.z0 + lz) * ny + t.y0 + ly) * nx + t.x0 + 2 * px;
      if constexpr (L0) {
        const double w0 = (double)v0 * s_out, w1 = (double)v1 * s_out;
        rz += f0[u] * w0;
        rz += f1[u] * w1;
        if constexpr (sizeof(R) == 4) {
          if (rd_old) {
            rzo += f0[u] * ((double)z0[u] * zs_old);
            rzo += f1[u] * ((double)z1[u] * zs_old);
          }
          znext(P, sc)[g] = v0;
          znext(P, sc)[g + 1] = v1;
        } else {
          znext<R>(P, sc)[g] = w0;
          znext<R>(P, sc)[g + 1] = w1;
        }
      } else {
        ((R *)L.x)[g] = v0;
        ((R *)L.x)[g + 1] = v1;
      }
    }
  }
  if constexpr (L0) write_partials(T, P.f0 + g0.block, rz, rzo);
}

// launchers ------------------------------------------------------------------

void launch_bdown(const Tables &T, TileList L, int l, int prec, int sel, hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l == 0 ? K_VDOWN_F : K_VDOWN_C;
  if (prec) {
    if (l == 0) FLD_LAUNCH(id, (k_bdown<float, true>), L.nblocks, kBlock, s, T, L, l, sel);
    else FLD_LAUNCH(id, (k_bdown<float, false>), L.nblocks, kBlock, s, T, L, l, sel);
  } else {
    if (l == 0) FLD_LAUNCH(id, (k_bdown<double, true>), L.nblocks, kBlock, s, T, L, l, sel);
    else FLD_LAUNCH(id, (k_bdown<double, false>), L.nblocks, kBlock, s, T, L, l, sel);
  }
}

template <typename R, bool L0>
static void launch_bup_t(const Tables &T, TileList L, int l, int id, int flexible,
                         int trilinear, hipStream_t s) {
  if (trilinear)
    FLD_LAUNCH(id, (k_bup<R, L0, true>), L.nblocks, kBlock, s, T, L, l, flexible);
  else
    FLD_LAUNCH(id, (k_bup<R, L0, false>), L.nblocks, kBlock, s, T, L, l, flexible);
}

void launch_bup(const Tables &T, TileList L, int l, int prec, int flexible, int trilinear,
                hipStream_t s) {
  if (!L.nblocks) return;
  const int id = l == 0 ? K_VUP_F : K_VUP_C;
  if (prec) {
    if (l == 0) launch_bup_t<float, true>(T, L, l, id, flexible, trilinear, s);
    else launch_bup_t<float, false>(T, L, l, id, flexible, trilinear, s);
  } else {
    // (the FP64 cycle's correction is piecewise constant)
    if (l == 0) launch_bup_t<double, true>(T, L, l, id, flexible, 0, s);
    else launch_bup_t<double, false>(T, L, l, id, flexible, 0, s);
  }
}

}  // namespace fld
