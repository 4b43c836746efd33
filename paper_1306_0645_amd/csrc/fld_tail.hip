// Tail of the V-cycle, one workgroup per problem: the coarsest level's
// Jacobi-CG solve and, above it, the levels from the tail's first down (each
// small): pre-smoothing and restriction down to the coarsest level, the solve,
// then prolongation and post-smoothing back up, in the order of the per-level
// path (red/black, red = even i+j+k).
//
// One workgroup on one CU is bound by latency: of a memory access, of a
// barrier and of a reduction, each paid once per phase.  So everything a
// thread needs is loaded at the start in one round of independent loads (its
// cell's coefficients on every level, one cell per thread; two x-pairs per
// thread of a level of up to 4096 cells), the values that cross threads live
// in LDS, reductions take one barrier (wave sums by DPP
// row operations, then every wave sums the 16 wave results), and a coarsest
// level of at most 64 cells is solved by one wave without any barrier.  The
// CG carries r.z and ||r||^2 through one reduction and scales by the
// reciprocal of the diagonal, divided once a solve (once an assembly where the
// operator is streamed).
// A coarsest level of up to 2 x 1024 cells keeps its operator in registers; one
// of up to 16 x 1024 (extents that stop halving early, such as 25^3 under
// 200^3) keeps r and q in registers, p in LDS and x in memory, and streams the
// operator and its reciprocal diagonal from the L2 in each iteration.  Measured per cycle
// (before: every phase through memory, three reductions of two barriers each
// per CG iteration, exact divisions): 8^3 and 4^3 levels of 64^3 and 256^3
// 21.3 -> 8.0 us, of 256^3 in FP64 24.8 -> 10.0 us; one 4^3 level 8.1 ->
// 2.8 us; 20^3 under 640^3 98 -> 48 us; 25^3 under 200^3 292 -> 133 us.
#include "fld_device.h"

namespace fld {

constexpr int kTW = kTailBlock / 64;  // waves of the tail block

// ---- one-barrier sums over the block ---------------------------------------

// red: [2][N][kTW] doubles; slot alternates from call to call, so that a
// call's writes never meet the reads of the call before
template <int N>
__device__ __forceinline__ void tail_sums(double (&v)[N], double *red, int &slot) {
  double *s = red + slot * 2 * kTW;
  slot ^= 1;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = wave_total(v[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) s[i * kTW + w] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = row_total(s[i * kTW + (lane & (kTW - 1))]);
}

// Orders a wave's LDS accesses before and after it, for values that pass
// between its lanes: its LDS operations execute in order, so this holds back
// the compiler alone and costs no instruction.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- coarsest solve ----------------------------------------------------------

// operator of one cell: its six faces, diagonal and its reciprocal, and the
// neighbours' indices
struct CgCell {
  double xp, xm, yp, ym, zp, zm, d, id;
  Nb n;
};

__device__ __forceinline__ void cg_load(CgCell &a, const LevelDev &L, int i, int j, int k) {
  a.n = nbrs(i, j, k, L.nx, L.ny, L.nz);
  a.xp = L.Tx[a.n.c];
  a.xm = L.Tx[a.n.xm];
  a.yp = L.Ty[a.n.c];
  a.ym = L.Ty[a.n.ym];
  a.zp = L.Tz[a.n.c];
  a.zm = L.Tz[a.n.zm];
  a.d = L.diag[a.n.c];
}

__device__ __forceinline__ void cg_load(CgCell &a, const LevelDev &L, int c) {
  cg_load(a, L, c % L.nx, (c / L.nx) % L.ny, c / (L.nx * L.ny));
}

__device__ __forceinline__ double cg_row(const CgCell &a, const double *p) {
  return a.d * p[a.n.c] - (a.xp * p[a.n.xp] + a.xm * p[a.n.xm] + a.yp * p[a.n.yp] +
                           a.ym * p[a.n.ym] + a.zp * p[a.n.zp] + a.zm * p[a.n.zm]);
}

// Jacobi-preconditioned CG in FP64 to a relative residual of 1e-12 (an
// effectively exact solve) on n cells, cell c = tid + u kTailBlock in slot u
// of the thread; f: right-hand side, x: solution.  Every thread of the block
// calls it.  WAVE: n <= 64, only wave 0 works and no barrier is taken.
// HOLD: the operator (cell[u], loaded by the caller) and x stay in registers;
// otherwise the operator is read in each iteration, two cells' loads at a
// time (all 16 at once would spill), x accumulates in xm (memory) and im holds
// the reciprocal diagonal, from k_coarsen.
template <int CPT, bool WAVE, bool HOLD>
__device__ __forceinline__ void coarse_cg(const LevelDev &L, CgCell (&cell)[HOLD ? CPT : 1],
                                          const double (&f)[CPT], double (&x)[HOLD ? CPT : 1],
                                          double *__restrict__ xm, const double *__restrict__ im,
                                          double *sp, double *red) {
  const int n = L.n;
  int slot = 0;
  auto sums = [&](double (&v)[2]) {
    if constexpr (WAVE) {
      v[0] = wave_total(v[0]);
      v[1] = wave_total(v[1]);
    } else {
      tail_sums<2>(v, red, slot);
    }
  };
  // !HOLD: the thread's first cell, and the step of kTailBlock cells, in
  // (x, y, z)
  const int i0 = HOLD ? 0 : (int)threadIdx.x % L.nx, j0 = HOLD ? 0 : (int)threadIdx.x / L.nx % L.ny,
            k0 = HOLD ? 0 : (int)threadIdx.x / (L.nx * L.ny);
  const int di = HOLD ? 0 : kTailBlock % L.nx, dj = HOLD ? 0 : kTailBlock / L.nx % L.ny,
            dk = HOLD ? 0 : kTailBlock / (L.nx * L.ny);
  double r[CPT];
  double a2[2] = {0.0, 0.0};  // ||r||^2, r.z
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const int c = threadIdx.x + u * kTailBlock;
    if constexpr (HOLD) x[u] = 0.0;
    r[u] = 0.0;
    if (c < n) {
      r[u] = f[u];
      double id;
      if constexpr (HOLD) {
        id = cell[u].id = 1.0 / cell[u].d;
      } else {
        xm[c] = 0.0;
        id = im[c];
      }
      const double t = r[u] * id;
      sp[c] = t;
      a2[0] += r[u] * r[u];
      a2[1] += r[u] * t;
    }
    if constexpr (!HOLD) {
      if ((u & 3) == 3) asm volatile("" ::: "memory");
    }
  }
  sums(a2);
  const double bb = a2[0];
  double rz = a2[1];
  if (!(bb > 0.0)) return;
  for (int it = 0; it < 1000; ++it) {
    // p is complete: the sums above ended with a barrier, as does the loop
    if constexpr (WAVE) wave_sync();
    double q[CPT];
    double a1[2] = {0.0, 0.0};
    int i = i0, j = j0, k = k0;
    // (the coordinates are opaque to the compiler: it would otherwise keep
    // every cell's addresses across the iterations, and spill them)
    if constexpr (!HOLD) asm volatile("" : "+v"(i), "+v"(j), "+v"(k));
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int c = threadIdx.x + u * kTailBlock;
      q[u] = 0.0;
      if (c < n) {
        if constexpr (HOLD) {
          q[u] = cg_row(cell[u], sp);
        } else {
          CgCell a;
          cg_load(a, L, i, j, k);
          q[u] = cg_row(a, sp);
        }
        a1[0] += sp[c] * q[u];
      }
      if constexpr (!HOLD) {
        if (u & 1) asm volatile("" ::: "memory");
        i += di;
        j += dj;
        k += dk;
        if (i >= L.nx) {
          i -= L.nx;
          ++j;
        }
        if (j >= L.ny) {
          j -= L.ny;
          ++k;
        }
      }
    }
    if constexpr (WAVE) {
      wave_sync();  // every lane has read p
      a1[0] = wave_total(a1[0]);
    } else {
      double b1[1] = {a1[0]};
      tail_sums<1>(b1, red, slot);
      a1[0] = b1[0];
    }
    const double alpha = rz / a1[0];
    double rd[CPT];
    a2[0] = a2[1] = 0.0;
    int c0 = threadIdx.x;
    if constexpr (!HOLD) asm volatile("" : "+v"(c0));
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int c = c0 + u * kTailBlock;
      rd[u] = 0.0;
      if (c < n) {
        if constexpr (HOLD) x[u] += alpha * sp[c];
        else xm[c] += alpha * sp[c];
        r[u] -= alpha * q[u];
        rd[u] = r[u] * (HOLD ? cell[HOLD ? u : 0].id : im[c]);
        a2[0] += r[u] * r[u];
        a2[1] += r[u] * rd[u];
      }
      if constexpr (!HOLD) {
        if ((u & 3) == 3) asm volatile("" ::: "memory");
      }
    }
    sums(a2);
    if (!(a2[0] > 1e-24 * bb)) break;  // converged (or NaN: stop)
    const double beta = a2[1] / rz;
    rz = a2[1];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const int c = threadIdx.x + u * kTailBlock;
      if (c < n) sp[c] = rd[u] + beta * sp[c];
    }
    if constexpr (!WAVE) __syncthreads();
  }
}

// ---- smoothing levels, one cell per thread, in LDS ---------------------------

template <typename R>
struct TailCell {
  R xp, xm, yp, ym, zp, zm, id;  // faces; 1 / diagonal
  R d;
  Nb n;
  int i, j, k;
  bool on, red;
};

template <typename R>
__device__ __forceinline__ void tail_load(TailCell<R> &a, const LevelDev &L) {
  const Coef<R> C = coefs<R>(L);
  const int c = threadIdx.x;
  a.on = c < L.n;
  a.red = false;
  if (!a.on) return;
  a.i = c % L.nx;
  a.j = (c / L.nx) % L.ny;
  a.k = c / (L.nx * L.ny);
  a.n = nbrs(a.i, a.j, a.k, L.nx, L.ny, L.nz);
  a.red = ((a.i + a.j + a.k) & 1) == 0;
  a.xp = C.tx[a.n.c];
  a.xm = C.tx[a.n.xm];
  a.yp = C.ty[a.n.c];
  a.ym = C.ty[a.n.ym];
  a.zp = C.tz[a.n.c];
  a.zm = C.tz[a.n.zm];
  a.d = C.d[a.n.c];
}

template <typename R, typename U>
__device__ __forceinline__ R tail_off(const TailCell<R> &a, const U &u) {
  return a.xp * u(a.n.xp) + a.xm * u(a.n.xm) + a.yp * u(a.n.yp) + a.ym * u(a.n.ym) +
         a.zp * u(a.n.zp) + a.zm * u(a.n.zm);
}

template <typename R>
__device__ __forceinline__ void tail_half(const TailCell<R> &a, R f, R *x, bool red) {
  auto xv = [&](int q) { return x[q]; };
  if (a.on && a.red == red) x[a.n.c] = (f + tail_off(a, xv)) * a.id;
  __syncthreads();
}

// nu sweeps from x = 0 (the first red half is f / d), then the residual into
// rs, and the coarse right-hand side of coarse cell tid (of LC): the 8
// children's residuals
template <typename R>
__device__ __forceinline__ R tail_down(TailCell<R> &a, R f, int nu, R *x, R *rs,
                                       const LevelDev &LF, const LevelDev &LC) {
  if (a.on) {
    a.id = recip(a.d);
    if (a.red) x[a.n.c] = f * a.id;
  }
  __syncthreads();
  tail_half(a, f, x, false);
  for (int s = 1; s < nu; ++s) {
    tail_half(a, f, x, true);
    tail_half(a, f, x, false);
  }
  auto xv = [&](int q) { return x[q]; };
  if (a.on) rs[a.n.c] = f - (a.d * x[a.n.c] - tail_off(a, xv));
  __syncthreads();
  R acc = 0;
  const int c = threadIdx.x;
  if (c < LC.n) {
    const int I = c % LC.nx, J = (c / LC.nx) % LC.ny, K = c / (LC.nx * LC.ny);
#pragma unroll
    for (int cz = 0; cz < 2; ++cz)
#pragma unroll
      for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx)
          acc += rs[((2 * K + cz) * LF.ny + 2 * J + cy) * LF.nx + 2 * I + cx];
  }
  __syncthreads();
  return acc;
}

// the correction e of the coarse level, folded into the first black half;
// then the rest of nu sweeps (black, red)
template <typename R>
__device__ __forceinline__ void tail_up(const TailCell<R> &a, R f, int nu, R *x, const R *e,
                                        const LevelDev &LF, const LevelDev &LC, bool tri) {
  if (a.on && !a.red) {
    const int nx = LF.nx, ny = LF.ny, nz = LF.nz, i = a.i, j = a.j, k = a.k;
    auto par = [&](int g, int b2, int c2) {
      return coarse_corr(e, g, b2, c2, LC.nx, LC.ny, LC.nz, tri);
    };
    const int im = i == 0 ? nx - 1 : i - 1, ip = i == nx - 1 ? 0 : i + 1;
    const int jm = j == 0 ? ny - 1 : j - 1, jp = j == ny - 1 ? 0 : j + 1;
    const int km = k == 0 ? nz - 1 : k - 1, kp = k == nz - 1 ? 0 : k + 1;
    const R s = a.xp * (x[a.n.xp] + par(ip, j, k)) + a.xm * (x[a.n.xm] + par(im, j, k)) +
                a.yp * (x[a.n.yp] + par(i, jp, k)) + a.ym * (x[a.n.ym] + par(i, jm, k)) +
                a.zp * (x[a.n.zp] + par(i, j, kp)) + a.zm * (x[a.n.zm] + par(i, j, km));
    x[a.n.c] = (f + s) * a.id;
  }
  __syncthreads();
  tail_half(a, f, x, true);
  for (int s = 1; s < nu; ++s) {
    tail_half(a, f, x, false);
    tail_half(a, f, x, true);
  }
}

// ---- the level above them, two x-pairs of cells per thread, in LDS -----------

// Red and black values lie in arrays of their own, at the pair's index q =
// (k ny + j) nx / 2 + i / 2: a cell's neighbours along y and z are the other
// colour's entries at q +- one row and plane, those along x at q itself and
// at q - 1 or q + 1.
template <typename R>
struct TopPair {
  R xo;                           // the face between the two cells
  R xr, yrp, yrm, zrp, zrm, dr;   // the red cell's other faces, diagonal
  R xb, ybp, ybm, zbp, zbm, db;   // the black cell's
  R fr, fb;
};

struct TopIdx {
  bool on;
  int q, side_r, side_b, yp, ym, zp, zm;
  int i, j, k;  // the red cell
};

__device__ __forceinline__ void top_index(TopIdx &a, const LevelDev &L, int q) {
  const int hx = L.nx >> 1;
  a.on = q < L.n >> 1;
  if (!a.on) return;
  const int px = q % hx, j = q / hx % L.ny, k = q / (hx * L.ny);
  const Nb n = nbrs(px, j, k, hx, L.ny, L.nz);
  const int odd = (j + k) & 1;
  a.q = q;
  a.side_r = odd ? n.xp : n.xm;
  a.side_b = odd ? n.xm : n.xp;
  a.yp = n.yp;
  a.ym = n.ym;
  a.zp = n.zp;
  a.zm = n.zm;
  a.i = 2 * px + odd;
  a.j = j;
  a.k = k;
}

template <typename R>
__device__ __forceinline__ void top_load(TopPair<R> &v, const TopIdx &a, const LevelDev &L) {
  typedef R R2 __attribute__((ext_vector_type(2)));
  if (!a.on) return;
  const Coef<R> C = coefs<R>(L);
  const bool odd = a.i & 1;
  auto pair = [&](const R *p, int q) { return ((const R2 *)p)[q]; };
  const R2 tx = pair(C.tx, a.q), yp = pair(C.ty, a.q), ym = pair(C.ty, a.ym),
           zp = pair(C.tz, a.q), zm = pair(C.tz, a.zm), d = pair(C.d, a.q),
           f = pair((const R *)L.f, a.q);
  // the face below the pair's first cell
  const R xm = C.tx[2 * (odd ? a.side_b : a.side_r) + 1];
  v.xo = tx.x;
  v.xr = odd ? tx.y : xm;
  v.xb = odd ? xm : tx.y;
  v.yrp = odd ? yp.y : yp.x;
  v.ybp = odd ? yp.x : yp.y;
  v.yrm = odd ? ym.y : ym.x;
  v.ybm = odd ? ym.x : ym.y;
  v.zrp = odd ? zp.y : zp.x;
  v.zbp = odd ? zp.x : zp.y;
  v.zrm = odd ? zm.y : zm.x;
  v.zbm = odd ? zm.x : zm.y;
  v.dr = odd ? d.y : d.x;
  v.db = odd ? d.x : d.y;
  v.fr = odd ? f.y : f.x;
  v.fb = odd ? f.x : f.y;
}

__device__ __forceinline__ void top_index(TopIdx (&a)[2], const LevelDev &L, int c) {
  top_index(a[0], L, c);
  top_index(a[1], L, c + kTailBlock);
}

template <typename R>
__device__ __forceinline__ void top_load(TopPair<R> (&v)[2], TopIdx (&a)[2], const LevelDev &L,
                                         int c) {
  top_index(a, L, c);
  top_load(v[0], a[0], L);
  top_load(v[1], a[1], L);
}

// sum of T x over the red cell's (black) neighbours, and the black cell's
template <typename R>
__device__ __forceinline__ R top_off_r(const TopPair<R> &v, const TopIdx &a, const R *xk) {
  return v.xo * xk[a.q] + v.xr * xk[a.side_r] + v.yrp * xk[a.yp] + v.yrm * xk[a.ym] +
         v.zrp * xk[a.zp] + v.zrm * xk[a.zm];
}

template <typename R>
__device__ __forceinline__ R top_off_b(const TopPair<R> &v, const TopIdx &a, const R *xr) {
  return v.xo * xr[a.q] + v.xb * xr[a.side_b] + v.ybp * xr[a.yp] + v.ybm * xr[a.ym] +
         v.zbp * xr[a.zp] + v.zbm * xr[a.zm];
}

template <typename R>
__device__ __forceinline__ void top_half_r(const TopPair<R> (&v)[2], const TopIdx (&a)[2], R *xr,
                                           const R *xk) {
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (a[u].on) xr[a[u].q] = (v[u].fr + top_off_r(v[u], a[u], xk)) * recip(v[u].dr);
  __syncthreads();
}

template <typename R>
__device__ __forceinline__ void top_half_b(const TopPair<R> (&v)[2], const TopIdx (&a)[2],
                                           const R *xr, R *xk) {
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (a[u].on) xk[a[u].q] = (v[u].fb + top_off_b(v[u], a[u], xr)) * recip(v[u].db);
  __syncthreads();
}

// nu sweeps from x = 0, and the coarse right-hand side of coarse cell tid:
// the residuals of its four red children (a black cell's is zero after the
// black half)
template <typename R>
__device__ __forceinline__ R top_down(const TopPair<R> (&v)[2], const TopIdx (&a)[2], int nu,
                                      R *xr, R *xk, R *rs, const LevelDev &LF,
                                      const LevelDev &LC) {
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (a[u].on) xr[a[u].q] = v[u].fr * recip(v[u].dr);
  __syncthreads();
  top_half_b(v, a, xr, xk);
  for (int s = 1; s < nu; ++s) {
    top_half_r(v, a, xr, xk);
    top_half_b(v, a, xr, xk);
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (a[u].on)
      rs[a[u].q] = v[u].fr - (v[u].dr * xr[a[u].q] - top_off_r(v[u], a[u], xk));
  __syncthreads();
  R acc = 0;
  const int c = threadIdx.x;
  if (c < LC.n) {
    const int I = c % LC.nx, J = (c / LC.nx) % LC.ny, K = c / (LC.nx * LC.ny);
#pragma unroll
    for (int cz = 0; cz < 2; ++cz)
#pragma unroll
      for (int cy = 0; cy < 2; ++cy) acc += rs[((2 * K + cz) * LF.ny + 2 * J + cy) * LC.nx + I];
  }
  return acc;
}

// the correction e of the coarse level at the red cells, then nu sweeps
// (black, red); the result goes to x in memory
template <typename R>
__device__ __forceinline__ void top_up(const TopPair<R> (&v)[2], const TopIdx (&a)[2], int nu,
                                       R *xr, R *xk, const R *e, const LevelDev &LF,
                                       const LevelDev &LC, bool tri) {
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (a[u].on)
      xr[a[u].q] += coarse_corr(e, a[u].i, a[u].j, a[u].k, LC.nx, LC.ny, LC.nz, tri);
  __syncthreads();
  for (int s = 0; s < nu; ++s) {
    top_half_b(v, a, xr, xk);
    top_half_r(v, a, xr, xk);
  }
  typedef R R2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (a[u].on) {
      const R r = xr[a[u].q], b = xk[a[u].q];
      R2 o;
      o.x = a[u].i & 1 ? b : r;
      o.y = a[u].i & 1 ? r : b;
      ((R2 *)(R *)LF.x)[a[u].q] = o;
    }
}

// The whole tail in LDS, every load of the pass issued at the start: TOP: a
// level of two pairs of cells per thread, then up to two levels of one cell
// per thread, then the coarsest.
template <typename R, bool TOP>
__device__ __forceinline__ void tail_lds(const Tables &T, int p, int lt, int lc, int nu_pre,
                                         int nu_post, bool tri, double *sp, double *red,
                                         R *const (&lx)[4]) {
  // (FP64: a top level's coefficients would not leave registers for the
  // others' and are loaded again on the way up)
  constexpr bool kKeep = TOP && sizeof(R) == 4;
  const int li = TOP ? lt + 1 : lt, ns = lc - li;
  const int c = threadIdx.x;
  R *xa = lx[0], *xb = lx[1], *xc = lx[2], *rs = lx[3];
  R *xr = (R *)(sp + kTailBlock), *xk = xr + kTailTop / 2, *rt = xk + kTailTop / 2;
  const LevelDev LT = T.lv[lt * T.nprob + p];
  const LevelDev L0 = T.lv[li * T.nprob + p];
  const LevelDev L1 = T.lv[min(li + 1, lc) * T.nprob + p];
  const LevelDev L2 = T.lv[lc * T.nprob + p];
  TopPair<R> tp[kKeep ? 2 : 1];
  TailCell<R> a, b;
  CgCell cell[1];
  R fa = 0, fb = 0, fcg = 0;
  if constexpr (TOP && !kKeep) {
    TopPair<R> t2[2];
    TopIdx ti[2];
    top_load(t2, ti, LT, c);
    fa = fcg = top_down(t2, ti, nu_pre, xr, xk, rt, LT, L0);
    asm volatile("" ::: "memory");
  }
  a.on = b.on = b.red = false;
  if (!TOP || ns >= 1) tail_load(a, L0);
  if (ns == 2) tail_load(b, L1);
  if (c < L2.n) cg_load(cell[0], L2, c);
  if constexpr (kKeep) {
    TopIdx ti[2];
    top_load(tp, ti, LT, c);
    fa = fcg = top_down(tp, ti, nu_pre, xr, xk, rt, LT, L0);
  }
  if constexpr (!TOP) {
    if (a.on) fa = ((const R *)L0.f)[c];
  }
  if (!TOP || ns >= 1) fcg = tail_down(a, fa, nu_pre, xa, rs, L0, L1);
  if (ns == 2) {
    fb = fcg;
    fcg = tail_down(b, fb, nu_pre, xb, rs, L1, L2);
  }
  const double f[1] = {c < L2.n ? (double)fcg : 0.0};
  double x[1] = {0.0};
  if (L2.n <= 64) {
    if (c < 64) coarse_cg<1, true, true>(L2, cell, f, x, nullptr, nullptr, sp, red);
  } else {
    coarse_cg<1, false, true>(L2, cell, f, x, nullptr, nullptr, sp, red);
  }
  R *xl = ns == 2 ? xc : (!TOP || ns == 1) ? xb : xa;
  if (c < L2.n) xl[c] = (R)x[0];
  __syncthreads();
  if (ns == 2) tail_up(b, fb, nu_post, xb, xc, L1, L2, tri);
  if (!TOP || ns >= 1) tail_up(a, fa, nu_post, xa, xb, L0, L1, tri);
  if constexpr (TOP) {
    // (the thread index is opaque: the compiler would otherwise keep the
    // indices, and in FP64 the coefficients, through the levels below)
    int c1 = c;
    asm volatile("" : "+v"(c1)::"memory");
    TopIdx ti[2];
    if constexpr (kKeep) {
      top_index(ti, LT, c1);
      top_up(tp, ti, nu_post, xr, xk, xa, LT, L0, tri);
    } else {
      TopPair<R> t2[2];
      top_load(t2, ti, LT, c1);
      top_up(t2, ti, nu_post, xr, xk, xa, LT, L0, tri);
    }
  } else if (a.on) {
    ((R *)L0.x)[c] = xa[c];
  }
}

// ---- smoothing levels through memory (more than kTailBlock cells) ------------

template <typename R>
struct LvlView {
  int nx, ny, nz, n;
  Coef<R> C;
  R *x, *f;
  __device__ __forceinline__ void ijk(int c, int &i, int &j, int &k) const {
    i = c % nx;
    j = (c / nx) % ny;
    k = c / (nx * ny);
  }
};

template <typename R>
__device__ __forceinline__ LvlView<R> lvl_view(const Tables &T, int l, int p) {
  const LevelDev L = T.lv[l * T.nprob + p];
  LvlView<R> v;
  v.nx = L.nx;
  v.ny = L.ny;
  v.nz = L.nz;
  v.n = L.n;
  v.C = coefs<R>(L);
  v.x = (R *)L.x;
  v.f = (R *)L.f;
  return v;
}

// first pre-sweep from x = 0 (red x = f/d, black from those red values)
template <typename R>
__device__ void mem_pre0(const LvlView<R> &V) {
  for (int c = threadIdx.x; c < V.n; c += kTailBlock) {
    int i, j, k;
    V.ijk(c, i, j, k);
    const Nb n = nbrs(i, j, k, V.nx, V.ny, V.nz);
    R v;
    if (((i + j + k) & 1) == 0) {
      v = V.f[c] * recip(V.C.d[c]);
    } else {
      auto red = [&](int q) { return V.f[q] * recip(V.C.d[q]); };
      v = (V.f[c] + offsum(V.C, n, red)) * recip(V.C.d[c]);
    }
    V.x[c] = v;
  }
}

template <typename R>
__device__ void mem_half(const LvlView<R> &V, int colour) {
  auto xv = [&](int q) { return V.x[q]; };
  for (int c = threadIdx.x; c < V.n; c += kTailBlock) {
    int i, j, k;
    V.ijk(c, i, j, k);
    if (((i + j + k) & 1) != colour) continue;
    const Nb n = nbrs(i, j, k, V.nx, V.ny, V.nz);
    V.x[c] = (V.f[c] + offsum(V.C, n, xv)) * recip(V.C.d[c]);
  }
}

// coarse right-hand side: fine residual summed over the 8 children
template <typename R>
__device__ void mem_restrict(const LvlView<R> &F, const LvlView<R> &Cv) {
  auto xv = [&](int q) { return F.x[q]; };
  for (int c = threadIdx.x; c < Cv.n; c += kTailBlock) {
    int I, J, K;
    Cv.ijk(c, I, J, K);
    R acc = 0;
    for (int cz = 0; cz < 2; ++cz)
      for (int cy = 0; cy < 2; ++cy)
        for (int cx = 0; cx < 2; ++cx) {
          const Nb n = nbrs(2 * I + cx, 2 * J + cy, 2 * K + cz, F.nx, F.ny, F.nz);
          acc += F.f[n.c] - (F.C.d[n.c] * F.x[n.c] - offsum(F.C, n, xv));
        }
    Cv.f[c] = acc;
  }
}

// black half-sweep with the coarse-grid correction folded in (red
// neighbours read as x + e(parent))
template <typename R>
__device__ void mem_prolong_black(const LvlView<R> &V, const LvlView<R> &Cv, bool tri) {
  for (int c = threadIdx.x; c < V.n; c += kTailBlock) {
    int i, j, k;
    V.ijk(c, i, j, k);
    if (((i + j + k) & 1) != 1) continue;
    const Nb n = nbrs(i, j, k, V.nx, V.ny, V.nz);
    const int im = i == 0 ? V.nx - 1 : i - 1, ip = i == V.nx - 1 ? 0 : i + 1;
    const int jm = j == 0 ? V.ny - 1 : j - 1, jp = j == V.ny - 1 ? 0 : j + 1;
    const int km = k == 0 ? V.nz - 1 : k - 1, kp = k == V.nz - 1 ? 0 : k + 1;
    auto par = [&](int a, int b2, int c2) {
      return coarse_corr(Cv.x, a, b2, c2, Cv.nx, Cv.ny, Cv.nz, tri);
    };
    const R s = V.C.tx[c] * (V.x[n.xp] + par(ip, j, k)) +
                V.C.tx[n.xm] * (V.x[n.xm] + par(im, j, k)) +
                V.C.ty[c] * (V.x[n.yp] + par(i, jp, k)) +
                V.C.ty[n.ym] * (V.x[n.ym] + par(i, jm, k)) +
                V.C.tz[c] * (V.x[n.zp] + par(i, j, kp)) +
                V.C.tz[n.zm] * (V.x[n.zm] + par(i, j, km));
    V.x[c] = (V.f[c] + s) * recip(V.C.d[c]);
  }
}

// the same CG for a coarsest level beyond the register path, its vectors in
// P.cs
template <typename R>
__device__ void mem_coarse_solve(const LevelDev &L, const ProbDev &P, double *red) {
  const int n = L.n, nx = L.nx, ny = L.ny, nz = L.nz;
  double *xs = P.cs, *rs = P.cs + n, *ps = P.cs + 2 * n, *qs = P.cs + 3 * n;
  const R *f = (const R *)L.f;
  R *xo = (R *)L.x;
  int slot = 0;
  double a2[2] = {0.0, 0.0};
  for (int c = threadIdx.x; c < n; c += kTailBlock) {
    const double v = (double)f[c], t = v / L.diag[c];
    rs[c] = v;
    xs[c] = 0.0;
    ps[c] = t;
    a2[0] += v * v;
    a2[1] += v * t;
  }
  tail_sums<2>(a2, red, slot);
  const double bb = a2[0];
  double rz = a2[1];
  if (bb > 0.0) {
    for (int it = 0; it < 1000; ++it) {
      __syncthreads();
      double a1[1] = {0.0};
      for (int c = threadIdx.x; c < n; c += kTailBlock) {
        const int i = c % nx, j = (c / nx) % ny, k = c / (nx * ny);
        const Nb nb = nbrs(i, j, k, nx, ny, nz);
        const double q = L.diag[c] * ps[c] -
                         (L.Tx[c] * ps[nb.xp] + L.Tx[nb.xm] * ps[nb.xm] +
                          L.Ty[c] * ps[nb.yp] + L.Ty[nb.ym] * ps[nb.ym] +
                          L.Tz[c] * ps[nb.zp] + L.Tz[nb.zm] * ps[nb.zm]);
        qs[c] = q;
        a1[0] += ps[c] * q;
      }
      tail_sums<1>(a1, red, slot);
      const double alpha = rz / a1[0];
      a2[0] = a2[1] = 0.0;
      for (int c = threadIdx.x; c < n; c += kTailBlock) {
        xs[c] += alpha * ps[c];
        const double r = rs[c] - alpha * qs[c];
        rs[c] = r;
        a2[0] += r * r;
        a2[1] += r * (r / L.diag[c]);
      }
      tail_sums<2>(a2, red, slot);
      if (!(a2[0] > 1e-24 * bb)) break;  // converged (or NaN: stop)
      const double beta = a2[1] / rz;
      rz = a2[1];
      for (int c = threadIdx.x; c < n; c += kTailBlock)
        ps[c] = rs[c] / L.diag[c] + beta * ps[c];
    }
  }
  for (int c = threadIdx.x; c < n; c += kTailBlock) xo[c] = (R)xs[c];
}

// CG over CPT cells per thread, right-hand side and solution in memory
template <typename R, int CPT, bool HOLD>
__device__ __forceinline__ void level_cg(const LevelDev &L, double *xm, double *sp,
                                         double *red) {
  CgCell cell[HOLD ? CPT : 1];
  double f[CPT], x[HOLD ? CPT : 1];
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const int c = threadIdx.x + u * kTailBlock;
    f[u] = 0.0;
    if (c < L.n) {
      f[u] = (double)((const R *)L.f)[c];
      if constexpr (HOLD) cg_load(cell[u], L, c);
    }
  }
  coarse_cg<CPT, false, HOLD>(L, cell, f, x, xm, xm + L.n, sp, red);
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    const int c = threadIdx.x + u * kTailBlock;
    if (c < L.n) ((R *)L.x)[c] = (R)(HOLD ? x[HOLD ? u : 0] : xm[c]);
  }
}

template <typename R, int CAP>
__global__ __launch_bounds__(kTailBlock) void k_vtail(Tables T, int nu_pre,
                                                     int nu_post, int trilinear, int sweeps) {
  const int p = blockIdx.x;
  const Scal &sc = T.sc[p];
  const ProbDev &P = T.pd[p];
  const int levels = P.levels, lt = sweeps ? P.tail_sweeps : P.tail, lc = levels - 1;
  if (!sc.active || levels < 2) return;
  constexpr bool kBig = CAP > kTailSmall;
  const LevelDev LC = T.lv[lc * T.nprob + p];
  if ((LC.n > kTailSmall) != kBig) return;  // (the other launch's)
  // the CG's direction; a level of more than kTailBlock cells keeps its
  // values and residuals behind the first kTailBlock entries
  __shared__ double sp[kBig ? CAP : kTailBlock + 3 * kTailTop / 2];
  __shared__ double red[2 * 2 * kTW];
  const bool tri = trilinear != 0;
  if constexpr (!kBig) {
    // (each level has an eighth of the cells of the one above)
    __shared__ R xa[kTailBlock], xb[kTailBlock / 8], xc[kTailBlock / 64], rs[kTailBlock];
    R *lx[4] = {xa, xb, xc, rs};
    const int n = T.lv[lt * T.nprob + p].n;
    if (n > kTailBlock && n <= kTailTop && lt < lc && lc - lt <= 3) {
      tail_lds<R, true>(T, p, lt, lc, nu_pre, nu_post, tri, sp, red, lx);
      return;
    }
    if (n <= kTailBlock && lt < lc && lc - lt <= 2) {
      tail_lds<R, false>(T, p, lt, lc, nu_pre, nu_post, tri, sp, red, lx);
      return;
    }
  }
  for (int l = lt; l < lc; ++l) {
    const LvlView<R> V = lvl_view<R>(T, l, p);
    mem_pre0(V);
    __syncthreads();
    for (int s2 = 1; s2 < nu_pre; ++s2) {
      mem_half(V, 0);
      __syncthreads();
      mem_half(V, 1);
      __syncthreads();
    }
    mem_restrict(V, lvl_view<R>(T, l + 1, p));
    __syncthreads();
  }
  if constexpr (!kBig) {
    if (LC.n <= 64) {
      if (threadIdx.x < 64) {
        CgCell cell[1];
        const int c = threadIdx.x;
        double f[1] = {0.0}, x[1];
        if (c < LC.n) {
          f[0] = (double)((const R *)LC.f)[c];
          cg_load(cell[0], LC, c);
        }
        coarse_cg<1, true, true>(LC, cell, f, x, nullptr, nullptr, sp, red);
        if (c < LC.n) ((R *)LC.x)[c] = (R)x[0];
      }
    } else if (LC.n <= kTailBlock) {
      level_cg<R, 1, true>(LC, P.cs, sp, red);
    } else {
      level_cg<R, 2, true>(LC, P.cs, sp, red);
    }
  } else {
    if (LC.n <= 4 * kTailBlock) level_cg<R, 4, false>(LC, P.cs, sp, red);
    else if (LC.n <= 8 * kTailBlock) level_cg<R, 8, false>(LC, P.cs, sp, red);
    else if (LC.n <= kTailBig) level_cg<R, 16, false>(LC, P.cs, sp, red);
    else mem_coarse_solve<R>(LC, P, red);
  }
  __syncthreads();
  for (int l = lc - 1; l >= lt; --l) {
    const LvlView<R> V = lvl_view<R>(T, l, p);
    mem_prolong_black(V, lvl_view<R>(T, l + 1, p), tri);
    __syncthreads();
    mem_half(V, 0);
    __syncthreads();
    for (int s2 = 1; s2 < nu_post; ++s2) {
      mem_half(V, 1);
      __syncthreads();
      mem_half(V, 0);
      __syncthreads();
    }
  }
}

// routes: 1: some problem's coarsest level has at most kTailSmall cells, 2:
// some problem's has more (a kernel each: the one holds its levels in LDS and
// registers, the other the LDS for the streamed solve)
void launch_vtail(const Tables &T, int prec, int nu_pre, int nu_post, int trilinear,
                  int routes, int sweeps, hipStream_t s) {
  if (!T.nprob) return;
  if (prec) {
    if (routes & 1)
      FLD_LAUNCH(K_COARSE_SOLVE, (k_vtail<float, kTailSmall>), T.nprob, kTailBlock, s, T,
                 nu_pre, nu_post, trilinear, sweeps);
    if (routes & 2)
      FLD_LAUNCH(K_COARSE_SOLVE, (k_vtail<float, kTailBig>), T.nprob, kTailBlock, s, T,
                 nu_pre, nu_post, trilinear, sweeps);
  } else {
    if (routes & 1)
      FLD_LAUNCH(K_COARSE_SOLVE, (k_vtail<double, kTailSmall>), T.nprob, kTailBlock, s, T,
                 nu_pre, nu_post, trilinear, sweeps);
    if (routes & 2)
      FLD_LAUNCH(K_COARSE_SOLVE, (k_vtail<double, kTailBig>), T.nprob, kTailBlock, s, T,
                 nu_pre, nu_post, trilinear, sweeps);
  }
}

}  // namespace fld
