// Device-side helpers shared by the HIP kernel files: tile addressing
// (XCD-aware block renumbering, range lists), periodic neighbour indices,
// deterministic block reductions, typed coefficient access and the V-cycle
// right-hand-side source.
#pragma once

#include <math.h>

#include <type_traits>

#define FLD_KERNELS 1
#include "fld_internal.h"

namespace fld {

// ---------------------------------------------------------------------------
// tile addressing
// ---------------------------------------------------------------------------

// Workgroups are dispatched round-robin over the 8 XCDs.  Renumber them so
// that XCD x processes the contiguous block range [start_x, start_x + cnt_x).
__device__ __forceinline__ int xcd_block(int nb) {
  const int b = blockIdx.x;
  const int x = b & 7, q = nb >> 3, rem = nb & 7;
  return x * q + (x < rem ? x : rem) + (b >> 3);
}

// The block's range of the list: its problem, its first table entry and the
// block's index in it.  The problem comes with the range, so that the kernel's
// loads of the problem's descriptors do not wait for the tile's.  A list of
// one range (a plain handle) carries it in the kernel arguments; up to 64
// ranges are searched by one load, a range per lane, and a ballot.
struct Range {
  int prob, first, block;
};

__device__ __forceinline__ Range get_range(const TileList &L) {
  const int b = xcd_block(L.nblocks);
  int p = L.prob, first = L.first, start = 0;
  if (L.nranges > 1) {
    int lo = 0;
    if (L.nranges <= 64) {
      const int lane = threadIdx.x & 63;
      const int r = lane < L.nranges ? lane : 0;
      const int rs = L.ranges[3 * r], rf = L.ranges[3 * r + 1], rp = L.ranges[3 * r + 2];
      lo = __popcll(__ballot(lane < L.nranges && rs <= b)) - 1;
      start = __builtin_amdgcn_readlane(rs, lo);
      first = __builtin_amdgcn_readlane(rf, lo);
      p = __builtin_amdgcn_readlane(rp, lo);
    } else {
      int hi = L.nranges - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (L.ranges[3 * mid] <= b) lo = mid; else hi = mid - 1;
      }
      start = L.ranges[3 * lo];
      first = L.ranges[3 * lo + 1];
      p = L.ranges[3 * lo + 2];
    }
  }
  return {p, first, b - start};
}

// The block's tile: idx is its index inside the full table (for per-tile
// partial sums).
__device__ __forceinline__ Tile get_tile(const TileList &L, int &idx) {
  const Range g = get_range(L);
  idx = g.first + g.block;
  const TileRec r = L.base[idx];
  return {g.prob, r.x0, r.y0, r.z0, (int)(r.ext & 255), (int)(r.ext >> 8 & 255),
          (int)(r.ext >> 16)};
}

__device__ __forceinline__ Tile get_tile(const TileList &L) {
  int idx;
  return get_tile(L, idx);
}

// Thread -> cells: a thread owns the column (i, j) of the tile and walks its
// planes.
struct Col {
  int i, j;
  bool on;
};

__device__ __forceinline__ Col tile_col(const Tile &t) {
  Col c;
  const int lx = threadIdx.x % t.tx, ly = threadIdx.x / t.tx;
  c.i = t.x0 + lx;
  c.j = t.y0 + ly;
  c.on = ly < t.ty;
  return c;
}

// linear indices of a cell and its 6 periodic neighbours
struct Nb {
  int c, xm, xp, ym, yp, zm, zp;
};

__device__ __forceinline__ Nb nbrs(int i, int j, int k, int nx, int ny, int nz) {
  Nb n;
  const int plane = nx * ny;
  const int row = k * plane + j * nx;
  n.c = row + i;
  n.xm = row + (i == 0 ? nx - 1 : i - 1);
  n.xp = row + (i == nx - 1 ? 0 : i + 1);
  n.ym = (j == 0) ? n.c + (ny - 1) * nx : n.c - nx;
  n.yp = (j == ny - 1) ? n.c - (ny - 1) * nx : n.c + nx;
  n.zm = (k == 0) ? n.c + (nz - 1) * plane : n.c - plane;
  n.zp = (k == nz - 1) ? n.c - (nz - 1) * plane : n.c + plane;
  return n;
}

// ---------------------------------------------------------------------------
// streaming access (NT): a value that no other block reads or wrote in this
// launch.  Marked as such it leaves its place in the caches to the cells that
// neighbouring tiles share; but a working set that stays in the caches from
// one launch to the next is then read from memory again.  So the launchers
// take NT from the size of all the problems together (Tables::stream).  The
// fused passes' face loads are never marked: their edge cells are shared, and
// marking them cost 4 %.
// ---------------------------------------------------------------------------

template <bool NT, typename V>
__device__ __forceinline__ auto stream_in(const V *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename V, typename W>
__device__ __forceinline__ void stream_out(V *p, W v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// ---------------------------------------------------------------------------
// reductions (deterministic)
// ---------------------------------------------------------------------------

// v of the lane that a DPP row operation names, 0 where there is none
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_get(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double lane_get(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// running sums within each row of 16 lanes: lane 15 holds the row's total
__device__ __forceinline__ double row_scan(double v) {
  v += dpp_get<0x111, 0xf>(v);  // row_shr:1
  v += dpp_get<0x112, 0xf>(v);
  v += dpp_get<0x114, 0xf>(v);
  v += dpp_get<0x118, 0xf>(v);
  return v;
}

// Sum over the wave, in every lane, by DPP moves (registers only: a
// butterfly of cross-lane LDS operations takes about four times as long).
// Every lane must be active.
__device__ __forceinline__ double wave_total(double v) {
  v = row_scan(v);
  v += dpp_get<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v += dpp_get<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return lane_get(v, 63);
}

// Sum of lanes 0 .. 15, in every lane.
__device__ __forceinline__ double row_total(double v) { return lane_get(row_scan(v), 15); }

// N sums of a tile into out[N * tile + i] (one LDS round for all of them)
template <int N>
__device__ __forceinline__ void write_sums(double *out, int tile, const double (&v)[N]) {
  constexpr int NW = kBlock / 64;
  __shared__ double sh[N][NW];
  double w[N];
#pragma unroll
  for (int i = 0; i < N; ++i) w[i] = wave_total(v[i]);
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) sh[i][threadIdx.x >> 6] = w[i];
  }
  __syncthreads();
  if (threadIdx.x < N) {
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) s += sh[threadIdx.x][k];
    out[N * tile + threadIdx.x] = s;
  }
}

__device__ __forceinline__ void write_partials(const Tables &T, int tile,
                                               double a0, double a1) {
  const double v[2] = {a0, a1};
  write_sums(T.part, tile, v);
}

// ---------------------------------------------------------------------------
// typed access to a level's coefficients
// ---------------------------------------------------------------------------

template <typename R>
struct Coef {
  const R *tx, *ty, *tz, *d;
};

template <typename R>
__device__ __forceinline__ Coef<R> coefs(const LevelDev &L);

template <>
__device__ __forceinline__ Coef<double> coefs<double>(const LevelDev &L) {
  return {L.Tx, L.Ty, L.Tz, L.diag};
}

template <>
__device__ __forceinline__ Coef<float> coefs<float>(const LevelDev &L) {
  return {L.Tx32, L.Ty32, L.Tz32, L.diag32};
}

// sum over the 6 neighbours of T_face * u_neighbour
template <typename R, typename U>
__device__ __forceinline__ R offsum(const Coef<R> &C, const Nb &n, const U &u) {
  return C.tx[n.c] * u(n.xp) + C.tx[n.xm] * u(n.xm) + C.ty[n.c] * u(n.yp) +
         C.ty[n.ym] * u(n.ym) + C.tz[n.c] * u(n.zp) + C.tz[n.zm] * u(n.zm);
}

__device__ __forceinline__ double recip(double d) { return 1.0 / d; }
__device__ __forceinline__ float recip(float d) {
  return __builtin_amdgcn_rcpf(d);  // ~1 ulp: ample for a preconditioner
}

// ---------------------------------------------------------------------------
// V-cycle right-hand side.  R = level precision, L0 = finest level (the
// right-hand side is the FP64 Krylov residual scaled by 1/s).
// ---------------------------------------------------------------------------

template <typename R, bool L0>
struct FSrc {
  using FT = std::conditional_t<L0, double, R>;
  const R *f;
  const double *r;
  double inv_s;
  // the value as stored, and scaled to the cycle's units
  __device__ __forceinline__ FT raw(int c) const {
    if constexpr (L0) return r[c];
    else return f[c];
  }
  __device__ __forceinline__ R scaled(FT v, double is) const {
    if constexpr (L0) return (R)(v * is);
    else return v;
  }
  __device__ __forceinline__ R operator()(int c) const {
    if constexpr (L0) return (R)(r[c] * inv_s);
    else return f[c];
  }
};

// Assembly and warm start of a problem are due: for the host-driven step
// whenever the problem takes part (the host launches them when due); for
// device-controlled stepping when its controller asked for them.
__device__ __forceinline__ bool asm_due(const Scal &sc) {
  return sc.live && (!sc.ctl || sc.stage == 1);
}
__device__ __forceinline__ bool warm_due(const Scal &sc) {
  return sc.live && (!sc.ctl || sc.stage == 2);
}

// the current residual buffer, and the other one
__device__ __forceinline__ double *rcur(const ProbDev &P, const Scal &sc) {
  return sc.rbuf ? P.r2 : P.r;
}
__device__ __forceinline__ double *rnext(const ProbDev &P, const Scal &sc) {
  return sc.rbuf ? P.r : P.r2;
}

// the newest z (after FIN_RZ), and the buffer that the fused cycle's
// post-sweep writes
template <typename R = float>
__device__ __forceinline__ R *zcur(const ProbDev &P, const Scal &sc) {
  if constexpr (sizeof(R) == 4) return sc.zbuf ? P.z32b : P.z32;
  else return sc.zbuf ? P.zb : P.z;
}
template <typename R = float>
__device__ __forceinline__ R *znext(const ProbDev &P, const Scal &sc) {
  if constexpr (sizeof(R) == 4) return sc.zbuf ? P.z32 : P.z32b;
  else return sc.zbuf ? P.z : P.zb;
}

template <typename R, bool L0>
__device__ __forceinline__ FSrc<R, L0> fsrc(const LevelDev &L, const ProbDev &P,
                                             const Scal &sc) {
  FSrc<R, L0> s;
  s.f = (const R *)L.f;
  s.r = rcur(P, sc);
  s.inv_s = sc.inv_s;
  return s;
}

// Coarse-grid correction at fine cell (gx, gy, gz) of a level whose coarse
// level has extents (cnx, cny, cnz) = half the fine ones.
//  trilinear = false: piecewise constant, e(parent)
//  trilinear = true:  cell-centred trilinear interpolation from the 8 nearest
//                     coarse cells, weights 3/4 (own parent) and 1/4 (the
//                     neighbour on the fine cell's side) per direction
template <typename R>
__device__ __forceinline__ R coarse_corr(const R *e, int gx, int gy, int gz,
                                         int cnx, int cny, int cnz,
                                         bool trilinear) {
  const int I = gx >> 1, J = gy >> 1, K = gz >> 1;
  if (!trilinear) return e[(K * cny + J) * cnx + I];
  const int I2 = (gx & 1) ? (I + 1 == cnx ? 0 : I + 1) : (I == 0 ? cnx - 1 : I - 1);
  const int J2 = (gy & 1) ? (J + 1 == cny ? 0 : J + 1) : (J == 0 ? cny - 1 : J - 1);
  const int K2 = (gz & 1) ? (K + 1 == cnz ? 0 : K + 1) : (K == 0 ? cnz - 1 : K - 1);
  const R a = (R)0.75, b = (R)0.25;
  const int r00 = (K * cny + J) * cnx, r01 = (K * cny + J2) * cnx;
  const int r10 = (K2 * cny + J) * cnx, r11 = (K2 * cny + J2) * cnx;
  const R zK = a * (a * e[r00 + I] + b * e[r00 + I2]) +
               b * (a * e[r01 + I] + b * e[r01 + I2]);
  const R zK2 = a * (a * e[r10 + I] + b * e[r10 + I2]) +
                b * (a * e[r11 + I] + b * e[r11 + I2]);
  return a * zK + b * zK2;
}

}  // namespace fld
