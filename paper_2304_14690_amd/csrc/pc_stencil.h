// WLS derivative rows evaluated where they are applied (Sec. 2.2, Eqs. 9-17),
// instead of read back from stored coefficients.
//
// Node targets with a full block of m^d grid points (m = 3 or 4).  The block
// is a tensor product of grid lines and the Gaussian weight of Eq. 17 a
// product over the axes, so the weighted fit of Eq. 16 is diagonal in
// products of the discrete orthogonal polynomials of each axis: with
// w_l = exp(-beta t_l^2) on the m lines of an axis (t in grid spacings),
// p0 = 1, p1, p2 monic and orthogonal under w, the products p_i p_j p_k of
// total degree <= 2 span the same space as Eq. 16's polynomial vector and
// are orthogonal under the product weight.  The fitted gradient at the node
// (p' the derivative, all at the node; <.> over the lines of an axis) is then
//   d/dx = <E>_x <A0>_y <A0>_z + <A1>_x <p1 A1>_y <A0>_z + <A1>_x <A0>_y <p1 A1>_z
// with A_i = w p_i / <w p_i p_i> and E = A1 + p2' A2, and likewise for the
// other axes: the coefficients that C^-1 A of Eq. 13 gives, without the
// normal matrix.  A node costs about 500 float64 operations in 3D and its
// position instead of 648 bytes of coefficients.
#pragma once

#include "pc_internal.h"

namespace pc {

// 1/x for normal x: the hardware reciprocal and two Newton steps.
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// exp(y) for y <= 709 (flushed to exp(-700) below -700): y = k ln 2 + r,
// |r| <= ln 2 / 2, and a degree-11 polynomial in r (the minimax fit of
// (exp(r) - 1 - r) / r^2, with its coefficients rounded, leaves 1.6e-17 of the
// result).
__device__ __forceinline__ double exp_fast(double y) {
  constexpr double LOG2E = 1.4426950408889634074, MAGIC = 6755399441055744.0;  // 1.5 2^52
  constexpr double LN2 = 6.9314718055994530942e-1, LN2_LO = 2.3190468138462995584e-17;
  y = fmax(y, -700.0);
  const double t = __builtin_fma(y, LOG2E, MAGIC);
  const double k = t - MAGIC;
  double r = __builtin_fma(-k, LN2, y);
  r = __builtin_fma(-k, LN2_LO, r);
  double p = 2.5100385495510319078e-8;
  p = __builtin_fma(p, r, 2.7620088445409748161e-7);
  p = __builtin_fma(p, r, 2.7557268459997064772e-6);
  p = __builtin_fma(p, r, 2.4801521295954375131e-5);
  p = __builtin_fma(p, r, 1.9841269863053616878e-4);
  p = __builtin_fma(p, r, 1.3888888917213716901e-3);
  p = __builtin_fma(p, r, 8.3333333333300618325e-3);
  p = __builtin_fma(p, r, 4.1666666666624127873e-2);
  p = __builtin_fma(p, r, 1.6666666666666667453e-1);
  p = __builtin_fma(p, r, 5.0000000000000010221e-1);
  p = __builtin_fma(p, r, 1.0);
  p = __builtin_fma(p, r, 1.0);
  // the low word of t is k: add it to the exponent
  const uint64_t tb = __builtin_bit_cast(uint64_t, t), pb = __builtin_bit_cast(uint64_t, p);
  const uint32_t hi = (uint32_t)(pb >> 32) + ((uint32_t)tb << 20);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | (uint32_t)pb);
}

// ---- node targets ---------------------------------------------------------------
// What the rows of a node need besides its position and block corner.
struct NodeFit {
  int32_t n[3];
  int per;               // bit a: axis a is periodic
  double off;            // grid point i at (i + off) h
  double h[3], ih[3];
  double hl[3];          // half the box length
  double inv_n0, inv_n1;
  double hsup2, eps;     // squared support radius, Eq. 17's shape parameter
  double beta[3], s[3];  // eps h^2 / hsup^2 and exp(-beta) per axis
};

NodeFit node_fit_args(const pc_geom* g);

// One axis of a node's fit: the vectors A0, A1 and E above over the block's
// lines and p1 at the node, in units of the grid spacing.
template <int MB>
struct AxisFit {
  double a0[MB], a1[MB], e[MB], p1;
  double W, N1, N2;  // <w>, <w p1 p1>, <w p2 p2> (the pivots of the normal matrix)
};

// t1: offset of the block's second line from the node in grid spacings (line
// l sits at y = l - 1, the node at y = -t1); beta and s as in NodeFit.  The
// weights are taken relative to the second line's (a common factor cancels).
template <int MB>
__device__ __forceinline__ AxisFit<MB> axis_fit(double t1, double beta, double s) {
  static_assert(MB == 3 || MB == 4, "block lines");
  AxisFit<MB> F;
  const double up = exp_fast(2.0 * beta * t1), dn = recip(up);
  const double w0 = s * up, w2 = s * dn, ys = -t1;
  if constexpr (MB == 3) {
    const double sum = w0 + w2, W = sum + 1.0, iW = recip(W);
    const double a = (w2 - w0) * iW;
    const double q0 = -1.0 - a, q1 = -a, q2 = 1.0 - a;
    const double v0 = w0 * q0, v1 = q1, v2 = w2 * q2;
    const double N1 = __builtin_fma(v0, q0, __builtin_fma(v1, q1, v2 * q2)), iN = recip(N1);
    F.a0[0] = w0 * iW; F.a0[1] = iW; F.a0[2] = w2 * iW;
    F.a1[0] = v0 * iN; F.a1[1] = v1 * iN; F.a1[2] = v2 * iN;
    // w p2 is proportional to (1, -2, 1), the only vector orthogonal to the
    // linear functions on three lines: A2 = (1, -2, 1) / 2
    const double c = __builtin_fma(2.0, ys, -(F.a1[0] + F.a1[2]));  // p2' at the node
    const double hc = 0.5 * c;
    F.e[0] = F.a1[0] + hc; F.e[1] = F.a1[1] - c; F.e[2] = F.a1[2] + hc;
    F.p1 = ys - a;
    F.W = W; F.N1 = N1; F.N2 = 4.0 / (1.0 / w0 + 4.0 + 1.0 / w2);
  } else {
    const double s2 = s * s, w3 = (s2 * s2) * (dn * dn);
    const double W = ((w0 + w2) + w3) + 1.0, iW = recip(W);
    const double a = __builtin_fma(2.0, w3, w2 - w0) * iW;
    const double q[4] = {-1.0 - a, -a, 1.0 - a, 2.0 - a};
    const double w[4] = {w0, 1.0, w2, w3}, y2[4] = {1.0, 0.0, 1.0, 4.0};
    double v[4], N1 = 0.0, b = 0.0;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      v[l] = w[l] * q[l];
      N1 = __builtin_fma(v[l], q[l], N1);
      b = __builtin_fma(v[l], y2[l], b);
    }
    const double iN = recip(N1);
    b *= iN;
    const double d = (w0 + w2 + 4.0 * w3) * iW;  // <w y^2> / <w>
    double u[4], N2 = 0.0;
#pragma unroll
    for (int l = 0; l < 4; ++l) {
      F.a0[l] = w[l] * iW;
      F.a1[l] = v[l] * iN;
      const double p2 = __builtin_fma(-b, q[l], y2[l]) - d;
      u[l] = w[l] * p2;
      N2 = __builtin_fma(u[l], p2, N2);
    }
    const double c = __builtin_fma(2.0, ys, -b) * recip(N2);  // p2' at the node over <w p2 p2>
#pragma unroll
    for (int l = 0; l < 4; ++l) F.e[l] = __builtin_fma(c, u[l], F.a1[l]);
    F.p1 = ys - a;
    F.W = W; F.N1 = N1; F.N2 = N2;
  }
  return F;
}

// The block of a node: low corner per axis (on a periodic axis the wrapped
// line) and the fit of every axis.  kappa (nullable): h / h_t per axis.
template <int D, int MB>
struct BlockFit {
  int c[3];
  AxisFit<MB> ax[D];
};

template <int D, int MB>
__device__ __forceinline__ BlockFit<D, MB> block_fit(const NodeFit& A, int32_t base,
                                                     const double (&x)[D],
                                                     double* kappa2 = nullptr) {
  BlockFit<D, MB> B;
  // flat index to lines: (c + 1/2) / n0 lies at least 1/(2 n0) from an
  // integer, far above the rounding of its float64 product
  const int flat = base < 0 ? ~base : base;
  int q = (int)(((double)flat + 0.5) * A.inv_n0);
  B.c[0] = flat - q * A.n[0];
  B.c[1] = q;
  B.c[2] = 0;
  if (D == 3) {
    const int z = (int)(((double)q + 0.5) * A.inv_n1);
    B.c[1] = q - z * A.n[1];
    B.c[2] = z;
  }
  double x1[D], rk2 = 0.0;
#pragma unroll
  for (int a = 0; a < D; ++a) {
    double x0 = ((double)B.c[a] + A.off) * A.h[a] - x[a];
    // a block that starts one box length back (periodic axis)
    const int back = (((A.per >> a) & 1) && x0 > A.hl[a]) ? A.n[a] : 0;
    x0 = ((double)(B.c[a] - back) + A.off) * A.h[a] - x[a];
    x1[a] = ((double)(B.c[a] - back + 1) + A.off) * A.h[a] - x[a];
    const double xe = ((double)(B.c[a] - back + MB - 1) + A.off) * A.h[a] - x[a];
    rk2 += fmax(x0 * x0, xe * xe);
  }
  double beta[D], s[D];
#pragma unroll
  for (int a = 0; a < D; ++a) {
    beta[a] = A.beta[a];
    s[a] = A.s[a];
  }
  // h_t = max(support, the farthest block point): beyond the support radius
  // only next to a wall, or with a support below the block's
  const double ht2 = fmax(rk2, A.hsup2);
  if (rk2 > A.hsup2) {
    const double er = A.eps / rk2;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      beta[a] = er * (A.h[a] * A.h[a]);
      s[a] = exp_fast(-beta[a]);
    }
  }
#pragma unroll
  for (int a = 0; a < D; ++a) {
    if (kappa2) kappa2[a] = A.h[a] * A.h[a] / ht2;
    B.ax[a] = axis_fit<MB>(x1[a] * A.ih[a], beta[a], s[a]);
  }
  return B;
}

// Offset of line l of axis a's block from its low corner, in lines; a line
// past the end of a periodic axis is one box length back.
template <bool WRAP>
__device__ __forceinline__ int line_off(const NodeFit& A, int a, int c, int l) {
  return WRAP && ((A.per >> a) & 1) && c + l >= A.n[a] ? l - A.n[a] : l;
}

// grad f at a node from f on its block; rd(l, j, k) reads line (l, j, k).
template <int D, int MB, typename RD>
__device__ __forceinline__ void block_grad(const NodeFit& A, const BlockFit<D, MB>& B,
                                           const RD& rd, double (&G)[D]) {
  const AxisFit<MB>& X = B.ax[0];
  const AxisFit<MB>& Y = B.ax[1];
  if constexpr (D == 2) {
    double gx = 0.0, gy = 0.0, xb = 0.0, yb = 0.0;
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      double s0 = 0.0, s1 = 0.0, se = 0.0;
#pragma unroll
      for (int l = 0; l < MB; ++l) {
        const double f = rd(l, j, 0);
        s0 = __builtin_fma(X.a0[l], f, s0);
        s1 = __builtin_fma(X.a1[l], f, s1);
        se = __builtin_fma(X.e[l], f, se);
      }
      gx = __builtin_fma(Y.a0[j], se, gx);
      xb = __builtin_fma(Y.a1[j], s1, xb);
      gy = __builtin_fma(Y.e[j], s0, gy);
    }
    G[0] = __builtin_fma(Y.p1, xb, gx) * A.ih[0];
    G[1] = __builtin_fma(X.p1, xb, gy) * A.ih[1];
  } else {
    const AxisFit<MB>& Z = B.ax[2];
    double gx = 0.0, gy = 0.0, gz = 0.0, hx = 0.0, hy = 0.0;
#pragma unroll
    for (int k = 0; k < MB; ++k) {
      double pe0 = 0.0, p10 = 0.0, p11 = 0.0, p00 = 0.0, p01 = 0.0, p0e = 0.0;
#pragma unroll
      for (int j = 0; j < MB; ++j) {
        double s0 = 0.0, s1 = 0.0, se = 0.0;
#pragma unroll
        for (int l = 0; l < MB; ++l) {
          const double f = rd(l, j, k);
          s0 = __builtin_fma(X.a0[l], f, s0);
          s1 = __builtin_fma(X.a1[l], f, s1);
          se = __builtin_fma(X.e[l], f, se);
        }
        pe0 = __builtin_fma(Y.a0[j], se, pe0);
        p10 = __builtin_fma(Y.a0[j], s1, p10);
        p11 = __builtin_fma(Y.a1[j], s1, p11);
        p00 = __builtin_fma(Y.a0[j], s0, p00);
        p01 = __builtin_fma(Y.a1[j], s0, p01);
        p0e = __builtin_fma(Y.e[j], s0, p0e);
      }
      gx = __builtin_fma(Z.a0[k], __builtin_fma(Y.p1, p11, pe0), gx);
      gy = __builtin_fma(Z.a0[k], __builtin_fma(X.p1, p11, p0e), gy);
      hx = __builtin_fma(Z.a1[k], p10, hx);
      hy = __builtin_fma(Z.a1[k], p01, hy);
      gz = __builtin_fma(Z.e[k], p00, gz);
    }
    G[0] = __builtin_fma(Z.p1, hx, gx) * A.ih[0];
    G[1] = __builtin_fma(Z.p1, hy, gy) * A.ih[1];
    G[2] = __builtin_fma(X.p1, hx, __builtin_fma(Y.p1, hy, gz)) * A.ih[2];
  }
}

// The coefficient of block point (l, j, k) in every component of the
// gradient (for inspection; the transfers apply the factors directly).
template <int D, int MB>
__device__ __forceinline__ void block_coef(const NodeFit& A, const BlockFit<D, MB>& B, int l, int j,
                                           int k, double (&c)[D]) {
  auto rd = [&](int a, int b, int d) { return a == l && b == j && d == k ? 1.0 : 0.0; };
  block_grad<D, MB>(A, B, rd, c);
}

// ---- grid targets ---------------------------------------------------------------
// A grid point's nodes lie scattered, but its coefficients are the weight
// times a quadratic in the node's offset t (Eq. 13: c_a = w q . (C^-1)_a):
//   c_a(t) = exp(-alpha |t|^2) (l0 + t . l + t . Q t)_a
// so a geometry keeps the d quadratics and alpha (the rows of C^-1 with the
// powers of 1/h_t folded in; their linear parts are symmetric in (a, b)) and
// the transfers evaluate the coefficients from the node positions: 12 (2D) or
// 28 (3D) float64 per grid point instead of 32 or 81 per precision.
constexpr int grid_rows(int d) { return d == 2 ? 12 : 28; }

// The grid points are stored by tiles of 256 points (one workgroup each), their
// shape by the grid (tile_shape).  The stencils of a tile share most of their
// nodes (1.6 distinct ones per point in 2D and 2.8 in 3D against 16 and 27
// entries), so a tile keeps the ascending list of its nodes and each stencil entry is a
// 16-bit place in that list: a workgroup gathers every node once into LDS and
// the entries are read from there (a place is the byte offset of its first
// pair there).  A tile's block of 4 k TP bytes holds the places, two to a
// word, [ceil(k/2)][TP], then the list.  A tile with more nodes than a list
// may hold (a cloud refined there) keeps its coefficients, in float64: its
// block holds the node indices, [k][TP], and its count is the complement of
// its place in GridFit.over; from GridFit.nover on there are none, and every
// entry's position and value are gathered from memory.
constexpr int TILE_LOG = 8;
constexpr int tile_points(int) { return 1 << TILE_LOG; }

// Points of a tile per axis, as powers of two: 32 x 8 and 16 x 4 x 4, or a shape
// that covers a thin or short grid with fewer tiles: the padding points of a
// tile hold rows and places and take threads like the others.  Another shape
// has to save more than an eighth of the tiles, since its nodes are more (32 x
// 2 x 4) or no fewer (8 x 8 x 4).
struct TileShape {
  int lx, ly, lz;

  int64_t tiles(int d, const int32_t* n) const {
    return ((int64_t)n[0] + (1 << lx) - 1 >> lx) * ((int64_t)n[1] + (1 << ly) - 1 >> ly) *
           (d == 2 ? 1 : (int64_t)n[2] + (1 << lz) - 1 >> lz);
  }
};

// rows: whether the geometry keeps rows.  With stored coefficients in 3D a wave's
// gathers touch fewer cache lines in rows of 32 (32 x 4 x 2 against 16 x 4 x 4,
// float32, 8 nodes a cell: 96^3 178 -> 168 us, 128^3 420 -> 402, float64 674 ->
// 626; 100 x 60 x 80, a seventh more tiles, 66 -> 78).
inline TileShape tile_shape(int d, const int32_t* n, bool rows) {
  constexpr TileShape S2[] = {{5, 3, 0}, {4, 4, 0}, {3, 5, 0}, {6, 2, 0}};
  constexpr TileShape S3[] = {{4, 2, 2}, {3, 3, 2}, {3, 2, 3}, {4, 1, 3}, {4, 3, 1},
                              {5, 1, 2}, {5, 2, 1}};
  TileShape best = d == 2 ? S2[0] : (rows ? S3[0] : TileShape{5, 2, 1});
  const int part = rows ? 8 : 16;  // the part of the tiles another shape has to save
  auto take = [&](const TileShape& t) {
    if (part * t.tiles(d, n) < (part - 1) * best.tiles(d, n)) best = t;
  };
  if (d == 2)
    for (const TileShape& t : S2) take(t);
  else
    for (const TileShape& t : S3) take(t);
  return best;
}

// Words of places in a tile's block.
constexpr int64_t tile_words(int d, int k) { return (int64_t)(k + 1) / 2 * tile_points(d); }
// LDS bytes from one node to the next: pairs (x, y), (v_x, v_y) in two planes
// in 2D; (x, y), (z, v_x), (v_y, v_z) next to each other in 3D, where the
// stride of 12 words keeps the lanes of a b128 read in different banks.
constexpr int tile_stride(int d) { return d == 2 ? 16 : 48; }
// Nodes a tile's LDS copy may hold: places are 16 bits, and the list has to
// fit the block.
constexpr int tile_cap(int d, int k) {
  const int64_t room = (int64_t)k * tile_points(d) - tile_words(d, k);
  const int64_t cap = d == 2 ? 2048 : 65536 / tile_stride(3);
  return (int)(cap < room ? cap : room);
}

// Nodes a 3D list may hold while the four workgroups that the registers allow
// still share a compute unit's LDS.  All workgroups of a launch take the LDS of
// its longest list, so a few denser tiles would slow the whole grid: up to 1 in
// LIST_SHARE of the tiles keep coefficients instead, where there are more than
// LIST_TILES (two generations of workgroups): 256^3 with surface points a third
// of a spacing apart 1543 -> 1373 us, 160^3 347 -> 325; on 48^3, one generation,
// 14 us with long lists and 19 with coefficients.  In 2D longer lists cost less
// than coefficients (1024^2 with a refined patch, float64: 42 against 53 us).
constexpr int LIST_NODES = 853, LIST_SHARE = 16, LIST_TILES = 2048;
inline int list_nodes(int d, int k, int64_t ntile) {
  const int cap = tile_cap(d, k);
  return d == 3 && ntile > LIST_TILES && cap > LIST_NODES ? LIST_NODES : cap;
}

struct GridFit {
  int32_t n[3], nt[3];     // grid points and tiles per axis
  int32_t lx, ly;          // points of a tile per axis (TileShape)
  int32_t k;
  int32_t clamp;           // row_weight's exponent needs its clamp
  double off, h[3];
  double L[3], iL[3];      // box length and its inverse on periodic axes, else 0
  int64_t ms;
  const int32_t* blk;      // [ntile][k * TP] words
  const int32_t* cnt;      // [ntile] nodes of the tile's list, or -1
  const double* rows;      // [ntile][grid_rows(d)][TP], or null: stored coefficients
  const double* over;      // [nover][d * k][TP]: coefficients of tiles without a list
  int32_t nover;
  const double* c64;       // [ntile][d * k][TP] (component a, entry i at a * k + i)
  const float* c32;        // or null
  const double* x;         // [d][ms] node positions
};

// Whether a geometry keeps rows at all.  A cloud much finer than the grid shares
// few nodes between grid points: its tiles outgrow their LDS lists from about
// 6 G (2D) or 2.4 G (3D) nodes on, and it streams stored coefficients.
inline bool grid_rows_kept(int d, int64_t G, int64_t M) { return M <= (d == 2 ? 5 : 2) * G; }

// Tiles that may keep coefficients: the sizes known before a build bound what it
// takes, so they are bounded by the nodes beyond one a grid point.  A 2D tile
// over its list has about 1250 of these, a 3D one over LIST_NODES 50 to 250 and
// one over the longest list 500 or more (tiles next to it some less; surface
// points alone, up to 1 in 32, do not fill one).
inline int64_t over_tiles(int d, int64_t ntile, int64_t G, int64_t M) {
  const bool large = d == 3 && ntile > LIST_TILES;
  const int64_t extra = M - G - (d == 3 && !large ? G / 32 : 0);
  if (extra <= 0 || !grid_rows_kept(d, G, M)) return 0;
  const int64_t t = extra / (d == 2 ? 1024 : (large ? 64 : 213));
  return t < ntile ? t : ntile;
}

GridFit grid_fit_args(const pc_geom* g);
inline int64_t grid_tiles(int d, const int32_t* n, bool rows) {
  return tile_shape(d, n, rows).tiles(d, n);
}

// A grid point by tile and place in the tile.
template <int D>
struct TilePoint {
  int64_t tile;
  int t;
  int c[3];  // grid lines

  __device__ __forceinline__ bool inside(const GridFit& A) const {
    return c[0] < A.n[0] && c[1] < A.n[1] && (D == 2 || c[2] < A.n[2]);
  }
  __device__ __forceinline__ int64_t flat(const GridFit& A) const {
    return ((int64_t)c[2] * A.n[1] + c[1]) * A.n[0] + c[0];
  }
  // Rounded as in the build of the rows: fused into the offset below, t would
  // differ from the offset that the rows belong to by 1e-16 of the box, 3e-14 of
  // a spacing at 280 points.
  __device__ __forceinline__ void position(const GridFit& A, double (&xt)[D]) const {
#pragma clang fp contract(off)
#pragma unroll
    for (int a = 0; a < D; ++a) xt[a] = ((double)c[a] + A.off) * A.h[a];
  }
};

template <int D>
__device__ __forceinline__ TilePoint<D> tile_point(const GridFit& A, int64_t tile, int t) {
  TilePoint<D> P;
  P.tile = tile;
  P.t = t;
  const uint32_t r = (uint32_t)tile / (uint32_t)A.nt[0];  // tiles are counted in 31 bits
  const int tx = (int)((uint32_t)tile - r * (uint32_t)A.nt[0]);
  const int tz = D == 3 ? (int)(r / (uint32_t)A.nt[1]) : 0;
  const int ty = (int)r - tz * A.nt[1];
  const int ly = D == 2 ? TILE_LOG - A.lx : A.ly;
  P.c[0] = (tx << A.lx) + (t & ((1 << A.lx) - 1));
  P.c[1] = (ty << ly) + ((t >> A.lx) & ((1 << ly) - 1));
  P.c[2] = D == 3 ? (tz << (TILE_LOG - A.lx - ly)) + (t >> (A.lx + ly)) : 0;
  return P;
}

// The same for flat grid index p.
template <int D>
__device__ __forceinline__ TilePoint<D> tile_point_of(const GridFit& A, int64_t p) {
  TilePoint<D> P;
  const int64_t r = p / A.n[0];
  P.c[0] = (int)(p - r * A.n[0]);
  P.c[2] = D == 3 ? (int)(r / A.n[1]) : 0;
  P.c[1] = (int)(r - (int64_t)P.c[2] * A.n[1]);
  const int lx = A.lx, ly = A.ly, lz = TILE_LOG - lx - ly;
  P.tile = ((int64_t)(P.c[2] >> lz) * A.nt[1] + (P.c[1] >> ly)) * A.nt[0] + (P.c[0] >> lx);
  P.t = ((P.c[2] & ((1 << lz) - 1)) << (lx + ly)) + ((P.c[1] & ((1 << ly) - 1)) << lx) +
        (P.c[0] & ((1 << lx) - 1));
  return P;
}

// Node of entry i of a grid point's stencil.
template <int D>
__device__ __forceinline__ int32_t grid_node(const GridFit& A, const TilePoint<D>& P, int i) {
  constexpr int TP = tile_points(D);
  const int32_t* b = A.blk + P.tile * ((int64_t)A.k * TP);
  if (A.cnt[P.tile] < 0) return b[(int64_t)i * TP + P.t];
  const uint32_t w = (uint32_t)b[(int64_t)(i >> 1) * TP + P.t];
  return b[tile_words(D, A.k) + ((i & 1) ? w >> 16 : w & 0xffffu) / tile_stride(D)];
}

// Row r: constants [D], linear parts (a <= b) [D (D + 1) / 2], squares and
// products (a <= b) [D (D + 1) / 2] per component, -alpha log2(e).
template <int D>
struct GridRows {
  double r[grid_rows(D)];
};

template <int D>
__device__ __forceinline__ GridRows<D> load_rows(const GridFit& A, const TilePoint<D>& P) {
  constexpr int TP = tile_points(D), NR = grid_rows(D);
  const double* b = A.rows + P.tile * ((int64_t)NR * TP) + P.t;
  GridRows<D> R;
#pragma unroll
  for (int i = 0; i < NR; ++i) R.r[i] = __builtin_nontemporal_load(b + i * TP);
  return R;
}

__host__ __device__ constexpr int sym(int d, int a, int b) {
  return a > b ? sym(d, b, a) : (d == 2 ? a + b : (a == 0 ? b : a + b + 1));
}

template <int D, int A>
__device__ __forceinline__ double row_poly_one(const GridRows<D>& R, const double (&t)[D]) {
  constexpr int S = D * (D + 1) / 2, Q = D + S + S * A;
  constexpr int LX = D + sym(D, A, 0), LY = D + sym(D, A, 1), LZ = D + sym(D, A, D - 1);
  double p = R.r[A];
  if constexpr (D == 2) {
    double f = __builtin_fma(t[0], R.r[Q], R.r[LX]);
    p = __builtin_fma(t[0], __builtin_fma(t[1], R.r[Q + 1], f), p);
    p = __builtin_fma(t[1], __builtin_fma(t[1], R.r[Q + 2], R.r[LY]), p);
  } else {
    double f = __builtin_fma(t[0], R.r[Q], R.r[LX]);
    f = __builtin_fma(t[1], R.r[Q + 1], f);
    p = __builtin_fma(t[0], __builtin_fma(t[2], R.r[Q + 2], f), p);
    f = __builtin_fma(t[1], R.r[Q + 3], R.r[LY]);
    p = __builtin_fma(t[1], __builtin_fma(t[2], R.r[Q + 4], f), p);
    p = __builtin_fma(t[2], __builtin_fma(t[2], R.r[Q + 5], R.r[LZ]), p);
  }
  return p;
}

template <int D>
__device__ __forceinline__ void row_poly(const GridRows<D>& R, const double (&t)[D],
                                         double (&P)[D]) {
  P[0] = row_poly_one<D, 0>(R, t);
  P[1] = row_poly_one<D, 1>(R, t);
  if constexpr (D == 3) P[2] = row_poly_one<D, 2>(R, t);
}

// Offset of a node at x from a grid point, the nearest image on periodic axes.
template <int D, bool PER>
__device__ __forceinline__ void grid_offset(const GridFit& A, const double (&x)[D],
                                            const double (&xt)[D], double (&t)[D]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int a = 0; a < D; ++a) {
    t[a] = x[a] - xt[a];
    if (PER) t[a] = __builtin_fma(-A.L[a], __builtin_rint(t[a] * A.iL[a]), t[a]);
  }
}

// exp(-alpha |t|^2) as 2^y, y = -alpha log2(e) |t|^2 = k + f, |f| <= 1/2: the
// product is never rounded on its own (both uses are fused), and the degree-11
// polynomial (the minimax fit of (2^f - 1 - f ln 2) / f^2, its coefficients and
// ln 2 rounded) leaves 2.7e-17.
// Without CLAMP y must stay above -1022; alpha |t|^2 <= eps, so it does up to
// eps = 690 (GridFit.clamp; two more operations an entry than without).
template <int D, bool CLAMP>
__device__ __forceinline__ double row_weight(const GridRows<D>& R, const double (&t)[D]) {
  constexpr double MAGIC = 6755399441055744.0;  // 1.5 2^52
  const double na = R.r[grid_rows(D) - 1];
  double r2 = t[0] * t[0];
#pragma unroll
  for (int a = 1; a < D; ++a) r2 = __builtin_fma(t[a], t[a], r2);
  double m = __builtin_fma(na, r2, MAGIC);
  if (CLAMP) m = fmax(m, MAGIC - 1000.0);
  double f = __builtin_fma(na, r2, MAGIC - m);
  if (CLAMP) f = fmax(f, -0.5);
  double p = 4.4541068401718916193e-10;
  p = __builtin_fma(p, f, 7.0709843005464476907e-9);
  p = __builtin_fma(p, f, 1.0178067252442298443e-7);
  p = __builtin_fma(p, f, 1.3215451605067549985e-6);
  p = __builtin_fma(p, f, 0.000015252733820815905329);
  p = __builtin_fma(p, f, 0.00015403530424814240039);
  p = __builtin_fma(p, f, 0.0013333558146423204744);
  p = __builtin_fma(p, f, 0.0096181291076186498546);
  p = __builtin_fma(p, f, 0.055504108664821582574);
  p = __builtin_fma(p, f, 0.24022650695910076149);
  p = __builtin_fma(p, f, 6.9314718055994530942e-1);
  p = __builtin_fma(p, f, 1.0);
  // the low word of m is k
  const int k = (int)(uint32_t)__builtin_bit_cast(uint64_t, m);
  const uint64_t pb = __builtin_bit_cast(uint64_t, p);
  const uint32_t hi = (uint32_t)(pb >> 32) + ((uint32_t)k << 20);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | (uint32_t)pb);
}

// The coefficients of entry i (node j) of a grid point at xt: from its rows,
// or the stored ones.
template <int D>
__device__ __forceinline__ void grid_coef(const GridFit& A, const TilePoint<D>& P,
                                          const double (&xt)[D], int i, int64_t j,
                                          double (&c)[D]) {
  if (!A.rows) {
    constexpr int TP = tile_points(D);
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const int64_t at = (P.tile * (D * A.k) + a * A.k + i) * TP + P.t;
      c[a] = A.c64 ? A.c64[at] : (double)A.c32[at];
    }
    return;
  }
  const GridRows<D> R = load_rows<D>(A, P);
  double x[D], t[D];
#pragma unroll
  for (int a = 0; a < D; ++a) x[a] = A.x[a * A.ms + j];
  grid_offset<D, true>(A, x, xt, t);
  row_poly<D>(R, t, c);
  const double w = row_weight<D, true>(R, t);
#pragma unroll
  for (int a = 0; a < D; ++a) c[a] *= w;
}

}  // namespace pc
