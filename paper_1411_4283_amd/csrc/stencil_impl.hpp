// Per-face weighted least-squares flux stencils (Sec. 2.2.1, eq. 'stencil equation
// solution'; neighbours, centring and weights of Sec. 2.4).
//
// The stencil s~ = W (A~^T W)^+ F~ is W z with z the minimum-norm solution of
// B^T z = F~, B = W A~ (N x M, N >= M, full column rank): z = B (B^T B)^-1 F~.  One
// wavefront owns one face:
//   1. rows: each lane builds its row(s) of B in registers -- the row's moments,
//      re-centred to x0 by the binomial theorem, divided by the zeroth moment and
//      scaled by the weight -- and puts them in LDS, 64 at a time; a row whose zeroth moment
//      is below kSmallCell is formed in double-double and rounded (the moments of a small
//      cut cell about its centre nearly cancel when shifted to x0);
//   2. G = B^T B on the FP64 matrix cores, rows of B as the contraction index; it stays in
//      their output layout, spread over all 64 lanes (Tile, WaveMatrix);
//   3. G is equilibrated to unit diagonal and inverted in place by symmetric sweeps over
//      blocks of four pivots on the matrix cores, with the right-hand side as one more row;
//      the pivots are the Cholesky pivots;
//   4. z from the semi-normal equations z = B G^-1 F~, a lane's rows times y, followed by one
//      step of refinement
//      with the residual F~ - B^T z computed from B itself in compensated arithmetic
//      (twice the working precision), which leaves the error of rounding B to FP64, a few
//      1e-17 cond(B), where the initial error is ~cond(B)^2 eps;
//   5. val = h^(D-2) W z.
// What bounds it, 64^3 minus a sphere, 3D order 4 (724k faces, 88 rows x 35 columns for most
// of them): the FP64 pipe, which vector FMAs and matrix instructions share on MI355X (32
// flop per cycle and SIMD either way), and the latency between dependent steps that two
// waves per SIMD leave.  8.7 ms; with lane i holding row i of G (29 of 64 lanes idle in the
// sweep, one exchange through LDS per pivot, a transposition of G by lane permutes) and
// every row in LDS (three waves on two SIMDs) it was 17.9 ms in six launches.  Of the 7.8 of
// the faces of up to 96 rows: header 0.6, rows of B 2.2 (3.8 before small cells' rows went by
// lines, coordinates without divisions and loads without flat instructions), G 1.4, sweep 2.0,
// first z 0.5, refinement 1.1 (0.2 in compensated sums).
// Under Neumann EB conditions (a separate kernel instance) the EB rows are the
// normal-derivative rows of eq. 'Neu moment eq for cp' and their values carry h^(D-1);
// the EB faces themselves have a one-entry stencil (their area) and are written by
// k_insufficient, the kernel of faces with fewer rows than monomials.
// Status: fewer rows than monomials or a non-finite entry flag the face.  A face is left to
// the Householder QR path (stencil_qr.hpp), which also decides rank deficiency, when
//   * its condition bound sqrt(||G^||_inf ||G^^-1||_F) (>= cond_2 of the equilibrated B,
//     and within 1.35x of it on the workloads) exceeds kCondRoute: with the rows of small
//     cells formed in double-double (below) the stencil is good to about 1.5e-16 cond,
//     which must stay below the 1e-11 it is held to;
//   * its smallest pivot square root is at most kRouteTol times the largest; or
//   * its refinement step moved the stencil by more than kSettleTol of its size (the error
//     left after the step is about the square of that fraction).
#pragma once

#include <algorithm>

#include "kernels.hpp"
#include "rows.hpp"
#include "rows_dd.hpp"

namespace cutcell {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr double kRouteTol = 1e-4;
constexpr double kRankTol = 1e-12;       // rank deficiency: min |R_kk| <= kRankTol max |R_kk|
constexpr double kCondRoute = 3e4;
constexpr double kSmallCell = 1e-3;      // rows (and EB flux vectors) of smaller cells in double-double
constexpr double kSettleTol = 1e-6;
// Faces whose bound on cond(G^) stays below this (cond(B) below about 3e3) refine in
// plain FP64.  Past it, z = B y and the residuals are summed in compensated arithmetic and
// z is kept as a double-double: the rounding of an FP64 product B y leaves in z a part
// outside the range of B, which the residual cannot see and refinement cannot remove,
// of relative size up to about cond(B) eps (4e-12 at cond(B) = 3e4, the routing bound).
constexpr double kDot2Cond = 1e7;
constexpr int kRefine = 1;
constexpr int kRefineBackward = 2;   // refinement steps of the adjoint's least-squares solve
constexpr int kStatusRoute = 100;        // internal: the face goes to the QR path

// Compensated dot product (Ogita, Rump and Oishi, SIAM J. Sci. Comput. 26(6), 2005,
// algorithm Dot2): s + c holds the running sum as if it were carried in twice the working
// precision.  The product's rounding error comes from the FMA, the sum's from TwoSum.
struct Dot2 {
  double s, c;
};
__device__ __forceinline__ void dot2_add(Dot2& a, double x, double y) {
#pragma clang fp contract(off)
  const double p = x * y;
  const double e = __builtin_fma(x, y, -p);
  const double s = a.s + p;
  const double bb = s - a.s;
  const double q = (a.s - (s - bb)) + (p - bb);
  a.s = s;
  a.c += q + e;
}
// a + b as an unevaluated sum s + c
__device__ __forceinline__ Dot2 dot2_join(Dot2 a, Dot2 b) {
#pragma clang fp contract(off)
  const double s = a.s + b.s;
  const double bb = s - a.s;
  const double q = (a.s - (s - bb)) + (b.s - bb);
  return Dot2{s, (a.c + b.c) + q};
}
__device__ __forceinline__ double dot2_merge(Dot2 a, Dot2 b) {
#pragma clang fp contract(off)
  const double s = a.s + b.s;
  const double bb = s - a.s;
  const double q = (a.s - (s - bb)) + (b.s - bb);
  return s + ((a.c + b.c) + q);
}

// 1/d from v_rcp_f64 and two Newton steps (each squares the relative error)
__device__ __forceinline__ double recip_f64(double d) {
  double r = __builtin_amdgcn_rcp(d);
  double e = fma(-d, r, 1.0);
  r = fma(r, e, r);
  e = fma(-d, r, 1.0);
  return fma(r, e, r);
}


// One row of B = W A~ about x0 (in units of h: x0h = x0 / h) from the row's stored
// moments m (overwritten) and centre; returns its weight in w, and false if the row
// holds a non-finite value.
template <int D, int Q>
__device__ __forceinline__ bool finish_row(const double* ctr, const double* x0h, double* m, double& w, double wpow) {
  constexpr int M = Dims<D, Q>::M;
  double delta[3] = {0, 0, 0};
  double d2 = 0;
  for (int ax = 0; ax < D; ++ax) {
    delta[ax] = ctr[ax] - x0h[ax];
    d2 += delta[ax] * delta[ax];
  }
  w = row_weight(d2, wpow);
  const double mu0 = m[0];
  recentre<D, Q>(m, delta);
  const double sc = w / mu0;
  bool finite = isfinite(sc);
  static_for<0, M>([&](auto I) {
    m[I] *= sc;
    finite = finite && isfinite(m[I]);
  });
  return finite;
}

// Neumann row of EB face e about x0 (eq. 'Neu moment eq for cp'): the flux of each
// monomial xi^p through the face, sum_d p_d nu_d^(p - e_d)(x0), over the face area m^0,
// times the row's weight.  The normal moments are stored about the cut cell's centre
// `ctr` and re-centred to x0 like the other rows.  Returns false on a non-finite value.
template <int D, int Q>
__device__ __forceinline__ bool neumann_row(const GeomPtrs& gp, int32_t e, const double* ctr, const double* x0h,
                                            double* m, double& w, double wpow) {
  constexpr int M = Dims<D, Q>::M, M1 = Dims<D, Q>::M1;
  double delta[3] = {0, 0, 0};
  double d2 = 0;
  for (int ax = 0; ax < D; ++ax) {
    delta[ax] = ctr[ax] - x0h[ax];
    d2 += delta[ax] * delta[ax];
  }
  w = row_weight(d2, wpow);
  const double sc = w / gp.eb_mom[(long long)e * M];
  static_for<0, M>([&](auto I) { m[I] = 0.0; });
  static_for<0, D>([&](auto AX) {
    double nu[M1];
    const double* src = gp.eb_nmom + ((long long)e * D + AX) * M1;
    static_for<0, M1>([&](auto I) { nu[I] = src[I]; });
    recentre<D, Q - 1>(nu, delta);
    static_for<0, M>([&](auto I) {
      constexpr int pd = kMono<D, Q>.e[I][AX];
      if constexpr (pd > 0) {
        constexpr int j = mono_index<D>(kMono<D, Q>.e[I][0] - (AX == 0), kMono<D, Q>.e[I][1] - (AX == 1),
                                        kMono<D, Q>.e[I][2] - (AX == 2));
        m[I] = fma((double)pd, nu[j], m[I]);
      }
    });
  });
  bool finite = isfinite(sc);
  static_for<0, M>([&](auto I) {
    m[I] *= sc;
    finite = finite && isfinite(m[I]);
  });
  return finite;
}

// ---- shape of the Gram matrix in the wave --------------------------------------------------
// G = B^T B (and its inverse) is spread over the wave in the output layout of the FP64
// matrix instructions: with r = lane / 16 and c = lane % 16, register q of tile (I, J) holds
// entry (16 I + r + 4 q, 16 J + c).  The MV (1 to 3) columns past the last full tile are
// kept as rows: ar[J] holds entry (16 MTF + r, 16 J + c) and t entry (16 MTF + r, 16 MTF +
// c % 4).  Row and column M hold the right-hand side while the matrix is inverted.
template <int D, int Q>
struct Tile {
  static constexpr int M = Dims<D, Q>::M, MT = Dims<D, Q>::MT;
  static constexpr int MTF = (MT > 1 && M - 16 * (MT - 1) <= 3) ? MT - 1 : MT;   // full tiles per side
  static constexpr int MV = M - 16 * MTF > 0 ? M - 16 * MTF : 0;                // trailing columns
  static constexpr int PI = 4 * MTF;        // rows of the tiles that one lane holds
  static_assert(MV > 0 || M < 16 * MTF, "the right-hand side needs a free row");
};

// Slot of component i of a vector in shared memory: the PI components of the tile rows of
// one lane (16 I + r + 4 q over I and q) are consecutive, so that a lane reads them with
// 16-byte loads; the trailing components follow.
template <int D, int Q>
__host__ __device__ constexpr int vec_slot(int i) {
  using TL = Tile<D, Q>;
  return i < 16 * TL::MTF ? TL::PI * (i % 4) + i / 4 : i;
}

// The matrix in registers, and the column scales of its rows and columns.
template <int D, int Q>
struct WaveMatrix {
  using TL = Tile<D, Q>;
  double a[TL::MTF][TL::MTF][4];
  double ar[TL::MTF];
  double t;
  double sj[TL::MTF];   // scale of column 16 J + c
  double st, sr;        // of columns 16 MTF + c % 4 and 16 MTF + r
  double sd;            // of component `lane`
};

// The lines of monomials along each direction: idx[dir][line][p] is the one with exponent p in
// `dir`, -1 past the order.
template <int D, int Q>
struct MonoLines {
  static constexpr int L = D == 3 ? (Q + 1) * (Q + 2) / 2 : Q + 1;
  int8_t idx[D][L][Q + 1];
  constexpr MonoLines() : idx{} {
    for (int dir = 0; dir < D; ++dir) {
      int n = 0;
      for (int i = 0; i < kNMono<D, Q>; ++i) {
        if (kMono<D, Q>.e[i][dir] != 0) continue;
        for (int p = 0; p <= Q; ++p) {
          int at = -1;
          for (int j = 0; j < kNMono<D, Q>; ++j) {
            bool same = kMono<D, Q>.e[j][dir] == p;
            for (int a = 0; a < D; ++a) same = same && (a == dir || kMono<D, Q>.e[j][a] == kMono<D, Q>.e[i][a]);
            if (same) at = j;
          }
          idx[dir][n][p] = (int8_t)at;
        }
        ++n;
      }
    }
  }
};
template <int D, int Q>
inline constexpr MonoLines<D, Q> kMonoLines{};

// Rows of small cells by lines of monomials (small_rows) or a lane per row (dd_row).  A row's
// terms unrolled are 27 kB of code in 3D order 4, but 7 kB and less where a row has at most 15
// moments, and there the exchanges cost more than they save: 3D order 4, 64^3 solves 9.14 and
// 1.04 ms (96 and 128 rows) by rows, 8.43 and 0.87 ms by lines; 2D order 4, 256^2 star 329 and
// 335 us; 3D order 2, 47^3 Neumann 816 and 876 us.  With Neumann EB faces, whose own rows need
// the code of dd_row in any case, by rows as well: 3D order 4, whole 40^3 builds 3.80 and 4.20 ms.
template <int D, int Q, bool NEU>
inline constexpr bool kSmallByLines = !NEU && Dims<D, Q>::M > 16;

// rows of small cells formed at a time
template <int D, int Q>
inline constexpr int kSmallBatch = 64 / MonoLines<D, Q>::L < 8 ? 64 / MonoLines<D, Q>::L : 8;

// What the lanes that form a small cell's row have to know of it.
struct SmallRow {
  dd delta[3], scale;     // (centre - x0) / h; weight over zeroth moment
  GlobalPtr<double> src;  // as in RowSource
  int dd_dir, slot;       // direction of a box face, else -1; the row's slot of Bs
};

// Shared memory of one face (one wave): 64 rows of B and one buffer used in turn for the EB
// normal moments, the tile transposition, the pivot blocks and z.  20.3 KB in 3D order 4, so
// that eight waves share the 160 KB of a CU, two on each SIMD; with every row in shared
// memory it was 26 KB at 88 rows and six waves.  The slots hold rows 0..63 (state 0), or
// rows 64 and up in the first slots instead of the ones that belong there (state 1); the
// contents of the slots concerned that are not in place are kept in registers, flat (18 per
// lane for 32 slots), and exchanged (RowSwap).  Rows held in registers row by row (140 a
// lane) left too few for the rest of the solve: 104 spilled, 3 of 13 ms.
template <int D, int Q>
struct FaceSmem {
  static constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS, M1 = Dims<D, Q>::M1;
  static constexpr int S = 64;
  double Bs[S * MS];
  union {
    double nus[D][M1];                              // EB normal moments about x0 (flux vector)
    double tr[256];                                 // one tile, for its transpose
    double vec[40];                                 // a vector that every lane reads
    struct {
      SmallRow small[kSmallBatch<D, Q>];            // rows of small cells being formed
      double slo[kSmallBatch<D, Q> * M];            // the low parts of their entries
    };
    struct {
      double buf[64];                               // the pivot block
      double pv[64];                                // the trailing rows' entries in its columns
    };
    struct {
      double zs[kMaxRows];                          // z = B y
      double zl[kMaxRows];                          // its low part where z is a double-double
    };
    struct {
      double ys[40];                                // y and w of the adjoint
      double wv[40];
      double gx[64];                                // its sums over the rows
      double g0[12];
    };
  };
  double dy[40];                                    // the vector y that multiplies B
};

// c ? x : y by value: between two lvalues ?: selects an address, which would keep a register
// array in memory.
__device__ __forceinline__ double pick(bool c, double x, double y) { return c ? x : y; }

// Everything about the face that the row and flux computations need.
struct FaceInfo {
  int32_t F;
  int gi, kind, dn;
  int32_t ref;
  int64_t n_vol, n_eb, phi0, rp;
  int N;
  double x0h[3];             // x0 / h
  double off[3];             // EB faces: centroid offset from the cut cell's centre (/h)
  int32_t owner_cell;        // EB faces: the cut cell
};

// x0 of the face (in units of h): the face centre, or for an EB face the centroid of its
// cut volume (whose offset from the cell centre is kept in fi.off).  Loads only.
template <int D, int Q>
__device__ __forceinline__ void face_x0(const GridDims& g, const GeomPtrs& gp, FaceInfo& fi) {
  constexpr int M = Dims<D, Q>::M;
  const int dn = fi.dn;
  for (int ax = 0; ax < 3; ++ax) { fi.x0h[ax] = 0.0; fi.off[ax] = 0.0; }
  fi.owner_cell = -1;
  if (fi.kind == 0) {
    int j[3];
    face_coords(g, dn, (int)(fi.ref - g.foff[dn]), j);
    for (int ax = 0; ax < D; ++ax) fi.x0h[ax] = (ax == dn) ? (double)j[ax] : j[ax] + 0.5;
    return;
  }
  const int32_t c = gp.eb_cell[fi.ref];
  fi.owner_cell = c;
  int cown[3];
  cell_coords(g, c, cown);
  const double* vm = gp.vol_mom + (long long)c * M;
  const double k0 = vm[0];
  for (int ax = 0; ax < D; ++ax) {
    fi.off[ax] = vm[1 + ax] / k0;          // first moments: degree-1 monomials e_1..e_D
    fi.x0h[ax] = cown[ax] + 0.5 + fi.off[ax];
  }
}

// x0 / h in double-double: exact for grid and box faces; for an EB face the cut cell's
// centre plus its first moments over its zeroth moment (face_x0 must have run).
template <int D, int Q>
__device__ __forceinline__ void face_x0_dd(const GridDims& g, const GeomPtrs& gp, const FaceInfo& fi, dd* x0) {
  constexpr int M = Dims<D, Q>::M;
  for (int ax = 0; ax < 3; ++ax) x0[ax] = dd_from(fi.x0h[ax]);
  if (fi.kind == 0) return;
  const int32_t c = fi.owner_cell;
  int cown[3];
  cell_coords(g, c, cown);
  const double* vm = gp.vol_mom + (long long)c * M;
  const dd k0 = dd_from(vm[0]);
  for (int ax = 0; ax < D; ++ax) x0[ax] = dd_add(dd_from(cown[ax] + 0.5), dd_div(dd_from(vm[1 + ax]), k0));
}

// Re-centred normal moments of an EB face about x0, component d in lane d, into sm.nus.
template <int D, int Q, class SM>
__device__ __forceinline__ void eb_normal_moments(const GridDims& g, const GeomPtrs& gp, const FaceInfo& fi, SM& sm,
                                                  int lane, const dd* x0dd) {
  constexpr int M = Dims<D, Q>::M, M1 = Dims<D, Q>::M1;
  const bool small = gp.vol_mom[(long long)fi.owner_cell * M] < kSmallCell;
  if (lane < D && !small) {
    double nu[M1];
    const double* src = gp.eb_nmom + ((long long)fi.ref * D + lane) * M1;
    static_for<0, M1>([&](auto I) { nu[I] = src[I]; });
    double dl[3] = {-fi.off[0], -fi.off[1], -fi.off[2]};   // (c - x0)/h
    recentre<D, Q - 1>(nu, dl);
    static_for<0, M1>([&](auto I) { sm.nus[lane][I] = nu[I]; });
  } else if (lane < D) {   // a small cut cell: the shift to its centroid in double-double
    dd nu[M1];
    const double* src = gp.eb_nmom + ((long long)fi.ref * D + lane) * M1;
    static_for<0, M1>([&](auto I) { nu[I] = dd_from(src[I]); });
    const int32_t c = fi.owner_cell;
    int cown[3];
    cell_coords(g, c, cown);
    dd dl[3] = {dd_from(0.0), dd_from(0.0), dd_from(0.0)};
    for (int ax = 0; ax < D; ++ax) dl[ax] = dd_sub(dd_from(cown[ax] + 0.5), x0dd[ax]);   // (c - x0)/h
    recentre_dd<D, Q - 1>(nu, dl);
    static_for<0, M1>([&](auto I) { sm.nus[lane][I] = nu[I].hi + nu[I].lo; });
  }
  lds_order();
}

// Entry `lane` of the flux vector F~ (0 for lanes >= M).
template <int D, int Q, class SM>
__device__ __forceinline__ double face_flux(const GridDims& g, const GeomPtrs& gp, const FaceInfo& fi, SM& sm,
                                            int lane, const dd* x0dd) {
  constexpr int M = Dims<D, Q>::M, Mf = Dims<D, Q>::Mf;
  const int dn = fi.dn;
  double fv = 0.0;
  if (fi.kind == 0) {
    // F~_p = face moment of p - e_d when p_d = 1 (reference normal +e_d)
    const double* fm = gp.face_mom[dn] + (fi.ref - g.foff[dn]) * Mf;
    if (lane < M) {
      constexpr auto& T = kMono<D, Q>;
      const int e0 = T.e[lane][0], e1 = T.e[lane][1], e2 = T.e[lane][2];
      const int pd = (dn == 0) ? e0 : (dn == 1 ? e1 : e2);
      if (pd == 1) {
        int s;
        if (D == 2) s = mono_index<1>(dn == 0 ? e1 : e0, 0, 0);
        else if (dn == 0) s = mono_index<2>(e1, e2, 0);
        else if (dn == 1) s = mono_index<2>(e0, e2, 0);
        else s = mono_index<2>(e0, e1, 0);
        fv = fm[s];
      }
    }
    return fv;
  }
  eb_normal_moments<D, Q>(g, gp, fi, sm, lane, x0dd);
  if (lane < M) {
    constexpr auto& T = kMono<D, Q>;
    for (int ax = 0; ax < D; ++ax) {
      int e[3] = {T.e[lane][0], T.e[lane][1], T.e[lane][2]};
      const int p = e[ax];
      if (p > 0) {
        e[ax] -= 1;
        fv += p * sm.nus[ax][mono_index<D>(e[0], e[1], e[2])];
      }
    }
  }
  lds_order();
  return fv;
}

// The wave's row `lane` of m into slot `lane` of Bs, for the lanes below n.
template <int D, int Q, class SM>
__device__ __forceinline__ void stage_rows(SM& sm, const double* m, int lane, int n) {
  constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS;
  lds_order();
  if (lane < n) static_for<0, M>([&](auto I) { sm.Bs[lane * MS + I] = m[I]; });
  lds_order();
}

// The slots of Bs that rows past 64 take in turn with rows 0, 1, ...: NX of them, flat.
template <int D, int Q, int NX>
struct RowSwap {
  static constexpr int MS = Dims<D, Q>::MS, FL = (NX * MS + 63) / 64;
  double f[FL > 0 ? FL : 1];
  template <class SM>
  __device__ __forceinline__ void save(const SM& sm, int lane) {
    lds_order();
    static_for<0, FL>([&](auto I) { f[I] = sm.Bs[lane + 64 * I]; });
    lds_order();
  }
  template <class SM>
  __device__ __forceinline__ void exchange(SM& sm, int lane) {
    lds_order();
    double t[FL > 0 ? FL : 1];
    static_for<0, FL>([&](auto I) { t[I] = sm.Bs[lane + 64 * I]; });
    lds_order();
    static_for<0, FL>([&](auto I) { sm.Bs[lane + 64 * I] = f[I]; });
    static_for<0, FL>([&](auto I) { f[I] = t[I]; });
    lds_order();
  }
};

// slot `lane` of Bs times the vector dy
template <int D, int Q, class SM>
__device__ __forceinline__ double row_product(const SM& sm, int lane) {
  constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS;
  double p[2] = {0.0, 0.0};
  static_for<0, M>([&](auto J) { p[J % 2] = fma(sm.Bs[lane * MS + J], sm.dy[J], p[J % 2]); });
  return p[0] + p[1];
}
template <int D, int Q, class SM>
__device__ __forceinline__ Dot2 row_product_dot2(const SM& sm, int lane) {
  constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS;
  Dot2 d0{0.0, 0.0}, d1{0.0, 0.0};
#pragma unroll 1
  for (int j = 0; j + 1 < M; j += 2) {
    dot2_add(d0, sm.Bs[lane * MS + j], sm.dy[j]);
    dot2_add(d1, sm.Bs[lane * MS + j + 1], sm.dy[j + 1]);
  }
  if constexpr (M % 2) dot2_add(d0, sm.Bs[lane * MS + M - 1], sm.dy[M - 1]);
  return dot2_join(d0, d1);
}

// G += the n (a multiple of 8) rows in Bs: tiles on and above the diagonal with
// v_mfma_f64_16x16x4f64, the trailing rows with v_mfma_f64_4x4x4f64 (four 4 x 4 blocks: the
// trailing columns against four columns of a tile each, which comes out in the tiles' own
// layout).
template <int D, int Q, class SM>
__device__ __forceinline__ void gram_rows(const SM& sm, int lane, int n, dbl4 (*acc)[Tile<D, Q>::MTF],
                                          WaveMatrix<D, Q>& W) {
  constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS, MTF = Tile<D, Q>::MTF, MV = Tile<D, Q>::MV;
  const int r = lane >> 4, c = lane & 15;
  const double* p = sm.Bs + r * MS;
  for (int k0 = 0; k0 < n; k0 += 8, p += 8 * MS) {
    double x[2][MTF], y[2] = {0.0, 0.0};   // two steps of four rows, loaded together
    static_for<0, 2>([&](auto U) {
      const double* pu = p + 4 * MS * U;
      static_for<0, MTF>([&](auto I) {
        if constexpr (16 * I + 15 < M) x[U][I] = pu[16 * I + c];
        else x[U][I] = pick(16 * I + c < M, pu[(16 * I + c < M) ? 16 * I + c : 0], 0.0);
      });
      if constexpr (MV > 0) y[U] = pick(c % 4 < MV, pu[(c % 4 < MV) ? 16 * MTF + c % 4 : 0], 0.0);
    });
    static_for<0, 2>([&](auto U) {
      static_for<0, MTF>([&](auto I) {
        static_for<I, MTF>([&](auto J) {
          acc[I][J] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[U][I], x[U][J], acc[I][J], 0, 0, 0);
        });
      });
      if constexpr (MV > 0) {
        static_for<0, MTF>([&](auto J) {
          W.ar[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(y[U], x[U][J], W.ar[J], 0, 0, 0);
        });
        W.t = __builtin_amdgcn_mfma_f64_4x4x4f64(y[U], y[U], W.t, 0, 0, 0);
      }
    });
  }
}

// L D L^T of the leading NP x NP block (2 <= NP <= 4) of a symmetric 4 x 4 matrix (d: the
// upper triangle, row by row), alike in every lane: the pivots, their reciprocals and the
// inverse of L below its unit diagonal (m: 10, 20, 21, 30, 31, 32).
template <int NP>
__device__ __forceinline__ void block_factor(const double* d, double* pv, double* rd, double* m) {
  const double a01 = d[1], a02 = d[2], a03 = d[3];
  pv[0] = d[0];
  rd[0] = recip_f64(pv[0]);
  const double l10 = a01 * rd[0], l20 = a02 * rd[0], l30 = a03 * rd[0];
  pv[1] = fma(-l10, a01, d[4]);
  rd[1] = recip_f64(pv[1]);
  m[0] = -l10;
  if constexpr (NP > 2) {
    const double a12 = fma(-l10, a02, d[5]), a13 = fma(-l10, a03, d[6]);
    const double l21 = a12 * rd[1], l31 = a13 * rd[1];
    pv[2] = fma(-l21, a12, fma(-l20, a02, d[7]));
    rd[2] = recip_f64(pv[2]);
    m[1] = fma(l21, l10, -l20);
    m[2] = -l21;
    if constexpr (NP > 3) {
      const double a23 = fma(-l21, a13, fma(-l20, a03, d[8]));
      const double l32 = a23 * rd[2];
      pv[3] = fma(-l32, a23, fma(-l31, a13, fma(-l30, a03, d[9])));
      rd[3] = recip_f64(pv[3]);
      m[3] = fma(-l32, m[1], fma(l31, l10, -l30));
      m[4] = fma(l32, l21, -l31);
      m[5] = -l32;
    }
  }
}

// In-place inverse of the scaled Gram matrix A by symmetric sweeps over blocks of four
// pivots K (A ends as -A^-1; a row that is no pivot ends as itself times A^-1, so row M, the
// right-hand side f, ends as A^-1 f).  With A_KK = L D L^T, R = the block's rows, Y = L^-1 R,
// Z = D^-1 Y and X = L^-T Z:
//   A_ij -= Y_i^T Z_j  (i, j not in K);  A_Kj = X_j;  A_iK = X_i^T;  A_KK = -A_KK^-1.
// (Y^T Z is the update of a Cholesky step, as accurate as one pivot at a time; with A_iK and
// A_KK^-1 A_Kj in its place the error grows by cond(A_KK).)  The rows of a block are one
// register of their tiles, and that register is, lane for lane, the operand that the matrix
// instructions want both for rows of B and, the matrix being symmetric, for columns of A:
// the update is one v_mfma_f64_16x16x4f64 per tile, and Y and X one v_mfma_f64_4x4x4f64 per
// tile column each, with no exchange between lanes.  Only the 4 x 4 block (which every lane
// factors) and the trailing rows' entries in columns K go through shared memory: 9 round
// trips in 3D order 4, where one pivot at a time takes 35, each with loads of the pivot row.
// Columns K come out of the same update with D^-1 L^-1 taken from Z there, and X then holds
// I - A_KK^-1 in them.  Returns in `piv` the pivot of component `lane`.
template <int D, int Q, class SM>
__device__ __forceinline__ void sweep(SM& sm, int lane, WaveMatrix<D, Q>& W, double& piv) {
  using TL = Tile<D, Q>;
  constexpr int M = TL::M, MTF = TL::MTF, MV = TL::MV;
  const int r = lane >> 4, c = lane & 15, s = c & 3;
  static_for<0, (M + 3) / 4>([&](auto KB) {
    constexpr int kb = KB, NP = M - 4 * kb < 4 ? M - 4 * kb : 4;
    constexpr bool TR = 4 * kb >= 16 * MTF;                   // the trailing block
    constexpr int Ip = TR ? 0 : kb / 4, q = kb % 4;
    double R[MTF];
    static_for<0, MTF>([&](auto J) {
      if constexpr (TR) R[J] = W.ar[J];
      else R[J] = W.a[Ip][J][q];
    });
    lds_order();
    if constexpr (TR) sm.buf[lane] = W.t;
    else sm.buf[lane] = R[Ip];
    if constexpr (MV > 0 && !TR) sm.pv[4 * c + r] = W.ar[Ip];
    lds_order();
    constexpr int off = TR ? 0 : 4 * q;
    double d[10];
    static_for<0, 4>([&](auto I) {
      static_for<I, 4>([&](auto J) { d[4 * I - I * (I - 1) / 2 + (J - I)] = sm.buf[16 * I + off + J]; });
    });
    double T = 0.0;                                           // columns of the trailing rows: entry (K_r, s)
    if constexpr (TR) T = W.t;
    else if constexpr (MV > 0) T = sm.pv[4 * (4 * q + r) + s];
    double pv[4], rd[4], m[6];
    block_factor<NP>(d, pv, rd, m);
    static_for<0, NP>([&](auto I) { piv = pick(lane == 4 * kb + I, pv[I], piv); });
    // L^-1 as the two operands: V entry (r, s), U entry (s, r); 1/d_r
    double V = (r == s && r < NP) ? 1.0 : 0.0, U = V;
    double rr = pick(r == 1, rd[1], rd[0]);
    V = pick(r == 1 && s == 0, m[0], V);
    U = pick(s == 1 && r == 0, m[0], U);
    if constexpr (NP > 2) {
      rr = pick(r == 2, rd[2], rr);
      static_for<0, 2>([&](auto I) {
        V = pick(r == 2 && s == I, m[1 + I], V);
        U = pick(s == 2 && r == I, m[1 + I], U);
      });
    }
    if constexpr (NP > 3) {
      rr = pick(r == 3, rd[3], rr);
      static_for<0, 3>([&](auto I) {
        V = pick(r == 3 && s == I, m[3 + I], V);
        U = pick(s == 3 && r == I, m[3 + I], U);
      });
    }
    // Y, -Z (with columns K put in place) and -X
    const bool inK = (TR || c / 4 == q) && (NP == 4 || s < NP);
    const double zK = inK ? V * rr : 0.0, xK = (inK && r == s) ? 1.0 : 0.0;
    double Y[MTF], Z[MTF], X[MTF], YT = 0.0, ZT = 0.0, XT = 0.0;
    static_for<0, MTF>([&](auto J) {
      Y[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(U, R[J], 0.0, 0, 0, 0);
      Z[J] = -Y[J] * rr;
      if constexpr (!TR && J == Ip) Z[J] += zK;
      X[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(V, Z[J], 0.0, 0, 0, 0);
      if constexpr (!TR && J == Ip) X[J] += xK;
    });
    if constexpr (MV > 0) {
      YT = __builtin_amdgcn_mfma_f64_4x4x4f64(U, T, 0.0, 0, 0, 0);
      ZT = -YT * rr;
      if constexpr (TR) {
        ZT += zK;
        XT = __builtin_amdgcn_mfma_f64_4x4x4f64(V, ZT, 0.0, 0, 0, 0) + xK;
      }
    }
    static_for<0, MTF>([&](auto I) {
      static_for<0, MTF>([&](auto J) {
        dbl4 t = {W.a[I][J][0], W.a[I][J][1], W.a[I][J][2], W.a[I][J][3]};
        t = __builtin_amdgcn_mfma_f64_16x16x4f64(Y[I], Z[J], t, 0, 0, 0);
        static_for<0, 4>([&](auto QQ) { W.a[I][J][QQ] = t[(int)QQ]; });
      });
    });
    if constexpr (MV > 0) {
      static_for<0, MTF>([&](auto J) {
        W.ar[J] = __builtin_amdgcn_mfma_f64_4x4x4f64(YT, Z[J], W.ar[J], 0, 0, 0);
      });
      W.t = __builtin_amdgcn_mfma_f64_4x4x4f64(YT, ZT, W.t, 0, 0, 0);
    }
    // rows K
    const bool rowK = NP == 4 || r < NP;
    static_for<0, MTF>([&](auto J) {
      if constexpr (TR) W.ar[J] = pick(rowK, -X[J], W.ar[J]);
      else W.a[Ip][J][q] = pick(rowK, -X[J], W.a[Ip][J][q]);
    });
    if constexpr (TR) W.t = pick(rowK, -XT, W.t);
  });
}

// dy = E (-W) x, the scaled inverse times x (component `lane` in lane `lane`, 0 from M on; x
// already carries its factor E), into sm.dy.
template <int D, int Q, class SM>
__device__ __forceinline__ void apply_inverse(SM& sm, int lane, const WaveMatrix<D, Q>& W, double x) {
  using TL = Tile<D, Q>;
  constexpr int M = TL::M, MTF = TL::MTF, MV = TL::MV, PI = TL::PI;
  const int r = lane >> 4, c = lane & 15;
  lds_order();
  if (lane < 16 * MTF + (MV > 0 ? 4 : 0)) sm.vec[vec_slot<D, Q>(lane)] = x;
  lds_order();
  double xr = 0.0;
  if constexpr (MV > 0) xr = sm.vec[16 * MTF + r];
  double xi[MTF][4];
  static_for<0, MTF>([&](auto I) { static_for<0, 4>([&](auto QQ) { xi[I][QQ] = sm.vec[PI * r + 4 * I + QQ]; }); });
  double y[MTF];
  static_for<0, MTF>([&](auto J) {
    double s0 = W.ar[J] * xr, s1 = 0.0;
    if constexpr (MV == 0) s0 = 0.0;
    static_for<0, MTF>([&](auto I) {
      static_for<0, 4>([&](auto QQ) {
        if constexpr (QQ % 2 == 0) s0 = fma(W.a[I][J][QQ], xi[I][QQ], s0);
        else s1 = fma(W.a[I][J][QQ], xi[I][QQ], s1);
      });
    });
    y[J] = sum_lane_rows(s0 + s1);
  });
  double yt = 0.0;
  if constexpr (MV > 0) {
    yt = (c < MV) ? W.t * sm.vec[16 * MTF + c % 4] : 0.0;
    static_for<0, MTF>([&](auto J) { yt = fma(W.ar[J], sm.vec[PI * (c % 4) + c / 4 + 4 * J], yt); });
    yt = sum_in_lane_row(yt);
  }
  lds_order();
  if (r == 0) static_for<0, MTF>([&](auto J) { if (16 * J + c < M) sm.dy[16 * J + c] = -(y[J] * W.sj[J]); });
  if constexpr (MV > 0)
    if (c == 0 && r < MV) sm.dy[16 * MTF + r] = -(yt * W.sr);
  lds_order();
}

// sum of -Bs[i][lane] z[i] over the first n (a multiple of 8) slots of Bs, z at zs[i + zoff]:
// two sums in turn
template <int D, int Q, class SM>
__device__ __forceinline__ void column_sum(const SM& sm, int lane, int n, int zoff, double& p0, double& p1) {
  constexpr int MS = Dims<D, Q>::MS;
  for (int i = 0; i < n; i += 8) {
    static_for<0, 8>([&](auto U) {
      const double b = sm.Bs[(i + U) * MS + lane], z = sm.zs[i + zoff + U];
      if constexpr (U % 2 == 0) p0 = fma(-b, z, p0);
      else p1 = fma(-b, z, p1);
    });
  }
}

// the same compensated, the low part of z in the compensation
template <int D, int Q, class SM>
__device__ __forceinline__ void column_sum_dot2(const SM& sm, int lane, int n, int zoff, Dot2& d0, Dot2& d1,
                                                double& lo) {
  constexpr int MS = Dims<D, Q>::MS;
  for (int i = 0; i < n; i += 2) {
    const double b0 = -sm.Bs[i * MS + lane], b1 = -sm.Bs[(i + 1) * MS + lane];
    dot2_add(d0, b0, sm.zs[i + zoff]);
    dot2_add(d1, b1, sm.zs[i + zoff + 1]);
    lo = fma(b0, sm.zl[i + zoff], lo);
    lo = fma(b1, sm.zl[i + zoff + 1], lo);
  }
}

// One direction's re-centring of line `ln` of a row (entries hi + lo, read from the row's
// moments in the first direction), scaled in the last: the same sums in the same order as in
// dd_row.  Returns false if it left a non-finite value.
template <int D, int Q>
__device__ __forceinline__ bool line_shift(int dir, int ln, const dd& delta, const dd& scale, const double* src,
                                           int dd_dir, double* hi, double* lo) {
  int id[Q + 1];
  dd m[Q + 1], pw[Q + 1];
  static_for<0, Q + 1>([&](auto I) {
    id[I] = kMonoLines<D, Q>.idx[dir][ln][I];
    m[I] = dd_from(0.0);
    if (id[I] >= 0) {
      if (dir > 0) m[I] = dd{hi[id[I]], lo[id[I]]};
      else {
        const int sl = dd_dir < 0 ? id[I] : face_slot<D, Q>(id[I], dd_dir);
        if (sl >= 0) m[I] = dd_from(src[sl]);
      }
    }
  });
  pw[0] = dd_from(1.0);
  static_for<1, Q + 1>([&](auto K) { pw[K] = dd_mul(pw[K - 1], delta); });
  static_for_down<1, Q + 1>([&](auto I) {
    dd acc = m[I];
    static_for<0, I>([&](auto C) {
      acc = dd_add(acc, dd_mul(dd_mul_d(pw[I - C], (double)binom(I, C)), m[C]));
    });
    m[I] = acc;
  });
  bool finite = true;
  if (dir == D - 1)
    static_for<0, Q + 1>([&](auto I) {
      m[I] = dd_mul(m[I], scale);
      finite = finite && (id[I] < 0 || dd_isfinite(m[I]));
    });
  static_for<0, Q + 1>([&](auto I) {
    if (id[I] >= 0) {
      hi[id[I]] = m[I].hi;
      lo[id[I]] = m[I].lo;
    }
  });
  return finite;
}

// The rows of the lanes in `mask` (this lane's: `rs`) in double-double, rounded into their
// slots of Bs; sets their weights.  A lane takes a line of monomials of a row, direction after
// direction -- the shifts of a line by the binomial theorem are the same sums in the same order
// as in recentre_dd -- and passes the results on through shared memory, so that a few small
// cells keep all lanes busy and the code is a loop over the directions.  One lane per row and
// its 105 unrolled terms (27 kB of code, run for every face near a small cell) took 0.92 of
// 9.14 ms of the 64^3 order-4 solves of up to 96 rows, 0.28 ms like this.
template <int D, int Q, class SM>
__device__ __forceinline__ void small_rows(SM& sm, int lane, unsigned long long mask, const RowSource& rs,
                                           const dd* x0, double wpow, double& w, bool& finite) {
  constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS, LN = MonoLines<D, Q>::L, P = kSmallBatch<D, Q>;
  const bool mine = (mask >> lane) & 1;
  const int rank = __popcll(mask & ((1ULL << lane) - 1)), n = __popcll(mask);
  SmallRow me{};
  if (mine) {
    double d2 = 0.0;
    for (int ax = 0; ax < 3; ++ax) me.delta[ax] = dd_from(0.0);
    for (int ax = 0; ax < D; ++ax) {
      me.delta[ax] = dd_sub(dd_from(rs.ctr[ax]), x0[ax]);
      d2 += me.delta[ax].hi * me.delta[ax].hi;
    }
    w = row_weight(d2, wpow);
    me.scale = dd_div(dd_from(w), dd_from(rs.src[0]));
    finite = finite && dd_isfinite(me.scale);
    me.src = rs.src;
    me.dd_dir = rs.dd;
    me.slot = lane;
  }
  const int k = lane / LN, ln = lane % LN;
#pragma unroll 1
  for (int b0 = 0; b0 < n; b0 += P) {
    lds_order();
    if (mine && rank >= b0 && rank < b0 + P) sm.small[rank - b0] = me;
    lds_order();
    const bool on = k < P && b0 + k < n;
    const SmallRow& row = sm.small[on ? k : 0];
    double* hi = sm.Bs + row.slot * MS;
    double* lo = sm.slo + (on ? k : 0) * M;
#pragma unroll 1
    for (int dir = 0; dir < D; ++dir) {
      if (on) finite = line_shift<D, Q>(dir, ln, row.delta[dir], row.scale, row.src, row.dd_dir, hi, lo) && finite;
      lds_order();
    }
  }
}

// Rows, Gram matrix, inverse and the refined semi-normal solve of one face with at most
// NPAD (64, 96 or 128) rows.  Leaves rows 0..63 of B in Bs and the ones past 64 in sw, the
// inverse in W, weights and z of rows lane and lane + 64 in wreg[], zreg[], and component
// `lane` of y in y.  Returns the face status, or kStatusRoute.
template <int D, int Q, int NPAD, bool NEU, class SM>
__device__ __forceinline__ int face_forward(const GridDims& g, const GeomPtrs& gp, const FaceInfo& fi,
                                            const int32_t* __restrict__ vol_cell, const int32_t* __restrict__ box_lf,
                                            const int32_t* __restrict__ col, SM& sm, int lane, WaveMatrix<D, Q>& W,
                                            RowSwap<D, Q, NPAD - 64>& sw, double* wreg, double* zreg, double& y,
                                            double wpow, bool* rank_low = nullptr) {
  using DM = Dims<D, Q>;
  using TL = Tile<D, Q>;
  constexpr int M = DM::M, MS = DM::MS, MTF = TL::MTF, MV = TL::MV, PI = TL::PI, NR = (NPAD + 63) / 64;
  const int N = fi.N;
  // rows in Bs (n0) and past 64 (n1), in eights (the rows past N are zero)
  const int n0 = (NR > 1 && N > 64) ? 64 : ((N + 7) & ~7);
  const int n1 = (NR > 1 && N > 64) ? ((N - 64 + 7) & ~7) : 0;

  // ---- rows of B ----------------------------------------------------------------------
  // Lane r builds rows r and r + 64: every row's index chain (col -> cell -> moments) is
  // issued before the first row is finished, so the dependent loads of all rows overlap.
  // The rows of small cells come from a second pass, which only the faces that have some
  // take.
  bool finite = true;
  dd x0dd[3];
  face_x0_dd<D, Q>(g, gp, fi, x0dd);
  RowSource rsrc[NR];
  static_for<0, NR>([&](auto R) {
    const int r = lane + 64 * R;
    if (r < N) rsrc[R] = row_source<D, Q>(g, gp, (int64_t)col[fi.rp + r] - fi.phi0, fi.n_vol, fi.n_eb, vol_cell,
                                          box_lf);
  });
  double b1[M];       // row lane + 64
  bool small[NR];
  static_for<0, NR>([&](auto R) {
    const int r = lane + 64 * R;
    double m[M];
    double wr = 0.0;
    small[R] = false;
    static_for<0, M>([&](auto I) { m[I] = 0.0; });
    if (r < N) {
      const bool neu_row = NEU && rsrc[R].eb >= 0;
      bool fin;
      if (neu_row) {
        small[R] = !(gp.eb_mom[(long long)rsrc[R].eb * M] >= kSmallCell);
        fin = neumann_row<D, Q>(gp, rsrc[R].eb, rsrc[R].ctr, fi.x0h, m, wr, wpow);
      } else {
        load_row_moments<D, Q>(rsrc[R], m);
        small[R] = !(m[0] >= kSmallCell);   // (or a non-finite moment)
        fin = finish_row<D, Q>(rsrc[R].ctr, fi.x0h, m, wr, wpow);
      }
      finite = finite && (fin || small[R]);
    }
    wreg[R] = wr;
    if constexpr (R == 0) stage_rows<D, Q>(sm, m, lane, FaceSmem<D, Q>::S);
    else static_for<0, M>([&](auto I) { b1[I] = m[I]; });
  });
  // row lane + 64 R of a small cell in double-double, into the lane's slot
  auto small_row = [&](auto R) {
    if constexpr (kSmallByLines<D, Q, NEU>) {
      const unsigned long long mask = __ballot(small[R]);
      if (mask) small_rows<D, Q>(sm, lane, mask, rsrc[R], x0dd, wpow, wreg[R], finite);
    } else if (small[R]) {
      dd md[M];
      finite = dd_row<D, Q, NEU>(gp, rsrc[R], x0dd, wpow, md, wreg[R]) && finite;
      static_for<0, M>([&](auto I) { sm.Bs[lane * MS + I] = md[I].hi; });
    }
    lds_order();
  };
  small_row(std::integral_constant<int, 0>{});
  const double fv = face_flux<D, Q>(g, gp, fi, sm, lane, x0dd);

  // ---- G = B^T B --------------------------------------------------------------------------
  const int r = lane >> 4, c = lane & 15;
  {
    dbl4 acc[MTF][MTF];
    static_for<0, MTF>([&](auto I) {
      static_for<0, MTF>([&](auto J) { acc[I][J] = dbl4{0, 0, 0, 0}; });
      W.ar[I] = 0.0;
    });
    W.t = 0.0;
    lds_order();
    gram_rows<D, Q>(sm, lane, n0, acc, W);
    if constexpr (NR > 1) {
      sw.save(sm, lane);
      stage_rows<D, Q>(sm, b1, lane, n1);
      small_row(std::integral_constant<int, 1>{});
      gram_rows<D, Q>(sm, lane, n1, acc, W);   // the slots are left in state 1
    }
    static_for<0, MTF>([&](auto I) {
      static_for<I, MTF>([&](auto J) { static_for<0, 4>([&](auto QQ) { W.a[I][J][QQ] = acc[I][J][(int)QQ]; }); });
    });
    // the tile below the diagonal is the transpose of the one above (skewed slots: no bank
    // conflicts); as another tile of the matrix instructions it would cost ten times as much
    if constexpr (MTF == 2) {
      lds_order();
      static_for<0, 4>([&](auto QQ) { sm.tr[16 * (r + 4 * QQ) + ((c + r + 4 * QQ) & 15)] = W.a[0][1][QQ]; });
      lds_order();
      static_for<0, 4>([&](auto QQ) { W.a[1][0][QQ] = sm.tr[16 * c + ((r + 4 * QQ + c) & 15)]; });
      lds_order();
    }
  }

  const bool allfinite = __all(finite) && __all(isfinite(fv));

  // ---- equilibrate to unit diagonal ---------------------------------------------------------
  // E = 1/sqrt(diag G); the diagonal goes through shared memory to component order and E
  // back to the rows and columns
  const bool act = lane < M;
  {
    static_for<0, MTF>([&](auto J) {
      double dg = W.a[J][J][0];
      static_for<1, 4>([&](auto QQ) { dg = pick(c / 4 == QQ, W.a[J][J][QQ], dg); });
      if (r == c % 4) sm.dy[16 * J + c] = dg;
    });
    if constexpr (MV > 0)
      if (r == c) sm.dy[16 * MTF + c] = W.t;
    lds_order();
    W.sd = act ? 1.0 / sqrt(sm.dy[lane < 40 ? lane : 0]) : 1.0;
    lds_order();
    if (lane < 16 * MTF + (MV > 0 ? 4 : 0)) sm.vec[vec_slot<D, Q>(lane)] = W.sd;
    if (lane < 40) sm.dy[lane] = act ? fv * W.sd : 0.0;      // the scaled right-hand side
    lds_order();
    double si[MTF][4];
    static_for<0, MTF>([&](auto I) {
      static_for<0, 4>([&](auto QQ) { si[I][QQ] = sm.vec[PI * r + 4 * I + QQ]; });
      W.sj[I] = sm.vec[PI * (c % 4) + c / 4 + 4 * I];
    });
    W.st = W.sr = 0.0;
    if constexpr (MV > 0) {
      W.sr = sm.vec[16 * MTF + r];
      W.st = sm.vec[16 * MTF + c % 4];
    }
    static_for<0, MTF>([&](auto J) {
      static_for<0, MTF>([&](auto I) {
        static_for<0, 4>([&](auto QQ) { W.a[I][J][QQ] *= si[I][QQ] * W.sj[J]; });
      });
      W.ar[J] *= W.sr * W.sj[J];
    });
    W.t *= W.sr * W.st;
  }
  // ||G^||_inf: the largest absolute column sum of the equilibrated Gram matrix
  double gnorm = 0.0;
  static_for<0, MTF>([&](auto J) {
    double s = (MV > 0) ? fabs(W.ar[J]) : 0.0;
    static_for<0, MTF>([&](auto I) { static_for<0, 4>([&](auto QQ) { s += fabs(W.a[I][J][QQ]); }); });
    gnorm = fmax(gnorm, sum_lane_rows(s));
  });
  if constexpr (MV > 0) {
    double s = (c < MV) ? fabs(W.t) : 0.0;
    static_for<0, MTF>([&](auto J) { s += fabs(W.ar[J]); });
    gnorm = fmax(gnorm, sum_in_lane_row(s));
  }
  // the right-hand side E F~ as row and column M
  if constexpr (MV > 0) {
    static_for<0, MTF>([&](auto J) { W.ar[J] = pick(r == MV, sm.dy[16 * J + c], W.ar[J]); });
    W.t = pick(r == MV, sm.dy[16 * MTF + c % 4], pick(c % 4 == MV, sm.dy[16 * MTF + r], W.t));
  } else {
    constexpr int rM = M % 4, qM = M / 4;
    W.a[0][0][qM] = pick(r == rM, sm.dy[c], W.a[0][0][qM]);
    static_for<0, 4>([&](auto QQ) { W.a[0][0][QQ] = pick(c == M, sm.dy[r + 4 * QQ], W.a[0][0][QQ]); });
  }

  // ---- invert; the pivots are the Cholesky pivots L_kk^2 -----------------------------------
  double piv = 0.0;
  sweep<D, Q>(sm, lane, W, piv);
  const double pd = piv > 0.0 ? piv : 0.0;       // (the tests square their bounds)
  const double pmax = wave_max_f64(act ? pd : 0.0);
  const double pmin = -wave_max_f64(act ? -pd : -1e300);
  const bool pivots_ok = (pmin > kRouteTol * kRouteTol * pmax) && (pmax > 0.0);
  double inv2 = 0.0;    // ||G^^-1||_F^2, from the entries of the inverse
  static_for<0, MTF>([&](auto J) {
    static_for<0, MTF>([&](auto I) {
      static_for<0, 4>([&](auto QQ) {
        const double v = pick(MV > 0 || (c < M && r + 4 * QQ < M), W.a[I][J][QQ], 0.0);
        inv2 = fma(v, v, inv2);
      });
    });
  });
  if constexpr (MV > 0) {
    double s = 0.0;   // the trailing rows, and the columns they stand for
    static_for<0, MTF>([&](auto J) { s = fma(W.ar[J], W.ar[J], s); });
    if (r < MV) inv2 = fma(2.0, s, inv2);
    if (r < MV && c < MV) inv2 = fma(W.t, W.t, inv2);
  }
  gnorm = wave_max_f64(gnorm);
  inv2 = sum_lane_rows(sum_in_lane_row(inv2));
  const double cbound = gnorm * sqrt(inv2);   // wave-uniform
  const bool cond_ok = cbound <= kCondRoute * kCondRoute;
  const bool dot2 = !(cbound <= kDot2Cond);

  // ---- semi-normal solve with one refinement step (compensated past kDot2Cond) ---------
  // y = G^-1 F~, with G^ = E G E: the first y is row M times E.  Lane r holds z of its rows
  // r, r + 64 (past kDot2Cond as zreg + zlo).
  lds_order();
  if constexpr (MV > 0) {
    if (r == MV) {
      static_for<0, MTF>([&](auto J) { sm.dy[16 * J + c] = W.ar[J] * W.sj[J]; });
      if (c < MV) sm.dy[16 * MTF + c] = W.t * W.st;
    }
  } else {
    if (r == M % 4 && c < M) sm.dy[c] = W.a[0][0][M / 4] * W.sj[0];
  }
  lds_order();
  y = 0.0;
  double dlast = 0.0;   // largest change of W z in the refinement step
  double zlo[NR];
  static_for<0, NR>([&](auto R) {
    zreg[R] = 0.0;
    zlo[R] = 0.0;
  });
  for (int it = 0; it <= kRefine; ++it) {
    if (act) y += sm.dy[lane];
    // z += B dy: the rows past 64 in state 1, then the others in state 0
    static_for_down<0, NR>([&](auto R) {
      double inc;
      if (dot2) {
        const Dot2 d = row_product_dot2<D, Q>(sm, lane);
        const dd zs2 = dd_add(dd{zreg[R], zlo[R]}, dd{d.s, d.c});
        zreg[R] = (R == 0 || lane < n1) ? zs2.hi : 0.0;
        zlo[R] = (R == 0 || lane < n1) ? zs2.lo : 0.0;
        inc = d.s + d.c;
      } else {
        inc = row_product<D, Q>(sm, lane);
        zreg[R] = (R == 0 || lane < n1) ? zreg[R] + inc : 0.0;
      }
      if (it == kRefine) dlast = fmax(dlast, fabs(wreg[R] * inc));
      if constexpr (R > 0) sw.exchange(sm, lane);
    });
    if (it == kRefine) break;
    // residual of B^T z = F~ (two interleaved sums, compensated past kDot2Cond, where the
    // low part of z enters the compensation); z goes through shared memory, B^T is read by
    // columns: rows 0..63, then the ones past 64
    lds_order();
    static_for<0, NR>([&](auto R) {
      sm.zs[lane + 64 * R] = zreg[R];
      if (dot2) sm.zl[lane + 64 * R] = zlo[R];
    });
    lds_order();
    double res = 0.0;
    const int cl = act ? lane : 0;
    if (dot2) {
      Dot2 d0{fv, 0.0}, d1{0.0, 0.0};
      double lo = 0.0;
      column_sum_dot2<D, Q>(sm, cl, n0, 0, d0, d1, lo);
      if constexpr (NR > 1) {
        sw.exchange(sm, lane);
        column_sum_dot2<D, Q>(sm, cl, n1, 64, d0, d1, lo);
      }
      d1.c += lo;
      res = dot2_merge(d0, d1);
    } else {
      double p0 = fv, p1 = 0.0;
      column_sum<D, Q>(sm, cl, n0, 0, p0, p1);
      if constexpr (NR > 1) {
        sw.exchange(sm, lane);
        column_sum<D, Q>(sm, cl, n1, 64, p0, p1);
      }
      res = p0 + p1;
    }
    apply_inverse<D, Q>(sm, lane, W, act ? res * W.sd : 0.0);
  }
  if (dot2) static_for<0, NR>([&](auto R) { zreg[R] += zlo[R]; });
  // has the refinement settled?  The step's change of the stencil W z against its size
  double smax = 0.0;
  static_for<0, NR>([&](auto R) { smax = fmax(smax, fabs(wreg[R] * zreg[R])); });
  dlast = wave_max_f64(dlast);
  smax = wave_max_f64(smax);
  const bool settled = dlast <= kSettleTol * smax;
  if (rank_low) *rank_low = !((pmin > kRankTol * kRankTol * pmax) && (pmax > 0.0));
  if (!allfinite) return CUTCELL_STATUS_NONFINITE;
  if (!pivots_ok || !cond_ok || !settled) return kStatusRoute;
  return CUTCELL_STATUS_OK;
}

struct StencilArgs {
  GridDims g;
  int G;
  double hscale;
  const int32_t* perm;
  long long nbin;
  const int32_t* fcode;
  const int32_t* fref;
  const GeomPtrs* geoms;
  const int64_t* counts;
  const int64_t* offs;
  const int32_t* vol_cell_ws;
  const int32_t* box_lf_ws;
  const int64_t* row_ptr;
  const int32_t* col;
  // schedule: workgroup b runs on XCD b % xcd (the dispatcher deals workgroups out to the
  // XCDs in turn) and walks that XCD's contiguous chunk of the bin with stride per_xcd
  int xcd;
  int per_xcd;
  double h;            // grid spacing (Neumann rows carry one more power of h)
  double wpow;         // weight exponent p of W = (2 |delta|)^-p
  int32_t* qr_list;    // faces left to the Householder QR path, and their count
  int32_t* qr_count;
  int route;           // 1: such faces go to the QR path; 0: the Gram path keeps every face
};

// Faces of a bin taken by workgroup blockIdx.x in turn (-1 when done).  With xcd = 1 and a
// grid of nbin workgroups this is one face per workgroup in bin order.
struct FaceWalk {
  long long chunk, k, base;
  int step;
  __device__ FaceWalk(const StencilArgs& A) {
    const int b = blockIdx.x;
    chunk = (A.nbin + A.xcd - 1) / A.xcd;
    base = (long long)(b % A.xcd) * chunk;
    k = b / A.xcd;
    step = A.per_xcd;
  }
  __device__ long long next() {
    if (k >= chunk) return -1;
    const long long t = base + k;
    k += step;
    return t;
  }
};

__device__ __forceinline__ FaceInfo face_info(const StencilArgs& A, long long t) {
  FaceInfo fi;
  fi.F = __builtin_amdgcn_readfirstlane(A.perm[t]);
  const int32_t code = __builtin_amdgcn_readfirstlane(A.fcode[fi.F]);
  fi.gi = code >> 4;
  fi.kind = (code >> 2) & 3;
  fi.dn = code & 3;
  fi.ref = __builtin_amdgcn_readfirstlane(A.fref[fi.F]);
  fi.n_vol = A.counts[4 * fi.gi + 0];
  fi.n_eb = A.counts[4 * fi.gi + 1];
  fi.phi0 = A.offs[fi.gi];
  fi.rp = A.row_ptr[fi.F];
  fi.N = __builtin_amdgcn_readfirstlane((int)(A.row_ptr[fi.F + 1] - fi.rp));
  return fi;
}

// One face per workgroup (WALK = false: face t of the bin, t from the XCD mapping), or a
// persistent workgroup that walks its chunk (WALK = true).  Two instances because the
// loop costs the single-face kernel registers.
template <int D, int Q, int NPAD, bool NEU>
__device__ __forceinline__ void stencil_face(const StencilArgs& A, long long t, FaceSmem<D, Q>& sm, int lane,
                                             double* __restrict__ val, int8_t* __restrict__ status, int32_t* flagged) {
  constexpr int NR = (NPAD + 63) / 64;
  FaceInfo fi = face_info(A, t);
  const GeomPtrs& gp = A.geoms[fi.gi];
  face_x0<D, Q>(A.g, gp, fi);
  WaveMatrix<D, Q> W;
  RowSwap<D, Q, NPAD - 64> sw;
  double wreg[NR], zreg[NR], y;
  bool rank_low = false;
  int st = face_forward<D, Q, NPAD, NEU>(A.g, gp, fi, A.vol_cell_ws + (long long)fi.gi * A.g.ncell,
                                         A.box_lf_ws + (long long)fi.gi * A.g.nboxslot, A.col, sm, lane, W, sw, wreg,
                                         zreg, y, A.wpow, &rank_low);
  if (st == kStatusRoute) {
    if (A.route) {   // the QR path writes this face's values and status
      if (lane == 0) A.qr_list[atomicAdd(A.qr_count, 1)] = fi.F;
      return;
    }
    st = rank_low ? CUTCELL_STATUS_RANK_DEFICIENT : CUTCELL_STATUS_OK;
  }
  static_for<0, NR>([&](auto R) {
    const int r = lane + 64 * R;
    if (r < fi.N) {
      double v = (st == CUTCELL_STATUS_OK) ? A.hscale * wreg[R] * zreg[R] : 0.0;
      if constexpr (NEU) {
        const int64_t k = (int64_t)A.col[fi.rp + r] - fi.phi0;
        if (k >= fi.n_vol && k < fi.n_vol + fi.n_eb) v *= A.h;
      }
      val[fi.rp + r] = v;
    }
  });
  if (lane == 0) {
    status[fi.F] = (int8_t)st;
    if (st != CUTCELL_STATUS_OK) atomicAdd(flagged, 1);
  }
}

// Waves per SIMD that the kernels are built for: two where the rows of B fill the registers
// (3D order 4, 200 to 256 of them, where 20.3 KB of shared memory allow no more), and at least
// four otherwise.  With one workgroup per face that is four in 2D order 4 (108 registers and
// 10.0 KB, which allow no more), four to five in 3D order 2 (92 to 116, 8.0 KB) and six in 2D
// order 2 (76, 6.0 KB), without spills.  What spills: persistent instances (WALK), 12 to 90
// registers, and Neumann instances in fourth order (3D: 20, 220 and 329 at 64, 96 and 128
// rows), which still take half the time that they took with every row in shared memory (3D,
// 40^3, whole build 6.5 and 3.6 ms).
template <int D, int Q>
constexpr int kWaves = Dims<D, Q>::M > 16 ? 2 : 4;

template <int D, int Q, int NPAD, bool WALK, bool NEU = false>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<D, Q>))) void k_stencil(
    StencilArgs A, double* __restrict__ val, int8_t* __restrict__ status, int32_t* flagged) {
  __shared__ __align__(16) FaceSmem<D, Q> sm;
  const int lane = threadIdx.x;
  FaceWalk walk(A);
  if constexpr (!WALK) {
    const long long t = walk.next();
    if (t >= 0 && t < A.nbin) stencil_face<D, Q, NPAD, NEU>(A, t, sm, lane, val, status, flagged);
  } else {
    for (long long t = walk.next(); t >= 0 && t < A.nbin; t = walk.next()) {
      stencil_face<D, Q, NPAD, NEU>(A, t, sm, lane, val, status, flagged);
      __syncthreads();   // the next face reuses the shared memory
    }
  }
}

// ---------------------------------------------------------------------------------------
// Adjoint of the stencil of one face (the derivative of the solution of Sec. 2.2.1).
// With s~ = W z, z = B y, y = G^-1 F~, G = B^T B and a given s~bar:
//   zbar = W s~bar,  Wbar_i = s~bar_i z_i (through s~ = W z),
//   w = G^-1 B^T zbar (a least-squares solve, refined like the forward), r = zbar - B w,
//   Bbar = r y^T - z w^T,  Fbar = w,  Abar = W Bbar,  Wbar_i += Bbar_i . A~_i.
// Bbar_i . B_i = r_i z_i - z_i (B w)_i needs no pass over the row.  The rows' moments
// get S(delta_i)^T Abar_i / mu0 - e_0 (Abar_i . A~_i) / mu0; that sum over the faces a
// row appears in is formed per Phi entry by k_moment_reduce from what this kernel keeps:
// y and w of the face, x0, and (W r, W z) per row.  For an EB face x0 is the centroid of
// the cut volume, so every row's delta and weight and the re-centred normal moments also
// depend on that volume's moments 0..D; their gradient goes to owner_grad.

template <int D, int Q, int NPAD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kWaves<D, Q>))) void k_stencil_backward(
    StencilArgs A, BackwardArgs B) {
  using DM = Dims<D, Q>;
  constexpr int M = DM::M, MS = DM::MS, Mf = DM::Mf, M1 = DM::M1, NR = (NPAD + 63) / 64;
  __shared__ __align__(16) FaceSmem<D, Q> sm;
  const long long t = blockIdx.x;
  if (t >= A.nbin) return;
  const int lane = threadIdx.x;
  FaceInfo fi = face_info(A, t);
  const GeomPtrs& gp = A.geoms[fi.gi];
  face_x0<D, Q>(A.g, gp, fi);
  const int32_t* vol_cell = A.vol_cell_ws + (long long)fi.gi * A.g.ncell;
  const int32_t* box_lf = A.box_lf_ws + (long long)fi.gi * A.g.nboxslot;
  const bool act = lane < M;
  const int N = fi.N;
  double* yw = B.face_yw + (long long)fi.F * 2 * M;
  double* og = B.owner_grad + (long long)fi.F * 4;
  if (lane < 4) B.face_x0[(long long)fi.F * 4 + lane] = (lane < 3) ? fi.x0h[lane] : 0.0;
  // a face whose stencil gets no cotangent contributes nothing: skip its solve
  bool any = false;
  for (int r = lane; r < N; r += 64) any = any || (B.val_bar[fi.rp + r] != 0.0);
  if (!__any(any)) {
    for (int r = lane; r < N; r += 64) {
      B.nz_rz[2 * (fi.rp + r)] = 0.0;
      B.nz_rz[2 * (fi.rp + r) + 1] = 0.0;
      if (B.weight_bar) B.weight_bar[fi.rp + r] = 0.0;
    }
    if (act) { yw[lane] = 0.0; yw[M + lane] = 0.0; }
    if (lane < 4) og[lane] = 0.0;
    return;
  }
  WaveMatrix<D, Q> G;
  RowSwap<D, Q, NPAD - 64> sw;
  double wreg[NR], zreg[NR], yl;
  const int st = face_forward<D, Q, NPAD, false>(A.g, gp, fi, vol_cell, box_lf, A.col, sm, lane, G, sw, wreg, zreg, yl,
                                                 A.wpow);
  // a flagged face has s = 0 whatever its inputs: no gradient (the forward status decides
  // for the faces the forward build solved by Householder QR)
  if (st == CUTCELL_STATUS_NONFINITE || B.fwd_status[fi.F] != CUTCELL_STATUS_OK) {
    for (int r = lane; r < N; r += 64) {
      B.nz_rz[2 * (fi.rp + r)] = 0.0;
      B.nz_rz[2 * (fi.rp + r) + 1] = 0.0;
      if (B.weight_bar) B.weight_bar[fi.rp + r] = 0.0;
    }
    if (act) { yw[lane] = 0.0; yw[M + lane] = 0.0; }
    if (lane < 4) og[lane] = 0.0;
    return;
  }
  // s~bar = h^(D-2) val_bar;  zbar = W s~bar
  double sb[NR], zbar[NR], bw[NR];
  static_for<0, NR>([&](auto R) {
    const int r = lane + 64 * R;
    sb[R] = (r < N) ? A.hscale * B.val_bar[fi.rp + r] : 0.0;
    zbar[R] = wreg[R] * sb[R];
    bw[R] = 0.0;
  });
  // w = G^-1 B^T zbar, refined:  w += G^-1 B^T (zbar - B w); lane p holds w_p, and dy ends
  // as w.  Rows 0..63 are in their slots (state 0), the ones past 64 change places with them.
  const int n0 = (NR > 1 && N > 64) ? 64 : ((N + 7) & ~7);
  const int n1 = (NR > 1 && N > 64) ? ((N - 64 + 7) & ~7) : 0;
  const int cl = act ? lane : 0;
  double wl = 0.0;
  for (int it = 0; it <= kRefineBackward; ++it) {
    lds_order();
    static_for<0, NR>([&](auto R) { sm.zs[lane + 64 * R] = bw[R] - zbar[R]; });
    lds_order();
    double p0 = 0.0, p1 = 0.0;
    column_sum<D, Q>(sm, cl, n0, 0, p0, p1);
    if constexpr (NR > 1) {
      sw.exchange(sm, lane);
      column_sum<D, Q>(sm, cl, n1, 64, p0, p1);
    }
    apply_inverse<D, Q>(sm, lane, G, act ? (p0 + p1) * G.sd : 0.0);
    if (act) wl += sm.dy[lane];
    lds_order();
    if (act) sm.dy[lane] = wl;
    lds_order();
    static_for_down<0, NR>([&](auto R) {
      const double s = row_product<D, Q>(sm, lane);
      bw[R] = (R == 0 || lane < n1) ? s : 0.0;
      if constexpr (R > 0) sw.exchange(sm, lane);
    });
  }
  if (act) {
    yw[lane] = yl;
    yw[M + lane] = wl;
    sm.ys[lane] = yl;
  }
  lds_order();
  // per row: r = zbar - B w;  Wbar;  (W r, W z) for the moment reduction;  EB x0 terms
  double gx[3] = {0, 0, 0};
  static_for<0, NR>([&](auto R) {
    const int r = lane + 64 * R;
    if (r < N) {
      const double Wt = wreg[R], zz = zreg[R];
      const double rr = zbar[R] - bw[R];
      const double bdot = zz * (rr - bw[R]);               // Bbar_i . B_i
      const double wtot = sb[R] * zz + bdot / Wt;          // dl/dW_i
      if (B.weight_bar) B.weight_bar[fi.rp + r] = wtot;
      B.nz_rz[2 * (fi.rp + r)] = Wt * rr;
      B.nz_rz[2 * (fi.rp + r) + 1] = Wt * zz;
      if (fi.kind == 1) {
        // delta_i = x_i/h - x0h: d B_ip / d delta_d = p_d B_i,p-e_d (weight fixed), and
        // dW/d delta_d = -p W delta_d / |delta|^2 outside half a cell (W = (2|delta|)^-p)
        const RowSource rs = row_source<D, Q>(A.g, gp, (int64_t)A.col[fi.rp + r] - fi.phi0, fi.n_vol, fi.n_eb,
                                              vol_cell, box_lf);
        double dl[3] = {0, 0, 0}, d2 = 0.0;
        for (int ax = 0; ax < D; ++ax) {
          dl[ax] = rs.ctr[ax] - fi.x0h[ax];
          d2 += dl[ax] * dl[ax];
        }
        double gd[3] = {0, 0, 0};
        static_for<0, M>([&](auto P) {
          constexpr int p = P;
          const double bb = rr * sm.ys[p] - zz * sm.dy[p];   // Bbar_ip
          static_for<0, D>([&](auto AX) {
            constexpr int ax = AX;
            constexpr int pd = kMono<D, Q>.e[p][ax];
            if constexpr (pd > 0) {
              constexpr int q = mono_index<D>(kMono<D, Q>.e[p][0] - (ax == 0), kMono<D, Q>.e[p][1] - (ax == 1),
                                              kMono<D, Q>.e[p][2] - (ax == 2));
              gd[ax] = fma(bb * pd, sm.Bs[lane * MS + q], gd[ax]);
            }
          });
        });
        if (sqrt(d2) >= 0.5)
          for (int ax = 0; ax < D; ++ax) gd[ax] += wtot * (-A.wpow * Wt * dl[ax] / d2);
        for (int ax = 0; ax < D; ++ax) gx[ax] -= gd[ax];   // d delta / d x0h = -1
      }
    }
    if constexpr (R + 1 < NR) sw.exchange(sm, lane);
  });
  // flux-vector gradient Fbar = w
  if (fi.kind == 0) {
    if (lane < 4) og[lane] = 0.0;
    if (act) {
      constexpr auto& T = kMono<D, Q>;
      const int dn = fi.dn;
      const int e0 = T.e[lane][0], e1 = T.e[lane][1], e2 = T.e[lane][2];
      const int pd = (dn == 0) ? e0 : (dn == 1 ? e1 : e2);
      if (pd == 1) {
        int s;
        if (D == 2) s = mono_index<1>(dn == 0 ? e1 : e0, 0, 0);
        else if (dn == 0) s = mono_index<2>(e1, e2, 0);
        else if (dn == 1) s = mono_index<2>(e0, e2, 0);
        else s = mono_index<2>(e0, e1, 0);
        B.grads[fi.gi].face_mom[dn][(fi.ref - A.g.foff[dn]) * Mf + s] = wl;
      }
    }
    return;
  }
  // EB face: F~_p = sum_d p_d nu'_{d, p - e_d} with nu' the normal moments re-centred by
  // delta0 = (c - x0)/h:  nu'bar_{d,q} = (q_d + 1) w_{q + e_d},  nubar = S(delta0)^T nu'bar,
  // and d nu'_{d,q} / d delta0_k = q_k nu'_{d, q - e_k}
  double gxh[3] = {0, 0, 0};
  for (int ax = 0; ax < D; ++ax) gxh[ax] = wave_sum_f64(gx[ax]);
  lds_order();
  {
    dd x0dd[3];
    face_x0_dd<D, Q>(A.g, gp, fi, x0dd);
    eb_normal_moments<D, Q>(A.g, gp, fi, sm, lane, x0dd);
  }
  double g0[3] = {0, 0, 0};
  if (lane < D) {
    double nb[M1];
    static_for<0, M1>([&](auto I) {
      constexpr int i = I;
      constexpr int q0 = kMono<D, Q - 1>.e[i][0], q1 = kMono<D, Q - 1>.e[i][1], q2 = kMono<D, Q - 1>.e[i][2];
      const int qd = (lane == 0) ? q0 : (lane == 1 ? q1 : q2);
      const int up = mono_index<D>(q0 + (lane == 0), q1 + (lane == 1), q2 + (lane == 2));
      nb[i] = (qd + 1) * sm.dy[up];
    });
    static_for<0, M1>([&](auto I) {
      constexpr int i = I;
      static_for<0, D>([&](auto K) {
        constexpr int k = K;
        constexpr int qk = kMono<D, Q - 1>.e[i][k];
        if constexpr (qk > 0) {
          constexpr int src = mono_index<D>(kMono<D, Q - 1>.e[i][0] - (k == 0), kMono<D, Q - 1>.e[i][1] - (k == 1),
                                            kMono<D, Q - 1>.e[i][2] - (k == 2));
          g0[k] = fma(nb[i] * qk, sm.nus[lane][src], g0[k]);
        }
      });
    });
    double d0[3] = {-fi.off[0], -fi.off[1], -fi.off[2]};
    recentre_T<D, Q - 1>(nb, d0);
    double* dst = B.grads[fi.gi].eb_nmom + ((long long)fi.ref * D + lane) * M1;
    static_for<0, M1>([&](auto I) { dst[I] = nb[I]; });
  }
  // dl/dx0h = sum over rows - dl/d delta0 (component c in lane c);  x0h_d = centre_d + m^{e_d} / m^0
  for (int k = 0; k < D; ++k)
    for (int q = 0; q < D; ++q) gxh[k] -= readlane_f64(g0[k], q);
  if (lane == 0) {
    const double* vm = gp.vol_mom + (long long)fi.owner_cell * M;
    const double m0 = vm[0];
    double gm = 0.0;
    for (int ax = 0; ax < D; ++ax) {
      og[1 + ax] = gxh[ax] / m0;
      gm -= gxh[ax] * vm[1 + ax] / (m0 * m0);
    }
    og[0] = gm;
    for (int ax = D; ax < 3; ++ax) og[1 + ax] = 0.0;
  }
}

// ---------------------------------------------------------------------------------------
// Launches

inline StencilArgs stencil_args(const Work& w, double hscale, const int32_t* perm, long long nbin,
                               const int64_t* row_ptr, const int32_t* col) {
  StencilArgs A;
  A.xcd = 1;
  A.per_xcd = 1;
  A.g = w.dims;
  A.G = w.G;
  A.hscale = hscale;
  A.perm = perm;
  A.nbin = nbin;
  A.fcode = w.fcode;
  A.fref = w.fref;
  A.geoms = w.geoms;
  A.counts = w.counts;
  A.offs = w.offs;
  A.vol_cell_ws = w.vol_cell;
  A.box_lf_ws = w.box_lf;
  A.row_ptr = row_ptr;
  A.col = col;
  A.h = 0.0;
  A.wpow = 5.0;
  A.qr_list = w.qr_list;
  A.qr_count = w.qr_count;
  A.route = 1;
  return A;
}

// Launch shape of one bin: xcd = 1 or the number of XCDs whose chunks the bin is split
// into; per_xcd = 0 for one workgroup per face, else the persistent workgroups per chunk.
struct BinSchedule {
  int xcd = 1;
  int per_xcd = 0;
  bool route = true;   // faces the Gram path cannot resolve go to the QR path
  bool same(const BinSchedule& o) const { return xcd == o.xcd && per_xcd == o.per_xcd && route == o.route; }
};

// Faces [perm, perm + nbin) of bins of at most NPAD rows.
template <int D, int Q, int NPAD>
void launch_rows(const Work& w, double hscale, const int32_t* perm, long long nbin, const int64_t* row_ptr,
                 const int32_t* col, double* val, int8_t* status, hipStream_t st, const BackwardArgs* bw,
                 BinSchedule sc, bool neu, double h, double wpow) {
  if (nbin <= 0) return;
  StencilArgs A = stencil_args(w, hscale, perm, nbin, row_ptr, col);
  A.wpow = wpow;
  if (bw) {
    hipLaunchKernelGGL((k_stencil_backward<D, Q, NPAD>), dim3((unsigned)nbin), dim3(64), 0, st, A, *bw);
    return;
  }
  const int X = sc.xcd > 1 ? sc.xcd : 1;
  const long long chunk = (nbin + X - 1) / X;
  const long long per = sc.per_xcd > 0 ? std::min<long long>(sc.per_xcd, chunk) : chunk;
  A.xcd = X;
  A.per_xcd = (int)per;
  A.route = sc.route ? 1 : 0;
  if (neu) {   // one workgroup per face (no persistent instance of the Neumann kernel)
    A.per_xcd = (int)chunk;
    A.h = h;
    hipLaunchKernelGGL((k_stencil<D, Q, NPAD, false, true>), dim3((unsigned)(X * chunk)), dim3(64), 0, st, A, val,
                       status, w.flagged);
    return;
  }
  if (per < chunk)
    hipLaunchKernelGGL((k_stencil<D, Q, NPAD, true>), dim3((unsigned)(X * per)), dim3(64), 0, st, A, val, status,
                       w.flagged);
  else
    hipLaunchKernelGGL((k_stencil<D, Q, NPAD, false>), dim3((unsigned)(X * per)), dim3(64), 0, st, A, val, status,
                       w.flagged);
}

// Explicit instantiations: each (dimension, order, most rows) lives in one
// stencil_d*q*.hip file, so the library's kernels compile in parallel.
#define CC_ROWS(DD, QQ, NPAD, EXT) \
  EXT template void launch_rows<DD, QQ, NPAD>(const Work&, double, const int32_t*, long long, const int64_t*, \
                                              const int32_t*, double*, int8_t*, hipStream_t, const BackwardArgs*, \
                                              BinSchedule, bool, double, double);
#define CC_ROWS_ALL(DD, QQ) CC_ROWS(DD, QQ, 64, extern) CC_ROWS(DD, QQ, 96, extern) CC_ROWS(DD, QQ, 128, extern)
CC_ROWS_ALL(2, 2) CC_ROWS_ALL(2, 4) CC_ROWS_ALL(3, 2) CC_ROWS_ALL(3, 4)

// Rows of the kernel that takes bin b.
constexpr int bin_width(int b) { return kBinRows * (b + 1) <= 64 ? 64 : (kBinRows * (b + 1) <= 96 ? 96 : 128); }

// The row bins of one (dimension, order), or those of one kernel width: bins that run on the
// same kernel with the same schedule share a launch (their faces follow each other in the
// order), so that a small build pays for two launches and no bin ends with a nearly empty chip.
template <int D, int Q>
int dispatch_row_bins(const Work& w, double hscale, const int32_t* bin_count, const int64_t* row_ptr,
                      const int32_t* col, double* val, int8_t* status, hipStream_t st, const BackwardArgs* bw,
                      const BinSchedule* sched, int only_width, bool neu, double h, double wpow) {
  constexpr int M = binom(Q + D, D);
  long long start = 0;
  for (int b = 0; b < kMaxBins;) {
    long long nb = bin_count[b];
    const bool skip = only_width > 0 && bin_width(b) != only_width;
    if (nb > 0 && kBinRows * (b + 1) < M && !skip)
      return fail(CUTCELL_E_INVALID_ARG, "internal: face with N >= M in a bin narrower than M");
    int e = b + 1;
    for (; e < kMaxBins && bin_width(e) == bin_width(b) && (bw || sched[e].same(sched[b])); ++e) nb += bin_count[e];
    if (!skip) {
      const auto launch = bin_width(b) == 64 ? launch_rows<D, Q, 64>
                                             : (bin_width(b) == 96 ? launch_rows<D, Q, 96> : launch_rows<D, Q, 128>);
      launch(w, hscale, w.perm + start, nb, row_ptr, col, val, status, st, bw, sched[b], neu, h, wpow);
    }
    start += nb;
    b = e;
  }
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

#define CC_DISPATCH(DD, QQ, EXT) \
  EXT template int dispatch_row_bins<DD, QQ>(const Work&, double, const int32_t*, const int64_t*, const int32_t*, \
                                             double*, int8_t*, hipStream_t, const BackwardArgs*, const BinSchedule*, \
                                             int, bool, double, double);
CC_DISPATCH(2, 2, extern) CC_DISPATCH(2, 4, extern) CC_DISPATCH(3, 2, extern) CC_DISPATCH(3, 4, extern)

}  // namespace cutcell
