// The Householder QR path (stencil_qr.hpp) with four wavefronts per face, for fourth order
// under Dirichlet EB conditions: the same steps, the work of each spread over the workgroup.
//   * rows: a thread per line of a row's monomials, direction after direction;
//   * factors: four lanes hold a column in registers, only the reflectors pass through shared
//     memory (four waves per SIMD leave 128 registers: 48 to 53 are spilled, in the parts in
//     double-double too; three waves: 447 us where four take 303, 64^3);
//   * refinement: the residuals by all waves, the triangular solves and reflectors by the
//     first.
//
// A build leaves a few hundred faces to this path, fewer than the chip takes at once, so what
// counts is the time of one face, a chain of dependent steps.  Whole kernel with one and four
// waves per face: 64^3 order 4 (778 faces) 467 and 303 us, four 32^3 (504) 394 and 265 us,
// 256^2 order-4 star (one face) 73 and 63 us; every face by QR: 3D, 28^3, whole build 28.4 and
// 19.3 ms, 2D, 200^2 5.0 and 4.4 ms.  In second order, and where Neumann rows (formed by a
// thread each) want the registers of a whole SIMD, one wave is as good or better: every face
// by QR, whole build, 2D order 2, 200^2 1.63 and 1.71 ms, Neumann 3D order 4, 24^3 18.4 and
// 19.0 ms.
#pragma once

#include "stencil_qr.hpp"

namespace cutcell {

constexpr int kWideThreads = 256;

template <int D, int Q>
struct WideSmem {
  static constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS, M1 = Dims<D, Q>::M1;
  double Bq[kMaxRows * MS];   // Householder factors: R on and above the diagonal, v below
  double tau[M];
  double rdiag[M];            // 1 / R_kk
  double colsc[M];            // column scales (powers of two)
  double fvh[M], fvl[M];      // F~
  double ys[M];               // y
  double zs[kMaxRows];        // z
  union {
    struct {
      double nuh[D][M1];      // EB normal moments about x0, high and low parts
      double nul[D][M1];
    };
    struct {
      double r1[kMaxRows], r1c[kMaxRows];   // the residuals (r1c: a part's correction)
    };
    double v[2][kMaxRows];    // reflectors
  };
  double r2[M];
  double sigma2;
  int bad, zero_col, done;
};

// Lanes of a column where the workgroup works on m columns: a power of two, within a wave.
constexpr int lanes_per_column(int threads, int m) {
  int G = threads / 64;
  while (G < 64 && 2 * G * m <= threads) G *= 2;
  return G;
}
__device__ __forceinline__ double group_sum_f64(double v, int G) {
  for (int o = G / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// t <- H_{M-1} ... H_0 t (Q^T t) or H_0 ... H_{M-1} t (Q t) by one wave, t in the row layout
// (lane r holds rows r, r + 64); the next reflector is read while the wave sums for this one
template <int D, int Q, bool TRANS>
__device__ __forceinline__ void reflectors(const WideSmem<D, Q>& sm, int N, int lane, double* t) {
  constexpr int M = Dims<D, Q>::M, MS = Dims<D, Q>::MS;
  auto entry = [&](int k, int r) {
    const double v = sm.Bq[r * MS + k];
    return r < k || r >= N ? 0.0 : (r == k ? 1.0 : v);
  };
  auto index = [](int i) { return TRANS ? i : M - 1 - i; };
  double v0 = entry(index(0), lane), v1 = entry(index(0), lane + 64), tau = sm.tau[index(0)];
#pragma unroll 1
  for (int i = 0; i < M; ++i) {
    const int kn = index(i + 1 < M ? i + 1 : i);
    const double n0 = entry(kn, lane), n1 = entry(kn, lane + 64), ntau = sm.tau[kn];
    const double td = tau * wave_sum_f64(fma(v1, t[1], v0 * t[0]));
    t[0] = fma(-td, v0, t[0]);
    t[1] = fma(-td, v1, t[1]);
    v0 = n0;
    v1 = n1;
    tau = ntau;
  }
}

template <int D, int Q>
__device__ void wide_face(const StencilArgs& A, int32_t F, WideSmem<D, Q>& sm, double* __restrict__ Bh,
                        double* __restrict__ Bl, int tid, double* __restrict__ val, int8_t* __restrict__ status,
                        int32_t* flagged) {
  using DM = Dims<D, Q>;
  constexpr int M = DM::M, MS = DM::MS, M1 = DM::M1, LN = MonoLines<D, Q>::L;
  constexpr int T = kWideThreads;
  const int lane = tid & 63;
  const bool first = tid < 64;   // the first wave
  FaceInfo fi = face_info_of(A, F);
  const GeomPtrs& gp = A.geoms[fi.gi];
  face_x0<D, Q>(A.g, gp, fi);
  const int N = fi.N;
  const int32_t* vol_cell = A.vol_cell_ws + (long long)fi.gi * A.g.ncell;
  const int32_t* box_lf = A.box_lf_ws + (long long)fi.gi * A.g.nboxslot;
  if (tid == 0) sm.bad = sm.zero_col = 0;

  // ---- rows and flux vector in double-double --------------------------------------------
  // Thread r knows row r; what the threads that form it need is left in its row of Bh.  The
  // high parts are formed in Bq, the low parts in Bl.
  static_assert(sizeof(SmallRow) <= MS * sizeof(double), "the row's facts must fit in its row of Bh");
  bool finite = true;
  double wreg = 0.0;
  dd x0[3];
  face_x0_dd<D, Q>(A.g, gp, fi, x0);
  if (tid < N) {
    const RowSource rs = row_source<D, Q>(A.g, gp, (int64_t)A.col[fi.rp + tid] - fi.phi0, fi.n_vol, fi.n_eb, vol_cell,
                                          box_lf);
    SmallRow me{};
    double d2 = 0.0;
    for (int ax = 0; ax < D; ++ax) {
      me.delta[ax] = dd_sub(dd_from(rs.ctr[ax]), x0[ax]);
      d2 += me.delta[ax].hi * me.delta[ax].hi;
    }
    wreg = row_weight(d2, A.wpow);
    me.scale = dd_div(dd_from(wreg), dd_from(rs.src[0]));
    finite = dd_isfinite(me.scale);
    me.src = rs.src;
    me.dd_dir = rs.dd;
    *(SmallRow*)(Bh + tid * MS) = me;
  }
  __syncthreads();
#pragma unroll 1
  for (int dir = 0; dir < D; ++dir) {
#pragma unroll 1
    for (int it = tid; it < N * LN; it += T) {
      const int r = it / LN;
      const SmallRow& row = *(const SmallRow*)(Bh + r * MS);
      finite = line_shift<D, Q>(dir, it % LN, row.delta[dir], row.scale, row.src, row.dd_dir, sm.Bq + r * MS,
                                Bl + r * MS) && finite;
    }
    __syncthreads();
  }
  if (first) {
    dd fv = dd_from(0.0);
    if (fi.kind == 0) {
      const double* fm = gp.face_mom[fi.dn] + (fi.ref - A.g.foff[fi.dn]) * DM::Mf;
      if (lane < M) {
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
          fv = dd_from(fm[s]);
        }
      }
    } else {
      // the normal moments about x0, a lane per line of each
      constexpr int LN1 = MonoLines<D, Q - 1>::L;
      const int ax = lane / LN1;
      const bool on = ax < D;
      const int32_t c = fi.owner_cell;
      int cown[3];
      cell_coords(A.g, c, cown);
      dd dl[3];
      static_for<0, D>([&](auto d) { dl[d] = dd_sub(dd_from(cown[d] + 0.5), x0[d]); });   // (c - x0)/h
      const double* src = gp.eb_nmom + ((long long)fi.ref * D + (on ? ax : 0)) * M1;
#pragma unroll 1
      for (int dir = 0; dir < D; ++dir) {
        dd delta = dl[0];
        static_for<1, D>([&](auto d) {
          delta.hi = pick(dir == d, dl[d].hi, delta.hi);
          delta.lo = pick(dir == d, dl[d].lo, delta.lo);
        });
        if (on)
          (void)line_shift<D, Q - 1>(dir, lane % LN1, delta, dd_from(1.0), src, -1, sm.nuh[ax], sm.nul[ax]);
        lds_order();
      }
    }
    if (fi.kind != 0) {
      if (lane < M) {
        constexpr auto& T = kMono<D, Q>;
        for (int ax = 0; ax < D; ++ax) {
          int e[3] = {T.e[lane][0], T.e[lane][1], T.e[lane][2]};
          const int p = e[ax];
          if (p > 0) {
            e[ax] -= 1;
            const int j = mono_index<D>(e[0], e[1], e[2]);
            fv = dd_add(fv, dd_mul_d(dd{sm.nuh[ax][j], sm.nul[ax][j]}, (double)p));
          }
        }
      }
    }
    finite = finite && dd_isfinite(fv);
    if (lane < M) {
      sm.fvh[lane] = fv.hi;
      sm.fvl[lane] = fv.lo;
    }
  }
  if (!finite) sm.bad = 1;
  __syncthreads();

  // ---- column scales: powers of two bringing every column to 2-norm in [1, 2) -------------
  constexpr int GM = lanes_per_column(T, M);
  const int jM = tid / GM, gM = tid % GM;
  {
    double c2 = 0.0;
    if (jM < M)
      for (int r = gM; r < N; r += GM) c2 = fma(sm.Bq[r * MS + jM], sm.Bq[r * MS + jM], c2);
    c2 = group_sum_f64(c2, GM);
    if (jM < M && gM == 0) {
      if (!(c2 > 0.0)) sm.zero_col = 1;
      const double s = (c2 > 0.0 && isfinite(c2)) ? ldexp(1.0, -ilogb(sqrt(c2))) : 1.0;
      sm.colsc[jM] = s;
      sm.fvh[jM] *= s;
      sm.fvl[jM] *= s;
    }
  }
  __syncthreads();
  for (int i = tid; i < N * MS; i += T) {
    const int c = i % MS;
    if (c >= M) continue;
    const double s = sm.colsc[c], h = sm.Bq[i] * s;
    Bh[i] = h;
    Bl[i] *= s;
    sm.Bq[i] = h;
  }
  __syncthreads();

  int st = CUTCELL_STATUS_OK;
  if (sm.bad) st = CUTCELL_STATUS_NONFINITE;
  else if (sm.zero_col) st = CUTCELL_STATUS_RANK_DEFICIENT;

  // ---- Householder QR of the FP64 part ----------------------------------------------------
  // Four lanes hold a column in registers, rows 4 i + g; the lanes of column k make the
  // reflector v (zero above row k) and hand it on through shared memory.
  double rmax = 0.0, rmin = 1e300;
  if (st == CUTCELL_STATUS_OK) {
    constexpr int RL = kMaxRows / 4, CH = 8;    // rows of a lane, in chunks of 32 rows of the face
    static_assert(4 * M <= T, "four lanes to a column");
    const int j = tid >> 2, g = tid & 3;
    double c[RL];
    static_for<0, RL>([&](auto I) { c[I] = (j < M && 4 * I + g < N) ? sm.Bq[(4 * I + g) * MS + (j < M ? j : 0)] : 0.0; });
    auto chunks = [&](auto&& fn) {
      static_for<0, RL / CH>([&](auto C) {
        if (4 * CH * C < N) static_for<CH * C, CH * (C + 1)>(fn);
      });
    };
    auto quad_sum = [](double v) {
      v += dpp_f64<0xB1>(v);    // quad_perm [1,0,3,2]
      return v + dpp_f64<0x4E>(v);    // quad_perm [2,3,0,1]
    };
#pragma unroll 1
    for (int k = 0; k < M; ++k) {
      double* v = sm.v[k & 1];
      if (j == k) {
        double s[2] = {0.0, 0.0}, al = 0.0;
        chunks([&](auto I) {
          const double x = 4 * I + g > k ? c[I] : 0.0;
          s[I % 2] = fma(x, x, s[I % 2]);
          al = 4 * I + g == k ? c[I] : al;
        });
        const double sigma2 = quad_sum(s[0] + s[1]), alpha = quad_sum(al);   // x^T x below row k
        double beta = alpha, tau = 0.0, inv = 0.0;
        if (sigma2 != 0.0) {
          beta = -copysign(sqrt(fma(alpha, alpha, sigma2)), alpha);
          tau = (beta - alpha) * recip_f64(beta);
          inv = recip_f64(alpha - beta);
        }
        chunks([&](auto I) {
          const int r = 4 * I + g;
          const double x = c[I] * inv;
          v[r] = r < k ? 0.0 : (r == k ? 1.0 : x);
          c[I] = r < k ? c[I] : (r == k ? beta : x);
        });
        if (g == 0) {
          sm.tau[k] = tau;
          sm.rdiag[k] = beta;
        }
      }
      __syncthreads();   // (the buffer of step k is written again at k + 2, after all read it)
      if (j > k && j < M) {
        double p[4] = {0.0, 0.0, 0.0, 0.0};
        chunks([&](auto I) { p[I % 4] = fma(v[4 * I + g], c[I], p[I % 4]); });
        const double ts = sm.tau[k] * quad_sum((p[0] + p[1]) + (p[2] + p[3]));
        asm volatile("" ::: "memory");   // read v again: kept, it would take the registers of a third wave per SIMD
        chunks([&](auto I) { c[I] = fma(-ts, v[4 * I + g], c[I]); });
      }
    }
    if (j < M) chunks([&](auto I) {
      if (4 * I + g < N) sm.Bq[(4 * I + g) * MS + j] = c[I];
    });
    for (int k = 0; k < M; ++k) {
      const double beta = fabs(sm.rdiag[k]);
      rmax = fmax(rmax, beta);
      rmin = fmin(rmin, beta);
    }
    if (!(rmin > kRankTol * rmax)) st = CUTCELL_STATUS_RANK_DEFICIENT;
    __syncthreads();
    if (tid < M) sm.rdiag[tid] = 1.0 / sm.rdiag[tid];
  }

  // ---- minimum-norm solution by refinement of the augmented system -------------------------
  for (int r = tid; r < kMaxRows; r += T) sm.zs[r] = 0.0;
  if (tid < M) sm.ys[tid] = 0.0;
  __syncthreads();
  if (st == CUTCELL_STATUS_OK) {
#pragma unroll 1
    for (int it = 0; it < kQrRefine; ++it) {
      // r1 = B y - z (rows) and r2 = F~ - B^T z (columns), with B = Bh + Bl: the Bh terms in
      // compensated arithmetic (Dot2), the Bl terms (below 2^-53 of them) plainly.  A thread
      // takes the even or the odd columns of a row, and the rows of a column that its group
      // leaves it.
      {
        static_assert(T == 2 * kMaxRows, "a row has two threads");
        const int r = tid % kMaxRows, odd = tid / kMaxRows;
        Dot2 d{odd ? 0.0 : -sm.zs[r], 0.0};
        double lo = 0.0;
        if (r < N) {
#pragma unroll 4
          for (int p = odd; p < M; p += 2) {
            const double yp = sm.ys[p];
            dot2_add(d, Bh[r * MS + p], yp);
            lo = fma(Bl[r * MS + p], yp, lo);
          }
        }
        d.c += lo;
        Dot2 e{0.0, 0.0};
        double elo = 0.0;
        if (jM < M) {
#pragma unroll 4
          for (int i = gM; i < N; i += GM) {
            dot2_add(e, -Bh[i * MS + jM], sm.zs[i]);
            elo = fma(-Bl[i * MS + jM], sm.zs[i], elo);
          }
        }
        e.c += elo;
        for (int o = GM / 2; o > 0; o >>= 1) {   // (every lane ends with the group's sum)
          const dd t = two_sum(e.s, __shfl_xor(e.s, o, 64));
          e = Dot2{t.hi, e.c + __shfl_xor(e.c, o, 64) + t.lo};
        }
        if (jM < M && gM == 0) sm.r2[jM] = dot2_merge(Dot2{sm.fvh[jM], sm.fvl[jM]}, e);
        if (odd) {
          sm.r1[r] = d.s;
          sm.r1c[r] = d.c;
        }
        __syncthreads();
        if (!odd) {
          const double v = dot2_merge(d, Dot2{sm.r1[r], sm.r1c[r]});
          sm.r1[r] = r < N ? v : 0.0;
        }
        __syncthreads();
      }
      // g = Q^T r1;  a = R^-T r2;  dy = R^-1 (a - g1);  dz = Q [a; g2]
      if (first) {
        double gr[2] = {sm.r1[lane], sm.r1[lane + 64]};
        reflectors<D, Q, true>(sm, N, lane, gr);
        const double a = solve_rt<D, Q>(sm, lane, (lane < M) ? sm.r2[lane] : 0.0);
        const double c = solve_r<D, Q>(sm, lane, (lane < M) ? a - gr[0] : 0.0);
        double tz[2] = {(lane < M) ? a : gr[0], gr[1]};
        reflectors<D, Q, false>(sm, N, lane, tz);
        double dmax = 0.0, zmax = 0.0;
        static_for<0, 2>([&](auto R) {
          const int r = lane + 64 * R;
          if (r < N) {
            const double z = sm.zs[r] + tz[R];
            sm.zs[r] = z;
            dmax = fmax(dmax, fabs(tz[R]));
            zmax = fmax(zmax, fabs(z));
          }
        });
        if (lane < M) sm.ys[lane] += c;
        dmax = wave_max_f64(dmax);
        zmax = wave_max_f64(zmax);
        if (lane == 0) sm.done = !(dmax > 0x1p-52 * zmax);
      }
      __syncthreads();
      if (sm.done) break;
    }
  }

  if (tid < N) val[fi.rp + tid] = (st == CUTCELL_STATUS_OK) ? A.hscale * wreg * sm.zs[tid] : 0.0;
  if (tid == 0) {
    status[fi.F] = (int8_t)st;
    if (st != CUTCELL_STATUS_OK) atomicAdd(flagged, 1);
  }
}

// As k_stencil_qr, a workgroup of four waves per face.
template <int D, int Q>
__global__ __launch_bounds__(kWideThreads, 4) void k_stencil_qr_wide(StencilArgs A, const int32_t* __restrict__ list,
                                                                    const int32_t* __restrict__ count_dev,
                                                                    long long count_host, double* __restrict__ bslots,
                                                                    double* __restrict__ val,
                                                                    int8_t* __restrict__ status, int32_t* flagged) {
  constexpr int MS = Dims<D, Q>::MS;
  __shared__ WideSmem<D, Q> sm;
  double* Bh = bslots + (long long)blockIdx.x * 2 * kMaxRows * MS;
  double* Bl = Bh + kMaxRows * MS;
  const long long n = count_dev ? (long long)*count_dev : count_host;
  for (long long t = blockIdx.x; t < n; t += gridDim.x) {
    wide_face<D, Q>(A, list[t], sm, Bh, Bl, threadIdx.x, val, status, flagged);
    __syncthreads();   // the next face reuses the shared memory and the slot
  }
}

}  // namespace cutcell
