// Adjoints of the operator apply and of the stencils (derivatives of Sec. 2.2 and
// Sec. 2.2.1).  Every output is produced by exactly one thread group in a fixed order, so
// repeated calls give identical bits (no floating-point atomics):
//   * the transpose (CSC) of the stencils is a stable radix sort of the CSR positions by
//     column, so each Phi entry lists its nonzeros in ascending CSR position;
//   * the apply adjoint scatters each volume's cotangent onto its at most 2D+1 faces in two
//     passes (a face is the high face of at most one volume and the low face of at most
//     one), then gathers Phi-bar through the transpose;
//   * the moment gradients of the rows are summed per Phi entry through the transpose.
#include <algorithm>
#include <string>

#include <hipcub/hipcub.hpp>

#include "kernels.hpp"
#include "rows.hpp"

namespace cutcell {

static inline unsigned nblocks(long long n, int t) { return (unsigned)((n + t - 1) / t); }

// ---- transpose -------------------------------------------------------------------------
__global__ void k_iota(int32_t* p, long long n) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) p[i] = (int32_t)i;
}

// col_ptr from the sorted columns: entry k starts at the first position whose key is >= k
__global__ void k_col_ptr(long long nnz, long long n_phi, const int32_t* __restrict__ keys,
                          int64_t* __restrict__ col_ptr) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i > nnz) return;
  const long long prev = (i == 0) ? -1 : keys[i - 1];
  const long long cur = (i == nnz) ? n_phi : keys[i];
  for (long long k = prev + 1; k <= cur; ++k) col_ptr[k] = i;
}

// The face of every CSR position, then of each listed one.  The first row and the last one
// reach to the ends of face_of, and no row past them, whatever row_ptr says of nnz.  Bound by
// the gather's lines; 1.4e7 nonzeros: 235 us as a binary search in row_ptr per nonzero, 21 +
// 95 us like this.
__global__ __launch_bounds__(256) void k_row_face(long long n_face, long long nnz, const int64_t* __restrict__ row_ptr,
                                                  int32_t* __restrict__ face_of) {
  constexpr int SW = 16;   // lanes per row
  const long long f = (blockIdx.x * 256LL + threadIdx.x) / SW;
  if (f > 0 && f >= n_face) return;
  const int64_t a = f > 0 ? max((int64_t)0, row_ptr[f]) : 0;
  const int64_t b = f + 1 < n_face ? min((int64_t)nnz, row_ptr[f + 1]) : nnz;
  for (int64_t j = a + threadIdx.x % SW; j < b; j += SW) face_of[j] = (int32_t)f;
}

// Workgroup b runs on XCD b % 8 and takes its positions from the b % 8-th eighth: the lines
// of face_of that neighbouring columns share are then fetched into one L2.
__global__ __launch_bounds__(256) void k_nz_face(long long nnz, const int32_t* __restrict__ face_of,
                                                 const int32_t* __restrict__ nz, int32_t* __restrict__ nz_face) {
  constexpr int U = 4;   // loads of a thread in flight
  const long long per = (long long)(gridDim.x / kXcds);   // workgroups per XCD
  const long long i0 = ((blockIdx.x % kXcds) * per + blockIdx.x / kXcds) * (256LL * U) + threadIdx.x;
  int32_t j[U], f[U];
#pragma unroll
  for (int u = 0; u < U; ++u) j[u] = i0 + 256 * u < nnz ? nz[i0 + 256 * u] : -1;
#pragma unroll
  for (int u = 0; u < U; ++u) f[u] = j[u] >= 0 ? face_of[j[u]] : 0;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (j[u] >= 0) nz_face[i0 + 256 * u] = f[u];
}

static int key_bits(long long n_phi) {
  int b = 1;
  while ((1LL << b) < n_phi) ++b;
  return b;
}

size_t transpose_temp_bytes(long long nnz, long long n_phi) {
  size_t temp = 0;
  if (nnz > 0)
    (void)hipcub::DeviceRadixSort::SortPairs(nullptr, temp, (const int32_t*)nullptr, (int32_t*)nullptr,
                                             (const int32_t*)nullptr, (int32_t*)nullptr, (int)nnz, 0,
                                             key_bits(n_phi), (hipStream_t)0);
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  return al(temp) + 2 * al(sizeof(int32_t) * (size_t)std::max<long long>(nnz, 1));
}

int build_transpose(long long n_face, long long n_phi, long long nnz, const int64_t* row_ptr, const int32_t* col,
                    int64_t* col_ptr, int32_t* nz, int32_t* nz_face, char* ws, size_t ws_bytes, hipStream_t st) {
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  size_t temp = 0;
  if (nnz > 0)
    CC_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, temp, (const int32_t*)nullptr, (int32_t*)nullptr,
                                              (const int32_t*)nullptr, (int32_t*)nullptr, (int)nnz, 0,
                                              key_bits(n_phi), st));
  const size_t need = al(temp) + 2 * al(sizeof(int32_t) * (size_t)std::max<long long>(nnz, 1));
  if (!ws || ws_bytes < need) return fail(CUTCELL_E_WORKSPACE, "transpose workspace too small: need " + std::to_string(need));
  int32_t* keys_out = (int32_t*)(ws + al(temp));
  int32_t* vals_in = (int32_t*)(ws + al(temp) + al(sizeof(int32_t) * (size_t)std::max<long long>(nnz, 1)));
  if (nnz > 0) {
    hipLaunchKernelGGL(k_iota, dim3(nblocks(nnz, 256)), dim3(256), 0, st, vals_in, nnz);
    CC_HIP(hipcub::DeviceRadixSort::SortPairs(ws, temp, col, keys_out, vals_in, nz, (int)nnz, 0, key_bits(n_phi), st));
    int32_t* face_of = vals_in;   // the sort has read it
    hipLaunchKernelGGL(k_row_face, dim3(nblocks(std::max<long long>(n_face, 1) * 16, 256)), dim3(256), 0, st, n_face,
                       nnz, row_ptr, face_of);
    hipLaunchKernelGGL(k_nz_face, dim3(nblocks(nblocks(nnz, 1024), kXcds) * kXcds), dim3(256), 0, st, nnz, face_of, nz, nz_face);
  }
  hipLaunchKernelGGL(k_col_ptr, dim3(nblocks(nnz + 1, 256)), dim3(256), 0, st, nnz, n_phi, keys_out, col_ptr);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

// ---- apply adjoint ------------------------------------------------------------------------
// dl/dflux_f = sum over the volumes v of f of sigma_vf * scale_v * lbar_v.  Pass 0 adds the
// volumes for which f is the high or the EB face (sigma = +1), pass 1 the volumes for which
// f is the low face (sigma = -1).
template <int D, int PASS>
__global__ __launch_bounds__(256) void k_face_cotangent(long long n_vol, const int32_t* __restrict__ vol_face,
                                                        const double* __restrict__ vol_scale,
                                                        const double* __restrict__ lbar, double* __restrict__ fbar) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= n_vol) return;
  constexpr int S = 2 * D + 1;
  const int32_t* vf = vol_face + v * S;
  const double c = vol_scale[v] * lbar[v];
  if (PASS == 0) {
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (vf[2 * d + 1] >= 0) fbar[vf[2 * d + 1]] += c;
    if (vf[2 * D] >= 0) fbar[vf[2 * D]] += c;
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d)
      if (vf[2 * d] >= 0) fbar[vf[2 * d]] -= c;
  }
}

// Phi-bar_k = sum over the nonzeros j of column k of val[j] * fbar[face(j)]
//
// SW lanes per Phi entry, U loads of a lane in flight.  Consecutive entries read consecutive
// values of the same face rows, so workgroup b (which MI355X runs on XCD b % 8) takes its
// entries from the b % 8-th eighth of them: the value lines that neighbouring entries share
// are then fetched into one L2 instead of eight.  Bound by the lines of the gathers (a column
// uses 7 of a value line's 16 doubles); 48^3, path radius 3 (2.7e7 nonzeros): 262 us with 32
// lanes, one load in flight and the entries dealt over the XCDs in turn, 250 us with 4 loads,
// 235 us with 16 lanes and 12 loads, 279 us with those and the entries dealt in turn.
template <int SW, int U>
__global__ __launch_bounds__(256) void k_phi_bar(long long n_phi, const int64_t* __restrict__ col_ptr,
                                                 const int32_t* __restrict__ nz, const int32_t* __restrict__ nz_face,
                                                 const double* __restrict__ val, const double* __restrict__ fbar,
                                                 double* __restrict__ phi_bar) {
  const long long per = (long long)(gridDim.x / kXcds);   // workgroups per XCD
  const long long blk = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
  const long long k = (blk * 256 + threadIdx.x) / SW;
  const int sl = threadIdx.x % SW;
  double s = 0.0;
  if (k < n_phi) {
    const int64_t a = col_ptr[k], b = col_ptr[k + 1];
    for (int64_t i = a + sl; i < b; i += SW * U) {
      int32_t j[U], f[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool in = i + SW * u < b;
        j[u] = in ? __builtin_nontemporal_load(nz + i + SW * u) : -1;
        f[u] = in ? __builtin_nontemporal_load(nz_face + i + SW * u) : 0;
      }
      double v[U], c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u] = j[u] >= 0 ? val[j[u]] : 0.0;
        c[u] = j[u] >= 0 ? fbar[f[u]] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) s = j[u] >= 0 ? fma(v[u], c[u], s) : s;
    }
  }
#pragma unroll
  for (int off = SW / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, SW);
  if (k < n_phi && sl == 0) phi_bar[k] = s;
}

// val-bar_j = fbar[f] * Phi[col[j]] over the rows of face f
template <int SW>
__global__ __launch_bounds__(256) void k_val_bar(long long n_face, const int64_t* __restrict__ row_ptr,
                                                 const int32_t* __restrict__ col, const double* __restrict__ fbar,
                                                 const double* __restrict__ phi, double* __restrict__ val_bar) {
  const long long gt = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const long long f = gt / SW;
  const int sl = threadIdx.x % SW;
  if (f >= n_face) return;
  const double c = fbar[f];
  const int64_t a = row_ptr[f], b = row_ptr[f + 1];
  for (int64_t j = a + sl; j < b; j += SW) val_bar[j] = c * phi[col[j]];
}

// scale-bar_v = lbar_v * sum over v's faces of sigma * flux (L_v = scale_v times that sum)
template <int D>
__global__ __launch_bounds__(256) void k_scale_bar(long long n_vol, const int32_t* __restrict__ vol_face,
                                                   const double* __restrict__ flux, const double* __restrict__ lbar,
                                                   double* __restrict__ scale_bar) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= n_vol) return;
  constexpr int S = 2 * D + 1;
  const int32_t* vf = vol_face + v * S;
  double s = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const int32_t lo = vf[2 * d], hi = vf[2 * d + 1];
    if (lo >= 0) s -= flux[lo];
    if (hi >= 0) s += flux[hi];
  }
  const int32_t e = vf[2 * D];
  if (e >= 0) s += flux[e];
  scale_bar[v] = lbar[v] * s;
}

template <int D>
static void apply_adjoint_t(long long n_face, long long n_vol, long long n_phi, const int64_t* row_ptr,
                            const int32_t* col, const double* val, const int32_t* vol_face, const double* vol_scale,
                            const Transpose& tr, const double* phi, const double* flux, const double* lbar,
                            double* phi_bar, double* val_bar, double* scale_bar, double* fbar, hipStream_t st) {
  constexpr int SW = (D == 3) ? 32 : 16;           // lanes of a face row
  constexpr int SC = 16, U = (D == 3) ? 12 : 4;    // lanes of a column and their loads in flight
  if (n_face > 0) hipLaunchKernelGGL(k_fill_f64, dim3(nblocks(n_face, 256)), dim3(256), 0, st, fbar, n_face, 0.0);
  if (n_vol > 0) {
    hipLaunchKernelGGL((k_face_cotangent<D, 0>), dim3(nblocks(n_vol, 256)), dim3(256), 0, st, n_vol, vol_face, vol_scale,
                       lbar, fbar);
    hipLaunchKernelGGL((k_face_cotangent<D, 1>), dim3(nblocks(n_vol, 256)), dim3(256), 0, st, n_vol, vol_face, vol_scale,
                       lbar, fbar);
    if (scale_bar)
      hipLaunchKernelGGL(k_scale_bar<D>, dim3(nblocks(n_vol, 256)), dim3(256), 0, st, n_vol, vol_face, flux, lbar,
                         scale_bar);
  }
  if (n_phi > 0) {
    const unsigned blocks = (nblocks(n_phi * SC, 256) + kXcds - 1) / kXcds * kXcds;
    hipLaunchKernelGGL((k_phi_bar<SC, U>), dim3(blocks), dim3(256), 0, st, n_phi, tr.col_ptr, tr.nz, tr.nz_face, val,
                       fbar, phi_bar);
  }
  if (val_bar && n_face > 0)
    hipLaunchKernelGGL(k_val_bar<SW>, dim3(nblocks(n_face * SW, 256)), dim3(256), 0, st, n_face, row_ptr, col, fbar, phi,
                       val_bar);
}

int apply_adjoint(int D, long long n_face, long long n_vol, long long n_phi, const int64_t* row_ptr,
                  const int32_t* col, const double* val, const int32_t* vol_face, const double* vol_scale,
                  const Transpose& tr, const double* phi, const double* flux, const double* lbar, double* phi_bar,
                  double* val_bar, double* scale_bar, double* fbar, hipStream_t st) {
  if (D == 3)
    apply_adjoint_t<3>(n_face, n_vol, n_phi, row_ptr, col, val, vol_face, vol_scale, tr, phi, flux, lbar, phi_bar,
                       val_bar, scale_bar, fbar, st);
  else
    apply_adjoint_t<2>(n_face, n_vol, n_phi, row_ptr, col, val, vol_face, vol_scale, tr, phi, flux, lbar, phi_bar,
                       val_bar, scale_bar, fbar, st);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

// ---- moment gradients of the rows -----------------------------------------------------------
// For Phi entry k with stored moments m (about its own centre) and each nonzero j of its
// column, in face f with x0:  Abar_j = (W r)_j y_f - (W z)_j w_f,  delta_j = x_k/h - x0/h,
//   g = sum_j S(delta_j)^T Abar_j,   dl/dm = g / m_0 - e_0 (g . m) / m_0^2
// (A~_j = S(delta_j) m / m_0, and the sum of Abar_j . A~_j over j is g . m / m_0).
// Volumes add the gradient through their EB face's centroid (owner_grad) and through
// 1/(kappa h^D) in the apply (scale_bar).
//
// One wave per Phi entry, a lane per nonzero.  The 2M doubles of a face come in slices: the
// wave reads a slice of its 64 faces with neighbouring lanes on neighbouring addresses, the
// next one while it sums this one, and hands each lane its face's part through LDS.  The lane
// sums meet in registers, two halves of the wave folding two moments into one register.
// Consecutive entries read the vectors of the same faces, so a workgroup takes four of them
// and workgroup b, which MI355X runs on XCD b % 8, takes them from the b % 8-th eighth.
// Bound by what comes through the caches (560 bytes per nonzero, 7 TB/s); 40^3, order 4, path
// radius 3 (1.4e7 nonzeros): 1450 us with the entries dealt over the XCDs in turn, each lane
// reading its face's vectors by itself and the lane sums in LDS, 1249 us without the first and
// the last, 1107 us like this.

// a' = the low halves of a and b, b' = their high halves: a' + b' holds a's sum over l, l ^ 32
// in the low half of the wave and b's in the high one; with 16: in the even and odd 16 lanes
__device__ __forceinline__ double fold32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double fold16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

template <int D, int Q>
__global__ __launch_bounds__(256, 2) void k_moment_reduce(ReduceArgs R) {
  constexpr int M = Dims<D, Q>::M, Mf = Dims<D, Q>::Mf;
  constexpr int NR = (M + 3) / 4;   // registers after both folds
  const long long per = (long long)(gridDim.x / kXcds);   // workgroups per XCD
  const long long blk = (blockIdx.x % kXcds) * per + blockIdx.x / kXcds;
  const long long k = 4 * blk + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (k >= R.n_phi) return;
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = R.G;           // offs[lo] <= k < offs[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (R.offs[mid] <= k) lo = mid;
    else hi = mid;
  }
  const int gi = lo;
  const GeomPtrs& gp = R.geoms[gi];
  const int64_t loc = k - R.offs[gi];
  const int64_t n_vol = R.counts[4 * gi + 0], n_eb = R.counts[4 * gi + 1];
  const int32_t* vol_cell = R.vol_cell_ws + (long long)gi * R.g.ncell;
  const RowSource rs =
      row_source<D, Q>(R.g, gp, loc, n_vol, n_eb, vol_cell, R.box_lf_ws + (long long)gi * R.g.nboxslot);
  double g[4 * NR];
  static_for<0, 4 * NR>([&](auto I) { g[I] = 0.0; });
  const int64_t a = R.tr.col_ptr[k], b = R.tr.col_ptr[k + 1];
  constexpr int W = (M % 5 == 0) ? 10 : 12;      // doubles of a slice
  constexpr int U = W / 2, NS = 2 * M / W;       // 16-byte loads of a lane, slices
  static_assert(NS * W == 2 * M && W % 2 == 0, "slices");
  typedef double dv2 __attribute__((ext_vector_type(2)));
  __shared__ dv2 slices[4][64 * U];
  dv2* const sl2 = slices[threadIdx.x >> 6];
  for (int64_t i0 = a; i0 < b; i0 += 64) {
    const int64_t i = i0 + lane < b ? i0 + lane : b - 1;   // past the end: the last one, not summed
    const int64_t j = R.tr.nz[i];
    const int32_t f = R.tr.nz_face[i];
    const double* at[U];    // the lane's part of a slice: piece (lane + 64 u) % U of face (lane + 64 u) / U
    static_for<0, U>([&](auto u) {
      const int t = lane + 64 * u;
      at[u] = R.face_yw + (long long)__shfl(f, t / U) * 2 * M + 2 * (t % U);
    });
    dv2 q[U];
    static_for<0, U>([&](auto u) { q[u] = *(const dv2*)at[u]; });
    const double wr = R.nz_rz[2 * j], wz = R.nz_rz[2 * j + 1];
    double dl[3] = {0, 0, 0};
    for (int ax = 0; ax < D; ++ax) dl[ax] = rs.ctr[ax] - R.face_x0[(long long)f * 4 + ax];
    double ab[M];
    static_for<0, NS>([&](auto S) {
      lds_order();
      static_for<0, U>([&](auto u) { sl2[lane + 64 * u] = q[u]; });
      lds_order();
      if constexpr (S + 1 < NS)
        static_for<0, U>([&](auto u) { q[u] = *(const dv2*)(at[u] + W * (S + 1)); });
      static_for<0, U>([&](auto u) {
        const dv2 v = sl2[lane * U + u];
        constexpr int e = W * S + 2 * u;   // e, e + 1: y up to M, then w
        if constexpr (e < M) ab[e] = wr * v.x;
        else ab[e - M] = fma(-wz, v.x, ab[e - M]);
        if constexpr (e + 1 < M) ab[e + 1] = wr * v.y;
        else ab[e + 1 - M] = fma(-wz, v.y, ab[e + 1 - M]);
      });
    });
    recentre_T<D, Q>(ab, dl);
    if (i0 + lane < b) static_for<0, M>([&](auto I) { g[I] += ab[I]; });
  }
  // lane l keeps moment c = 4 (l % 16) + {0, 2, 1, 3}[l / 16]
  double s[NR];
  static_for<0, NR>([&](auto I) {
    s[I] = sum_in_lane_row(fold16(fold32(g[4 * I], g[4 * I + 1]), fold32(g[4 * I + 2], g[4 * I + 3])));
  });
  double tot = s[0];
  static_for<1, NR>([&](auto I) { tot = (lane & 15) == I ? s[I] : tot; });
  const int row = lane >> 4, c = 4 * (lane & 15) + ((row & 1) << 1 | row >> 1);
  const int sl = c >= M ? -1 : rs.dd < 0 ? c : face_slot<D, Q>(c, rs.dd);   // where the moment is stored
  const double m0 = rs.src[0];
  const double gm = wave_sum_f64(sl >= 0 ? tot * rs.src[sl] : 0.0);
  if (sl < 0) return;
  double out = tot / m0;
  if (c == 0) out -= gm / (m0 * m0);
  const GradPtrs& gr = R.grads[gi];
  if (rs.dd < 0 && loc < n_vol) {
    const long long vg = R.offs[(R.G + 1) + gi] + loc;          // global volume index
    if (c == 0 && R.scale_bar) out -= R.scale_bar[vg] * R.vol_scale[vg] / m0;   // d(1/(kappa h^D))/d kappa
    const int32_t fe = R.vol_face[vg * (2 * D + 1) + 2 * D];
    if (fe >= 0 && c <= D) out += R.owner_grad[(long long)fe * 4 + c];
    gr.vol_mom[(long long)rs.cell * M + c] = out;
  } else if (rs.dd < 0) {
    gr.eb_mom[(loc - n_vol) * M + c] = out;
  } else {
    // box face: only the transverse moments are stored; the face kernel has already
    // written their flux-vector part
    gr.face_mom[rs.dd][rs.loc * Mf + sl] += out;
  }
}

int reduce_moments(const cutcell_opts& o, const ReduceArgs& R, hipStream_t st) {
  if (R.n_phi <= 0) return CUTCELL_OK;
  const dim3 grid(nblocks((R.n_phi + 3) / 4, kXcds) * kXcds), block(256);
  if (o.dim == 2 && o.order == 2) hipLaunchKernelGGL((k_moment_reduce<2, 2>), grid, block, 0, st, R);
  else if (o.dim == 2 && o.order == 4) hipLaunchKernelGGL((k_moment_reduce<2, 4>), grid, block, 0, st, R);
  else if (o.dim == 3 && o.order == 2) hipLaunchKernelGGL((k_moment_reduce<3, 2>), grid, block, 0, st, R);
  else if (o.dim == 3 && o.order == 4) hipLaunchKernelGGL((k_moment_reduce<3, 4>), grid, block, 0, st, R);
  else return fail(CUTCELL_E_UNSUPPORTED, "order/dimension");
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

}  // namespace cutcell
