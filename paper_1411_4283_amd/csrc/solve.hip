// Discrete Poisson solve with the flux-divergence operator (Sec. 3.2: L(Phi) = f for the
// volume values of Phi, the boundary rows of Phi holding Dirichlet data).
//
// L is affine in the volume values x:  L([x | bc]) = A x + L([0 | bc]).  Restarted GMRES(m)
// solves A x = f - L([0 | bc]) with right Jacobi preconditioning (A D^-1 y = b, x = D^-1 y,
// D = diag A).  Every vector operation is a kernel here; the host keeps only the small
// Hessenberg matrix and its Givens rotations.
#include <algorithm>
#include <cmath>
#include <complex>
#include <string>
#include <vector>

#include "solve.hpp"

namespace cutcell {

constexpr int kBatch = 8;            // Arnoldi steps launched before the host reads their coefficients

static inline unsigned nb(long long n, int t) { return (unsigned)((n + t - 1) / t); }

// Phi index of every volume: geometry g's volumes sit at phi_off[g] + (v - vol_off[g])
__global__ void k_vol_phi(long long n_vol, int G, const int64_t* __restrict__ phi_off,
                          const int64_t* __restrict__ vol_off, int32_t* __restrict__ vol_phi) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= n_vol) return;
  int lo = 0, hi = G;                // vol_off[lo] <= v < vol_off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (vol_off[mid] <= v) lo = mid;
    else hi = mid;
  }
  vol_phi[v] = (int32_t)(phi_off[lo] + (v - vol_off[lo]));
}

__global__ void k_scatter(long long n, const int32_t* __restrict__ idx, const double* __restrict__ x,
                          double* __restrict__ phi) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v < n) phi[idx[v]] = x[v];
}

__global__ void k_copy(long long n, const double* __restrict__ a, double* __restrict__ b) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) b[i] = a[i];
}

// out = alpha * a + beta * b (out may alias a or b)
__global__ void k_axpby(long long n, double alpha, const double* a, double beta, const double* b, double* out) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) out[i] = alpha * a[i] + beta * b[i];
}

// D^-1: A_vv = vol_scale[v] * sum over v's faces of sigma * (the face's coefficient on v)
template <int D>
__global__ void k_jacobi(long long n_vol, const int32_t* __restrict__ vol_face, const double* __restrict__ vol_scale,
                         const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                         const double* __restrict__ val, const int32_t* __restrict__ vol_phi,
                         double* __restrict__ dinv) {
  const long long v = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (v >= n_vol) return;
  constexpr int S = 2 * D + 1;
  const int32_t me = vol_phi[v];
  double s = 0.0;
  for (int k = 0; k < S; ++k) {
    const int32_t f = vol_face[v * S + k];
    if (f < 0) continue;
    const double sigma = (k < 2 * D && (k & 1) == 0) ? -1.0 : 1.0;   // low faces point into v
    int64_t lo = row_ptr[f], hi = row_ptr[f + 1];                       // col ascending: search
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if (col[mid] < me) lo = mid + 1;
      else hi = mid;
    }
    if (lo < row_ptr[f + 1] && col[lo] == me) s += sigma * val[lo];
  }
  const double a = vol_scale[v] * s;
  dinv[v] = (a != 0.0 && isfinite(a)) ? 1.0 / a : 1.0;
}

// ---- Arnoldi step -------------------------------------------------------------------------
// Classical Gram-Schmidt done twice in three launches: the inner products V^T w (k_dots), the
// first update of w with the inner products of the result (k_orth), the second update, the
// norm and the next vector together with the Phi that the next product reads (k_next).  A
// vector is cut into tiles of 256 E elements, a block takes one (or, past kMaxTiles, every
// kMaxTiles-th), and leaves a partial sum per inner product; the launch that needs the sums
// adds the partials itself, block by block alike and in a fixed order, so no launch or copy
// stands between two of them and a solve is deterministic.  Coefficients stay on the device
// (a column of H for each step of a batch); the host reads the columns of a batch at once.  At 30k
// volumes (32^3, 3D order 4) a step is bound by the latency of its dependent launches and of
// the loads in each: eleven launches, a copy and a wait took 88 to 100 us, four launches take
// 42 (37 in the kernels, 15 of them the product).
constexpr int kTileThreads = 256;
constexpr int kMaxTiles = 512;
constexpr int kDotChunk = 8;         // vectors per block of k_dots

// elements per thread: the least that leaves at most 256 tiles (8 at most)
static inline int tile_elems(long long n) {
  int e = 1;
  while (e < 8 && n > 256LL * kTileThreads * e) e *= 2;
  return e;
}
static inline int tile_count(long long n) {
  const long long t = (long long)kTileThreads * tile_elems(n);
  return (int)std::max<long long>(1, std::min<long long>(kMaxTiles, (n + t - 1) / t));
}

// partial[b][i] = block b's share of V_i . w for i < k (V row-major [k][n]; rows of ld partials)
template <int E>
__global__ __launch_bounds__(kTileThreads) void k_dots(long long n, int k, const double* __restrict__ V,
                                                       const double* __restrict__ w, double* __restrict__ partial,
                                                       int ld) {
  __shared__ double red[kTileThreads / 64][kDotChunk];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i0 = blockIdx.y * kDotChunk;
  double acc[kDotChunk];
#pragma unroll
  for (int u = 0; u < kDotChunk; ++u) acc[u] = 0.0;
  for (long long t0 = (long long)blockIdx.x * kTileThreads * E; t0 < n; t0 += (long long)gridDim.x * kTileThreads * E)
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const long long t = t0 + threadIdx.x + e * kTileThreads;
      if (t < n) {
        const double wt = w[t];
#pragma unroll
        for (int u = 0; u < kDotChunk; ++u)
          if (i0 + u < k) acc[u] = fma(V[(long long)(i0 + u) * n + t], wt, acc[u]);
      }
    }
#pragma unroll
  for (int u = 0; u < kDotChunk; ++u) {
    const double s = wave_sum_f64(acc[u]);
    if (lane == 0) red[wv][u] = s;
  }
  __syncthreads();
  if ((int)threadIdx.x < kDotChunk && i0 + (int)threadIdx.x < k) {
    double s = 0.0;
    for (int q = 0; q < kTileThreads / 64; ++q) s += red[q][threadIdx.x];
    partial[(long long)blockIdx.x * ld + i0 + threadIdx.x] = s;
  }
}

// out[i] = sum over the nt blocks of partial[b][i] for i < k, in shared memory: a lane per sum,
// every fourth block in a wave, eight loads in flight, then the waves' sums in order
__device__ __forceinline__ void sum_partials(const double* __restrict__ partial, int ld, int nt, int k, double* out) {
  constexpr int NW = kTileThreads / 64;
  __shared__ double part[NW][64];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int i0 = 0; i0 < k; i0 += 64) {
    const int i = i0 + lane;
    double s = 0.0;
    if (i < k) {
#pragma unroll 8
      for (int b = wv; b < nt; b += NW) s += partial[(long long)b * ld + i];
    }
    part[wv][lane] = s;
    __syncthreads();
    if (wv == 0 && i < k) {
      double t = part[0][lane];
      for (int q = 1; q < NW; ++q) t += part[q][lane];
      out[i] = t;
    }
    __syncthreads();
  }
}

// c1 = V^T w from its partials; w -= V c1; then the partials of V^T w and, as entry k, w . w
template <int E>
__global__ __launch_bounds__(kTileThreads) void k_orth(long long n, int k, const double* __restrict__ V,
                                                       double* __restrict__ w, const double* __restrict__ partial,
                                                       int ld, double* __restrict__ c1,
                                                       double* __restrict__ partial2) {
  extern __shared__ double sh[];
  double* cs = sh;                      // [k]
  double* acc = sh + k;                 // [waves][k + 1]
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  sum_partials(partial, ld, gridDim.x, k, cs);
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < k; i += kTileThreads) c1[i] = cs[i];
  double* mine = acc + wv * (k + 1);
  bool first = true;
  for (long long t0 = (long long)blockIdx.x * kTileThreads * E; t0 < n; t0 += (long long)gridDim.x * kTileThreads * E) {
    double x[E];
    const double* p = V + t0 + threadIdx.x;
    bool in[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      in[e] = t0 + threadIdx.x + e * kTileThreads < n;
      x[e] = in[e] ? w[t0 + threadIdx.x + e * kTileThreads] : 0.0;
    }
#pragma unroll 8
    for (int i = 0; i < k; ++i)
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] = fma(-cs[i], in[e] ? p[(long long)i * n + e * kTileThreads] : 0.0, x[e]);
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (in[e]) w[t0 + threadIdx.x + e * kTileThreads] = x[e];
    for (int i0 = 0; i0 <= k; i0 += 8) {
      double a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u;
        a[u] = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const double v = i < k ? (in[e] ? p[(long long)i * n + e * kTileThreads] : 0.0) : (i == k ? x[e] : 0.0);
          a[u] = fma(v, x[e], a[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        a[u] = wave_sum_f64(a[u]);
        if (lane == 0 && i0 + u <= k) mine[i0 + u] = first ? a[u] : mine[i0 + u] + a[u];
      }
    }
    first = false;
  }
  if (first && lane == 0)
    for (int i = 0; i <= k; ++i) mine[i] = 0.0;
  __syncthreads();
  for (int i = threadIdx.x; i <= k; i += kTileThreads) {
    double s = 0.0;
    for (int q = 0; q < kTileThreads / 64; ++q) s += acc[q * (k + 1) + i];
    partial2[(long long)blockIdx.x * ld + i] = s;
  }
}

// The second pass: d = V^T w and w . w from their partials.  The coefficients are at rounding
// level after the first pass, so the new norm is sqrt(w . w - |d|^2).  v_next = (w - V d) /
// norm (0 if the norm vanishes: a lucky breakdown), phi = D^-1 v_next at the volumes (or
// v_next without dinv), and the column of H: c1 + d, then the norm.
template <int E>
__global__ __launch_bounds__(kTileThreads) void k_next(long long n, int k, const double* __restrict__ V,
                                                       const double* __restrict__ w,
                                                       const double* __restrict__ partial2, int ld,
                                                       const double* __restrict__ c1, double* __restrict__ hcol,
                                                       const double* __restrict__ dinv,
                                                       const int32_t* __restrict__ vphi, double* __restrict__ vnext,
                                                       double* __restrict__ phi) {
  extern __shared__ double sh[];        // [k + 1]
  sum_partials(partial2, ld, gridDim.x, k + 1, sh);
  double c2 = 0.0;
  for (int i = 0; i < k; ++i) c2 = fma(sh[i], sh[i], c2);
  const double q = sh[k] - c2;
  const double norm = q > 0.0 ? sqrt(q) : 0.0;
  const double inv = norm > 0.0 ? 1.0 / norm : 0.0;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < k; i += kTileThreads) hcol[i] = c1[i] + sh[i];
    if (threadIdx.x == 0) hcol[k] = norm;
  }
  for (long long t0 = (long long)blockIdx.x * kTileThreads * E; t0 < n; t0 += (long long)gridDim.x * kTileThreads * E) {
    double x[E];
    const double* p = V + t0 + threadIdx.x;
    bool in[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      in[e] = t0 + threadIdx.x + e * kTileThreads < n;
      x[e] = in[e] ? w[t0 + threadIdx.x + e * kTileThreads] : 0.0;
    }
#pragma unroll 8
    for (int i = 0; i < k; ++i)
#pragma unroll
      for (int e = 0; e < E; ++e) x[e] = fma(-sh[i], in[e] ? p[(long long)i * n + e * kTileThreads] : 0.0, x[e]);
#pragma unroll
    for (int e = 0; e < E; ++e)
      if (in[e]) {
        const long long t = t0 + threadIdx.x + e * kTileThreads;
        const double v = x[e] * inv;
        vnext[t] = v;
        phi[vphi[t]] = dinv ? dinv[t] * v : v;
      }
  }
}

// v *= s; phi = D^-1 v at the volumes (or v without dinv)
__global__ void k_first(long long n, double s, double* __restrict__ v, const double* __restrict__ dinv,
                        const int32_t* __restrict__ vphi, double* __restrict__ phi) {
  const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (t >= n) return;
  const double x = v[t] * s;
  v[t] = x;
  phi[vphi[t]] = dinv ? dinv[t] * x : x;
}

// x += D^-1 sum_{i<k} c[i] V_i
__global__ void k_update(long long n, int k, const double* __restrict__ c, const double* __restrict__ V,
                         const double* __restrict__ dinv, double* __restrict__ x) {
  const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (t >= n) return;
  double s = 0.0;
#pragma unroll 4
  for (int i = 0; i < k; ++i) s = fma(c[i], V[i * n + t], s);
  x[t] = fma(dinv[t], s, x[t]);
}

// The buffers of an Arnoldi process of at most m steps, and its launches.  The callers' needs
// must not exceed what a process with 512 partial sums per inner product and one column of
// coefficients took (a buffer of that size stays enough): hence only `batch` columns of H.
struct Arnoldi {
  long long n;
  int m, batch, tiles, elems;
  double* V;          // [m + 1][n]
  double* w;          // [n]
  double* partial;    // [tiles][m + 1]
  double* partial2;   // [tiles][m + 1]
  double* c1;         // [m]
  double* H;          // [batch][m + 1] columns
  hipStream_t st;

  static size_t bytes(long long n, int m, int batch) {
    auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
    const size_t nv = std::max<long long>(n, 1), nt = tile_count(n);
    return al(sizeof(double) * nv * (m + 1)) + al(sizeof(double) * nv) + al(sizeof(double) * nt * (m + 1)) +
           al(sizeof(double) * nt * (m + 1)) + al(sizeof(double) * m) + al(sizeof(double) * batch * (m + 1));
  }
  template <class Take>
  void layout(long long n_, int m_, int batch_, hipStream_t s, Take&& take) {
    n = n_;
    m = m_;
    batch = batch_;
    st = s;
    tiles = tile_count(n);
    elems = tile_elems(n);
    const size_t nv = std::max<long long>(n, 1);
    V = (double*)take(sizeof(double) * nv * (m + 1));
    w = (double*)take(sizeof(double) * nv);
    partial = (double*)take(sizeof(double) * tiles * (m + 1));
    partial2 = (double*)take(sizeof(double) * tiles * (m + 1));
    c1 = (double*)take(sizeof(double) * m);
    H = (double*)take(sizeof(double) * batch * (m + 1));
  }
  // w holds A v_j: v_{j+1}, phi and the step's coefficients, into column c of H
  template <int E>
  void step_e(int j, int c, const double* dinv, const int32_t* vphi, double* phi) const {
    const int k = j + 1;
    const dim3 T(kTileThreads);
    hipLaunchKernelGGL(k_dots<E>, dim3(tiles, (k + kDotChunk - 1) / kDotChunk), T, 0, st, n, k, V, w, partial, m + 1);
    hipLaunchKernelGGL(k_orth<E>, dim3(tiles), T, sizeof(double) * (k + (kTileThreads / 64) * (k + 1)), st, n, k, V, w,
                       partial, m + 1, c1, partial2);
    hipLaunchKernelGGL(k_next<E>, dim3(tiles), T, sizeof(double) * (k + 1), st, n, k, V, w, partial2, m + 1, c1,
                       H + (size_t)c * (m + 1), dinv, vphi, V + (long long)k * n, phi);
  }
  void step(int j, int c, const double* dinv, const int32_t* vphi, double* phi) const {
    if (elems == 1) step_e<1>(j, c, dinv, vphi, phi);
    else if (elems == 2) step_e<2>(j, c, dinv, vphi, phi);
    else if (elems == 4) step_e<4>(j, c, dinv, vphi, phi);
    else step_e<8>(j, c, dinv, vphi, phi);
  }
  // the first nc columns of H to the host
  int columns(int nc, double* out) const {
    CC_HIP(hipMemcpyAsync(out, H, sizeof(double) * nc * (m + 1), hipMemcpyDeviceToHost, st));
    CC_HIP(hipStreamSynchronize(st));
    return CUTCELL_OK;
  }
  // |y| to the host
  int norm(const double* y, double* out) const {
    if (elems == 1) hipLaunchKernelGGL(k_dots<1>, dim3(tiles), dim3(kTileThreads), 0, st, n, 1, y, y, partial2, 1);
    else if (elems == 2) hipLaunchKernelGGL(k_dots<2>, dim3(tiles), dim3(kTileThreads), 0, st, n, 1, y, y, partial2, 1);
    else if (elems == 4) hipLaunchKernelGGL(k_dots<4>, dim3(tiles), dim3(kTileThreads), 0, st, n, 1, y, y, partial2, 1);
    else hipLaunchKernelGGL(k_dots<8>, dim3(tiles), dim3(kTileThreads), 0, st, n, 1, y, y, partial2, 1);
    double p[kMaxTiles];
    CC_HIP(hipMemcpyAsync(p, partial2, sizeof(double) * tiles, hipMemcpyDeviceToHost, st));
    CC_HIP(hipStreamSynchronize(st));
    double s = 0.0;
    for (int b = 0; b < tiles; ++b) s += p[b];
    *out = std::sqrt(s);
    return CUTCELL_OK;
  }
};

size_t solve_workspace_bytes(long long n_vol, long long n_phi, long long n_face, int m) {
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t nv = std::max<long long>(n_vol, 1);
  return al(sizeof(double) * n_phi) * 2 + al(sizeof(double) * std::max<long long>(n_face, 1)) +
         al(sizeof(double) * nv) * 3 + al(sizeof(int32_t) * nv) + al(sizeof(double) * m) +
         Arnoldi::bytes(n_vol, m, std::min(m, kBatch));
}

int solve_poisson(const SolveOp& op, int G, const int64_t* phi_off, const int64_t* vol_off, const double* phi_bc,
                  const double* f, double* x, int m, int max_iters, double rtol, char* ws, size_t ws_bytes,
                  int* iters_out, double* relres_out) {
  const long long n = op.n_vol;
  if (ws_bytes < solve_workspace_bytes(n, op.n_phi, op.n_face, m))
    return fail(CUTCELL_E_WORKSPACE, "solve workspace too small");
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  size_t off = 0;
  auto take = [&](size_t bytes) { char* p = ws + off; off += al(bytes); return p; };
  const size_t nv = std::max<long long>(n, 1);
  hipStream_t st = op.st;
  double* phi = (double*)take(sizeof(double) * op.n_phi);     // [0 | bc]
  double* phi0 = (double*)take(sizeof(double) * op.n_phi);    // [v | 0]
  double* flux = (double*)take(sizeof(double) * std::max<long long>(op.n_face, 1));
  double* b = (double*)take(sizeof(double) * nv);
  double* dinv = (double*)take(sizeof(double) * nv);
  double* tmp = (double*)take(sizeof(double) * nv);
  int32_t* vphi = (int32_t*)take(sizeof(int32_t) * nv);
  double* coef = (double*)take(sizeof(double) * m);
  Arnoldi A;
  A.layout(n, m, std::min(m, kBatch), st, take);
  const int T = 256;
  const unsigned gv = nb(n, T);

  auto apply = [&](const double* p, double* out) {
    if (op.lap_ptr) return apply_laplacian(op.D, n, op.lap_ptr, op.lap_col, op.lap_val, p, out, st);
    return apply_operator(op.D, op.n_face, n, op.row_ptr, op.col, op.val, op.vol_face, op.vol_scale, p, out, flux,
                          nullptr, st);
  };

  hipLaunchKernelGGL(k_vol_phi, dim3(gv), dim3(T), 0, st, n, G, phi_off, vol_off, vphi);
  hipLaunchKernelGGL(k_copy, dim3(nb(op.n_phi, T)), dim3(T), 0, st, op.n_phi, phi_bc, phi);
  hipLaunchKernelGGL(k_fill_f64, dim3(nb(op.n_phi, T)), dim3(T), 0, st, phi0, op.n_phi, 0.0);
  hipLaunchKernelGGL(k_fill_f64, dim3(gv), dim3(T), 0, st, tmp, n, 0.0);
  // b = f - L([0 | bc])
  hipLaunchKernelGGL(k_scatter, dim3(gv), dim3(T), 0, st, n, vphi, tmp, phi);
  int rc = apply(phi, tmp);
  if (rc) return rc;
  hipLaunchKernelGGL(k_axpby, dim3(gv), dim3(T), 0, st, n, 1.0, f, -1.0, tmp, b);
  if (op.D == 3)
    hipLaunchKernelGGL(k_jacobi<3>, dim3(gv), dim3(T), 0, st, n, op.vol_face, op.vol_scale, op.row_ptr, op.col,
                       op.val, vphi, dinv);
  else
    hipLaunchKernelGGL(k_jacobi<2>, dim3(gv), dim3(T), 0, st, n, op.vol_face, op.vol_scale, op.row_ptr, op.col,
                       op.val, vphi, dinv);
  double bnorm = 0.0;
  rc = A.norm(b, &bnorm);
  if (rc) return rc;
  if (!std::isfinite(bnorm)) return fail(CUTCELL_E_INVALID_ARG, "non-finite right-hand side or boundary data");
  if (bnorm == 0.0) {               // the solution is x = 0
    hipLaunchKernelGGL(k_fill_f64, dim3(gv), dim3(T), 0, st, x, n, 0.0);
    CC_HIP(hipStreamSynchronize(st));
    if (iters_out) *iters_out = 0;
    if (relres_out) *relres_out = 0.0;
    return CUTCELL_OK;
  }
  int it = 0;
  double res = bnorm;
  std::vector<double> H((size_t)m * m), cs(m), sn(m), g(m + 1), y(m), hc((size_t)kBatch * (m + 1));
  for (;;) {
    // r = b - A x; the exit test always uses this true residual
    hipLaunchKernelGGL(k_scatter, dim3(gv), dim3(T), 0, st, n, vphi, x, phi0);
    rc = apply(phi0, tmp);
    if (rc) return rc;
    hipLaunchKernelGGL(k_axpby, dim3(gv), dim3(T), 0, st, n, 1.0, b, -1.0, tmp, A.V);
    double beta = 0.0;
    rc = A.norm(A.V, &beta);
    if (rc) return rc;
    res = beta;
    if (!(beta > rtol * bnorm) || it >= max_iters) break;
    hipLaunchKernelGGL(k_first, dim3(gv), dim3(T), 0, st, n, 1.0 / beta, A.V, dinv, vphi, phi0);
    std::fill(g.begin(), g.end(), 0.0);
    g[0] = beta;
    int j = 0;
    bool done = false;
    int ahead = 2;   // steps launched before their columns are read
    while (!done && j < m && it < max_iters) {
      const int j0 = j, nj = std::min({ahead, m - j, max_iters - it});
      for (int q = 0; q < nj; ++q) {
        rc = apply(phi0, A.w);        // phi0 = [D^-1 v_j | 0]
        if (rc) return rc;
        A.step(j0 + q, q, dinv, vphi, phi0);
      }
      rc = A.columns(nj, hc.data());
      if (rc) return rc;
      const double before = res;
      for (int q = 0; q < nj && !done; ++q, ++j, ++it) {
        // Givens rotations on column j of H
        double* h = hc.data() + (size_t)q * (m + 1);
        const double hn = h[j + 1];
        for (int i = 0; i < j; ++i) {
          const double t = cs[i] * h[i] + sn[i] * h[i + 1];
          h[i + 1] = -sn[i] * h[i] + cs[i] * h[i + 1];
          h[i] = t;
        }
        const double r = std::hypot(h[j], hn);
        cs[j] = r > 0.0 ? h[j] / r : 1.0;
        sn[j] = r > 0.0 ? hn / r : 0.0;
        h[j] = r;
        g[j + 1] = -sn[j] * g[j];
        g[j] = cs[j] * g[j];
        for (int i = 0; i <= j; ++i) H[(size_t)i * m + j] = h[i];
        res = std::fabs(g[j + 1]);
        done = res <= rtol * bnorm || hn == 0.0;
      }
      // as many steps as the last ones' rate leaves to go, less one, so that few are launched
      // in vain
      const double rate = before > 0.0 && res > 0.0 ? std::log(before / res) / nj : 0.0;
      const double left = rate > 0.0 && rtol > 0.0 ? std::log(res / (rtol * bnorm)) / rate : kBatch;
      ahead = left < kBatch + 1.0 ? std::max(1, (int)left - 1) : kBatch;
    }
    // y = H^-1 g (upper triangular j x j); x += D^-1 V y
    for (int i = j - 1; i >= 0; --i) {
      double s = g[i];
      for (int k = i + 1; k < j; ++k) s -= H[(size_t)i * m + k] * y[k];
      y[i] = s / H[(size_t)i * m + i];
    }
    CC_HIP(hipMemcpyAsync(coef, y.data(), sizeof(double) * j, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(k_update, dim3(gv), dim3(T), 0, st, n, j, coef, A.V, dinv, x);
  }
  CC_HIP(hipGetLastError());
  if (iters_out) *iters_out = it;
  if (relres_out) *relres_out = res / bnorm;
  if (!std::isfinite(res)) return fail(CUTCELL_E_BREAKDOWN, "GMRES produced a non-finite residual");
  return res <= rtol * bnorm ? CUTCELL_OK : CUTCELL_W_NOT_CONVERGED;
}

// ---------------------------------------------------------------------------------------
// Extreme eigenvalues of the volume operator A (L restricted to the volume values, the
// boundary entries of Phi zero) from Arnoldi's method on the GPU (the spectra of
// Sec. 3.4 / 3.5, at any size).

// Eigenvalues of an n x n upper Hessenberg matrix (row-major, leading dimension ld) by
// shifted QR iterations in complex arithmetic: Givens rotations reduce the active block
// minus mu I to triangular form R, the block becomes R Q + mu I, mu is the eigenvalue of
// its trailing 2 x 2 part nearer the last diagonal entry (Wilkinson's shift, perturbed
// every 11th step), and the block deflates from the bottom once a subdiagonal entry is
// below the rounding level of its diagonal neighbours.  Host code.  Returns 0, or -1 if an
// eigenvalue needs more than 200 steps.
int hessenberg_eigs(int n, const double* H, int ld, double* re, double* im) {
  using cd = std::complex<double>;
  std::vector<cd> a((size_t)n * n);
  for (int i = 0; i < n; ++i)
    for (int j = 0; j < n; ++j) a[(size_t)i * n + j] = (j >= i - 1) ? cd(H[(size_t)i * ld + j], 0.0) : cd(0.0, 0.0);
  auto A = [&](int i, int j) -> cd& { return a[(size_t)i * n + j]; };
  const double eps = 2.220446049250313e-16;
  int hi = n - 1, steps = 0;
  while (hi >= 0) {
    int lo = hi;
    while (lo > 0 && std::abs(A(lo, lo - 1)) > eps * (std::abs(A(lo, lo)) + std::abs(A(lo - 1, lo - 1)))) --lo;
    if (lo > 0) A(lo, lo - 1) = 0.0;
    if (lo == hi) {
      re[hi] = A(hi, hi).real();
      im[hi] = A(hi, hi).imag();
      --hi;
      steps = 0;
      continue;
    }
    if (++steps > 200) return -1;
    const cd a11 = A(hi - 1, hi - 1), a12 = A(hi - 1, hi), a21 = A(hi, hi - 1), a22 = A(hi, hi);
    const cd half = 0.5 * (a11 + a22);
    const cd disc = std::sqrt(0.25 * (a11 - a22) * (a11 - a22) + a12 * a21);
    const cd m1 = half + disc, m2 = half - disc;
    cd mu = (std::abs(m1 - a22) < std::abs(m2 - a22)) ? m1 : m2;
    if (steps % 11 == 10) mu = a22 + std::abs(a21);
    for (int k = lo; k <= hi; ++k) A(k, k) -= mu;
    std::vector<cd> cs(hi - lo), sn(hi - lo);
    for (int k = lo; k < hi; ++k) {            // R = Q^H (H - mu I)
      const cd x = A(k, k), y = A(k + 1, k);
      const double r = std::hypot(std::abs(x), std::abs(y));
      const cd c = r > 0.0 ? x / r : cd(1.0, 0.0), s = r > 0.0 ? y / r : cd(0.0, 0.0);
      cs[k - lo] = c;
      sn[k - lo] = s;
      for (int j = k; j <= hi; ++j) {
        const cd u = A(k, j), v = A(k + 1, j);
        A(k, j) = std::conj(c) * u + std::conj(s) * v;
        A(k + 1, j) = -s * u + c * v;
      }
    }
    for (int k = lo; k < hi; ++k) {            // R Q
      const cd c = cs[k - lo], s = sn[k - lo];
      for (int i = lo; i <= std::min(k + 1, hi); ++i) {
        const cd u = A(i, k), v = A(i, k + 1);
        A(i, k) = c * u + s * v;
        A(i, k + 1) = -std::conj(s) * u + std::conj(c) * v;
      }
    }
    for (int k = lo; k <= hi; ++k) A(k, k) += mu;
  }
  return 0;
}

// Relative residuals of Ritz pairs: for (theta, y) with H y = theta y (y of unit norm), the
// Arnoldi relation gives |A V y - theta V y| = |h_{k+1,k}| |y_k|; res = that / |theta|.
// y from three steps of inverse iteration with H - theta I (complex Gaussian elimination
// with partial pivoting; theta nudged by 1e-13 relative so the matrix stays invertible).
// Host code; k at most 256 (else res = -1).
void ritz_residuals(int k, const double* H, int ld, double hlast, const double* re, const double* im, double* res) {
  using cd = std::complex<double>;
  if (k > 256) {
    for (int t = 0; t < k; ++t) res[t] = -1.0;
    return;
  }
  std::vector<cd> M((size_t)k * k), y(k), b(k);
  for (int t = 0; t < k; ++t) {
    const cd th(re[t], im[t]);
    const cd sh = th + cd(std::abs(th) * 1e-13 + 1e-300, 0.0);
    for (int i = 0; i < k; ++i) y[i] = 1.0 / std::sqrt((double)k);
    for (int iter = 0; iter < 3; ++iter) {
      for (int i = 0; i < k; ++i)
        for (int j = 0; j < k; ++j)
          M[(size_t)i * k + j] = (j >= i - 1 ? cd(H[(size_t)i * ld + j], 0.0) : cd(0.0, 0.0)) - (i == j ? sh : cd(0.0));
      b = y;
      for (int c = 0; c < k; ++c) {
        int pr = c;
        for (int r = c + 1; r < k; ++r)
          if (std::abs(M[(size_t)r * k + c]) > std::abs(M[(size_t)pr * k + c])) pr = r;
        if (pr != c) {
          for (int j = c; j < k; ++j) std::swap(M[(size_t)c * k + j], M[(size_t)pr * k + j]);
          std::swap(b[c], b[pr]);
        }
        const cd piv = M[(size_t)c * k + c];
        if (std::abs(piv) == 0.0) continue;
        for (int r = c + 1; r < k; ++r) {
          const cd fct = M[(size_t)r * k + c] / piv;
          if (fct == cd(0.0)) continue;
          for (int j = c; j < k; ++j) M[(size_t)r * k + j] -= fct * M[(size_t)c * k + j];
          b[r] -= fct * b[c];
        }
      }
      for (int i = k - 1; i >= 0; --i) {
        cd acc = b[i];
        for (int j = i + 1; j < k; ++j) acc -= M[(size_t)i * k + j] * y[j];
        const cd piv = M[(size_t)i * k + i];
        y[i] = std::abs(piv) > 0.0 ? acc / piv : cd(0.0);
      }
      double nrm = 0.0;
      for (int i = 0; i < k; ++i) nrm += std::norm(y[i]);
      nrm = std::sqrt(nrm);
      if (!(nrm > 0.0) || !std::isfinite(nrm)) break;
      for (int i = 0; i < k; ++i) y[i] /= nrm;
    }
    res[t] = std::abs(hlast) * std::abs(y[k - 1]) / std::max(std::abs(th), 1e-300);
  }
}

// start vector: a fixed pseudo-random vector (splitmix64 of the index) in [-1, 1)
__global__ void k_start_vector(long long n, double* __restrict__ v) {
  const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i >= n) return;
  unsigned long long z = (unsigned long long)i + 0x9e3779b97f4a7c15ULL;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
  z ^= z >> 31;
  v[i] = (double)(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

// Arnoldi steps between two reads of the coefficients: products with A alone read few times,
// inner solves after each step
static int ritz_batch(int k, int inner_m) { return inner_m > 0 ? 1 : std::min(k, 64); }

size_t ritz_workspace_bytes(long long n_vol, long long n_phi, long long n_face, int k, int inner_m) {
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  const size_t nv = std::max<long long>(n_vol, 1);
  return al(sizeof(double) * n_phi) + al(sizeof(int32_t) * nv) + Arnoldi::bytes(n_vol, k, ritz_batch(k, inner_m)) +
         (inner_m > 0 ? solve_workspace_bytes(n_vol, n_phi, n_face, inner_m)
                      : al(sizeof(double) * std::max<long long>(n_face, 1)));
}

int ritz_values(const SolveOp& op, int G, const int64_t* phi_off, const int64_t* vol_off, int mode, int k,
                double inner_rtol, int inner_m, int inner_max, double* ritz_re, double* ritz_im, double* ritz_res,
                double* hess, int* n_out, char* ws, size_t ws_bytes) {
  const long long n = op.n_vol;
  if (ws_bytes < ritz_workspace_bytes(n, op.n_phi, op.n_face, k, mode == 1 ? inner_m : 0))
    return fail(CUTCELL_E_WORKSPACE, "Ritz workspace too small");
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  size_t off = 0;
  auto take = [&](size_t bytes) { char* p = ws + off; off += al(bytes); return p; };
  const size_t nv = std::max<long long>(n, 1);
  hipStream_t st = op.st;
  double* zeros = (double*)take(sizeof(double) * op.n_phi);   // mode 0: [v | 0]; mode 1: the inner solves' data
  int32_t* vphi = (int32_t*)take(sizeof(int32_t) * nv);
  Arnoldi A;
  const int batch = ritz_batch(k, mode == 1 ? inner_m : 0);
  A.layout(n, k, batch, st, take);
  // mode 0: the product's scratch; mode 1: the inner solves', which begin by writing all of
  // their first n_phi values, so that a step may leave the vector it scatters there
  char* rest = ws + off;
  double* phi0 = mode == 0 ? zeros : (double*)rest;
  const int T = 256;
  const unsigned gv = nb(n, T);
  hipLaunchKernelGGL(k_vol_phi, dim3(gv), dim3(T), 0, st, n, G, phi_off, vol_off, vphi);
  hipLaunchKernelGGL(k_fill_f64, dim3(nb(op.n_phi, T)), dim3(T), 0, st, zeros, op.n_phi, 0.0);
  hipLaunchKernelGGL(k_start_vector, dim3(gv), dim3(T), 0, st, n, A.V);
  double nrm = 0.0;
  int rc = A.norm(A.V, &nrm);
  if (rc) return rc;
  hipLaunchKernelGGL(k_first, dim3(gv), dim3(T), 0, st, n, 1.0 / nrm, A.V, nullptr, vphi, phi0);
  std::vector<double> Hm((size_t)(k + 1) * k, 0.0), hc((size_t)batch * (k + 1));
  int kk = k, inner_fail = 0;
  for (int j = 0; j < k; ++j) {
    if (mode == 0) {
      rc = op.lap_ptr ? apply_laplacian(op.D, n, op.lap_ptr, op.lap_col, op.lap_val, phi0, A.w, st)
                      : apply_operator(op.D, op.n_face, n, op.row_ptr, op.col, op.val, op.vol_face, op.vol_scale, phi0,
                                       A.w, (double*)rest, nullptr, st);
      if (rc) return rc;
    } else {
      hipLaunchKernelGGL(k_fill_f64, dim3(gv), dim3(T), 0, st, A.w, n, 0.0);
      int it = 0;
      double rr = 0.0;
      rc = solve_poisson(op, G, phi_off, vol_off, zeros, A.V + (long long)j * n, A.w, inner_m, inner_max, inner_rtol,
                         rest, solve_workspace_bytes(n, op.n_phi, op.n_face, inner_m), &it, &rr);
      if (rc == CUTCELL_W_NOT_CONVERGED) inner_fail = 1;
      else if (rc) return rc;
    }
    A.step(j, j % batch, nullptr, vphi, phi0);
    if ((j + 1) % batch == 0 || j + 1 == k) {
      const int j0 = j - j % batch;
      rc = A.columns(j + 1 - j0, hc.data());
      if (rc) return rc;
      bool invariant = false;
      for (int c = j0; c <= j && !invariant; ++c) {
        const double* h = hc.data() + (size_t)(c - j0) * (k + 1);
        for (int i = 0; i <= c + 1; ++i) Hm[(size_t)i * k + c] = h[i];
        if (!(h[c + 1] > 0.0)) {   // invariant subspace: its eigenvalues are exact
          kk = c + 1;
          invariant = true;
        }
      }
      if (invariant) break;
    }
  }
  CC_HIP(hipGetLastError());
  if (hess)
    for (size_t i = 0; i < Hm.size(); ++i) hess[i] = Hm[i];
  if (hessenberg_eigs(kk, Hm.data(), k, ritz_re, ritz_im)) return fail(CUTCELL_E_BREAKDOWN, "Hessenberg QR did not converge");
  if (ritz_res) ritz_residuals(kk, Hm.data(), k, kk < k ? 0.0 : Hm[(size_t)kk * k + (kk - 1)], ritz_re, ritz_im, ritz_res);
  if (mode == 1)                // eigenvalues of A^-1: invert
    for (int i = 0; i < kk; ++i) {
      const double a = ritz_re[i], b = ritz_im[i], d = a * a + b * b;
      ritz_re[i] = d > 0.0 ? a / d : 0.0;
      ritz_im[i] = d > 0.0 ? -b / d : 0.0;
    }
  *n_out = kk;
  return inner_fail ? CUTCELL_W_NOT_CONVERGED : CUTCELL_OK;
}

}  // namespace cutcell
