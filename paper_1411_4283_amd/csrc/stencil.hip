// Host side of the stencil solves: launches per bin (the kernels are in stencil_impl.hpp,
// instantiated per dimension and order in stencil_d*q*.hip), the faces with fewer rows
// than monomials, the template copies, and the launch-schedule autotuner.
#include "stencil_impl.hpp"

namespace cutcell {

// Faces with fewer rows than monomials: zero stencil, status INSUFFICIENT_ROWS -- except,
// under Neumann EB conditions, the EB faces, whose one-row stencil is their area
// |A_f| = h^(D-1) m^0 (the flux is the prescribed data).
__global__ void k_insufficient(const int32_t* __restrict__ perm, long long n, const int64_t* __restrict__ row_ptr,
                               double* val, int8_t* status, int32_t* flagged, const int32_t* __restrict__ fcode,
                               const int32_t* __restrict__ fref, const GeomPtrs* __restrict__ geoms, int neumann,
                               double hd1, int M) {
  long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t F = perm[t];
  const int32_t code = fcode[F];
  if (neumann && ((code >> 2) & 3) == 1) {
    const double area = hd1 * geoms[code >> 4].eb_mom[(long long)fref[F] * M];
    const bool ok = isfinite(area);
    val[row_ptr[F]] = ok ? area : 0.0;
    status[F] = ok ? CUTCELL_STATUS_OK : CUTCELL_STATUS_NONFINITE;
    if (!ok) atomicAdd(flagged, 1);
    return;
  }
  for (int64_t j = row_ptr[F]; j < row_ptr[F + 1]; ++j) val[j] = 0.0;
  status[F] = CUTCELL_STATUS_INSUFFICIENT_ROWS;
  atomicAdd(flagged, 1);
}

// Faces whose system is bitwise that of their template face: the template's values (the
// same rows in the same order) and status.  One wave per face.
__global__ __launch_bounds__(64) void k_copy_template(const int32_t* __restrict__ perm, long long n,
                                                      const int32_t* __restrict__ tmpl,
                                                      const int64_t* __restrict__ row_ptr, double* val, int8_t* status,
                                                      int32_t* flagged) {
  const long long t = blockIdx.x;
  if (t >= n) return;
  const int32_t F = perm[t];
  const int32_t T = tmpl[F];
  const int64_t a = row_ptr[F], b = row_ptr[T];
  const int N = (int)(row_ptr[F + 1] - a);
  for (int i = threadIdx.x; i < N; i += 64) val[a + i] = val[b + i];
  if (threadIdx.x == 0) {
    const int8_t s = status[T];
    status[F] = s;
    if (s != CUTCELL_STATUS_OK) atomicAdd(flagged, 1);
  }
}

// faces with fewer rows than monomials carry no gradient
__global__ void k_insufficient_backward(const int32_t* __restrict__ perm, long long n,
                                        const int64_t* __restrict__ row_ptr, int M, BackwardArgs B) {
  long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (t >= n) return;
  const int32_t F = perm[t];
  for (int64_t j = row_ptr[F]; j < row_ptr[F + 1]; ++j) {
    B.nz_rz[2 * j] = 0.0;
    B.nz_rz[2 * j + 1] = 0.0;
    if (B.weight_bar) B.weight_bar[j] = 0.0;
  }
  for (int p = 0; p < 2 * M; ++p) B.face_yw[(long long)F * 2 * M + p] = 0.0;
  for (int k = 0; k < 4; ++k) {
    B.owner_grad[(long long)F * 4 + k] = 0.0;
    B.face_x0[(long long)F * 4 + k] = 0.0;
  }
}

static int run_bins(const Work& w, const cutcell_opts& o, const int32_t* bin_count, const int64_t* row_ptr,
                    const int32_t* col, double* val, int8_t* status, hipStream_t st, const BackwardArgs* bw,
                    const BinSchedule* sched, int only_width = 0) {
  double hscale = 1.0;
  for (int d = 0; d < o.dim - 2; ++d) hscale *= o.h;   // h^(D-2)
  const bool neu = o.eb_bc == CUTCELL_BC_NEUMANN;
  const bool qr_all = !bw && o.factorization == CUTCELL_FACTOR_QR;
  const bool route = o.factorization != CUTCELL_FACTOR_GRAM;
  BinSchedule sc[kMaxBins];
  for (int b = 0; b < kMaxBins; ++b) {
    sc[b] = sched[b];
    sc[b].route = route;
  }
  int rc = CUTCELL_E_UNSUPPORTED;
  if (qr_all) {
    // every face of the row bins (or of those of one width) by Householder QR
    long long first = 0, n = 0;
    for (int b = 0; b < kMaxBins; ++b) {
      if (only_width == 0 || bin_width(b) == only_width) n += bin_count[b];
      else if (bin_width(b) < only_width) first += bin_count[b];
    }
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, w.qr_count, 1LL, (int32_t)n);
    rc = solve_qr_faces(w, o, w.perm + first, nullptr, n, row_ptr, col, val, status, st);
    if (rc != CUTCELL_OK) return rc;
  } else {
#define CC_RB(DD, QQ) \
  if (o.dim == DD && o.order == QQ) \
    rc = dispatch_row_bins<DD, QQ>(w, hscale, bin_count, row_ptr, col, val, status, st, bw, sc, only_width, neu, o.h, \
                                   o.weight_custom ? o.weight_power : 5.0);
    CC_RB(2, 2) CC_RB(2, 4) CC_RB(3, 2) CC_RB(3, 4)
#undef CC_RB
    if (rc == CUTCELL_E_UNSUPPORTED) return fail(CUTCELL_E_UNSUPPORTED, "order/dimension");
    if (rc != CUTCELL_OK) return rc;
    // the faces the Gram path left to Householder QR (their count is on the device), unless
    // the launch of one width alone is asked for
    if (!bw && route && only_width == 0) {
      rc = solve_qr_faces(w, o, w.qr_list, w.qr_count, 0, row_ptr, col, val, status, st);
      if (rc != CUTCELL_OK) return rc;
    }
  }
  // after the bins: faces with fewer rows than monomials, and the template copies (the
  // templates are solved by then: same stream)
  const int M = binom(o.order + o.dim, o.dim);
  long long start = 0;
  for (int b = 0; b < kMaxBins; ++b) start += bin_count[b];
  const long long ninsuf = (only_width == 0) ? bin_count[kMaxBins] : 0;
  const long long ncopy = (only_width == 0 && !bw) ? bin_count[kMaxBins + 1] : 0;
  if (ncopy > 0)
    hipLaunchKernelGGL(k_copy_template, dim3((unsigned)ncopy), dim3(64), 0, st, w.perm + start + bin_count[kMaxBins],
                       ncopy, w.tmpl, row_ptr, val, status, w.flagged);
  if (ninsuf > 0 && bw)
    hipLaunchKernelGGL(k_insufficient_backward, dim3((unsigned)((ninsuf + 255) / 256)), dim3(256), 0, st,
                       w.perm + start, ninsuf, row_ptr, M, *bw);
  else if (ninsuf > 0)
    hipLaunchKernelGGL(k_insufficient, dim3((unsigned)((ninsuf + 255) / 256)), dim3(256), 0, st, w.perm + start,
                       ninsuf, row_ptr, val, status, w.flagged, w.fcode, w.fref, w.geoms, (int)neu,
                       o.dim == 3 ? o.h * o.h : o.h, M);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

static void schedules_from(const cutcell_tuning* t, BinSchedule* sc) {
  for (int b = 0; b < kMaxBins; ++b) {
    sc[b] = BinSchedule{};
    if (t) {
      sc[b].xcd = t->xcd_chunks[b] > 1 ? t->xcd_chunks[b] : 1;
      sc[b].per_xcd = t->blocks_per_xcd[b] > 0 ? t->blocks_per_xcd[b] : 0;
    }
  }
}

int solve_stencils(const Work& w, const cutcell_opts& o, const int32_t* bin_count, long long n_face,
                   const int64_t* row_ptr, const int32_t* col, double* val, int8_t* status, hipStream_t st) {
  (void)n_face;
  BinSchedule sc[kMaxBins];
  schedules_from(o.tuning, sc);
  return run_bins(w, o, bin_count, row_ptr, col, val, status, st, nullptr, sc);
}

int backward_stencils(const Work& w, const cutcell_opts& o, const int32_t* bin_count, const int64_t* row_ptr,
                      const int32_t* col, const BackwardArgs& bw, hipStream_t st) {
  BinSchedule sc[kMaxBins];
  schedules_from(nullptr, sc);
  return run_bins(w, o, bin_count, row_ptr, col, nullptr, nullptr, st, &bw, sc);
}

// Times the launch schedules on these faces (HIP events, best of `reps`).  Bins of one kernel
// width run as one launch as long as their schedules agree, so the candidates are timed per
// width, without the QR launch that all bins share, and every bin of a width gets the same
// one.  A schedule replaces the default where it is faster by more than kTuneMargin (best of a
// few runs differ by about 1 %), and the choice as a whole has to be so in the whole solve:
// schedules kept per bin had parted the launches, 64 geometries of 48^3, order 4, 286 ms
// against 259 with the default.  Then solves all bins with the choice, so val/status hold the
// same stencils as an untuned build.
constexpr double kTuneMargin = 0.02;

int tune_stencils(const Work& w, const cutcell_opts& o, const int32_t* bin_count, const int64_t* row_ptr,
                  const int32_t* col, double* val, int8_t* status, hipStream_t st, cutcell_tuning* out, int reps,
                  double* best_ms) {
  int dev = 0, cus = 256;
  CC_HIP(hipGetDevice(&dev));
  CC_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int X = kXcds;
  const int resident = std::max(1, cus / X) * 4;   // workgroups per XCD at one wave per SIMD
  const BinSchedule launch[] = {{1, 0}, {X, 0}, {X, resident}, {X, 2 * resident}, {1, X * resident}};
  struct Events {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    ~Events() {
      if (e0) (void)hipEventDestroy(e0);
      if (e1) (void)hipEventDestroy(e1);
    }
  } ev;
  CC_HIP(hipEventCreate(&ev.e0));
  CC_HIP(hipEventCreate(&ev.e1));
  // one run of the bins of a width (all of them: 0) under schedules s; *ms becomes the less
  auto timed = [&](const BinSchedule* s, int width, double* ms) -> int {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, w.flagged, 4LL, 0);   // and qr_count
    CC_HIP(hipEventRecord(ev.e0, st));
    const int rc = run_bins(w, o, bin_count, row_ptr, col, val, status, st, nullptr, s, width);
    if (rc) return rc;
    CC_HIP(hipEventRecord(ev.e1, st));
    CC_HIP(hipEventSynchronize(ev.e1));
    float t = 0.f;
    CC_HIP(hipEventElapsedTime(&t, ev.e0, ev.e1));
    *ms = std::min(*ms, (double)t);
    return CUTCELL_OK;
  };
  BinSchedule plain[kMaxBins], sc[kMaxBins];
  schedules_from(nullptr, plain);
  schedules_from(nullptr, sc);
  double warm = 1e300;   // the default is timed first: not with cold caches
  int wrc = timed(plain, 0, &warm);
  if (wrc) return wrc;
  bool tuned = false;
  for (int b = 0, e = 0; b < kMaxBins; b = e) {
    long long n = 0;
    for (e = b; e < kMaxBins && bin_width(e) == bin_width(b); ++e) n += bin_count[e];
    for (int i = b; i < e; ++i) best_ms[i] = -1.0;
    if (n == 0) continue;
    double best = 1e300, bound = 1e300;
    for (const BinSchedule& cand : launch) {
      BinSchedule trial[kMaxBins];
      for (BinSchedule& t : trial) t = cand;
      double tmin = 1e300;
      for (int r = 0; r < reps; ++r) {
        const int rc = timed(trial, bin_width(b), &tmin);
        if (rc) return rc;
      }
      if (&cand == launch) {   // the default
        best = tmin;
        bound = tmin * (1.0 - kTuneMargin);
      } else if (tmin < bound) {
        best = bound = tmin;
        tuned = true;
        for (int i = b; i < e; ++i) sc[i] = cand;
      }
    }
    for (int i = b; i < e; ++i)
      if (bin_count[i] > 0) best_ms[i] = best;
  }
  if (tuned) {
    double with = 1e300, without = 1e300;
    for (int r = 0; r <= reps; ++r) {
      int rc = timed(plain, 0, &without);
      if (!rc) rc = timed(sc, 0, &with);
      if (rc) return rc;
    }
    if (!(with < without * (1.0 - kTuneMargin))) schedules_from(nullptr, sc);
  }
  for (int b = 0; b < kMaxBins; ++b) {
    out->xcd_chunks[b] = sc[b].xcd;
    out->blocks_per_xcd[b] = sc[b].per_xcd;
    out->split[b] = 0;
  }
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, w.flagged, 4LL, 0);   // and qr_count
  return run_bins(w, o, bin_count, row_ptr, col, val, status, st, nullptr, sc);
}

}  // namespace cutcell
