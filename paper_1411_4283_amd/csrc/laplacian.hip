// The operator as one sparse matrix over volumes (Sec. 2.2, eq. 'laplacian over V'):
//   L_v = vol_scale[v] * sum over v's faces f of sigma_vf s_f^T Phi = sum_k lap_v[k] Phi[k],
// lap_v the sigma-signed, volume-scaled merge of the stencil rows of v's <= 2D+1 faces.
// The apply is then one CSR gather per volume: for a regular 3D volume at path radius 3
// about 129 entries instead of the ~264 face entries it shares, and no flux array.
//
// One wave per volume merges the face rows through a hash table of columns in shared memory.
// The rows go in one after the other (their columns are distinct, so the lanes of a row
// never meet in an entry): a column's values are summed in the order of its rows, and the
// sum is scaled by vol_scale.  The columns that a row adds are listed; those of the first
// row come sorted, so a column's place in the merged row is its place among them plus the
// number of later ones below it.  A count pass and a fill pass; the result does not depend
// on the launch.  What bounds it is the latency of a row's insertion behind the one before
// it.  48^3, path radius 3 (100k volumes, 4.6e7 face entries read): count 0.10, fill 0.32 ms;
// with every entry's place found by binary searches in the other rows, in both passes, and
// the merged rows in 24 KB of shared memory, 2.36 and 2.81 ms.
#include <algorithm>
#include <cstddef>

#include "gather.hpp"
#include "scan.hpp"
#include "solve.hpp"

namespace cutcell {

constexpr int kLapPad = 1024;   // >= (2D+1) rows of <= kMaxRows entries
constexpr int kLapFast = 512;   // hash table of the fill for rows of at most 7/8 of that

// Hash table of at most CAP columns, and with FILL their sums and the list of them (which is
// read 16 bytes at a time).
template <int CAP, bool FILL>
struct __align__(16) LapTable {
  int32_t key[CAP];
  double sum[FILL ? CAP : 1];
  int32_t list[FILL ? CAP + 8 : 4];   // columns in the order they were added
  uint16_t slot[FILL ? CAP + 8 : 1];  // and their entries
};

// Adds column c (of the lanes with `on`) to the table: its entry, and whether it is new
// there.  A full table (rows other than the counted ones) ends the search.
template <int CAP>
__device__ __forceinline__ int lap_insert(int32_t* key, bool on, int32_t c, bool* fresh) {
  int h = (int)(((unsigned)c * 2654435769u) >> 22) & (CAP - 1);
  bool go = on;
  *fresh = false;
  for (int probe = 0; probe < CAP && __any(go); ++probe) {
    if (go) {
      const int32_t old = atomicCAS(&key[h], -1, c);
      *fresh = old == -1;
      go = old != -1 && old != c;
      if (go) h = (h + 1) & (CAP - 1);
    }
  }
  return h;
}

template <int D, int CAP, bool FILL>
__device__ __forceinline__ void merge_row(LapTable<CAP, FILL>& tb, long long v, const int32_t* __restrict__ vol_face,
                                          const double* __restrict__ vol_scale, const int64_t* __restrict__ row_ptr,
                                          const int32_t* __restrict__ col, const double* __restrict__ val,
                                          int32_t* __restrict__ count, const int64_t* __restrict__ lap_ptr,
                                          int32_t* __restrict__ lap_col, double* __restrict__ lap_val,
                                          int32_t* too_long) {
  constexpr int S = 2 * D + 1;
  using Table = LapTable<CAP, FILL>;
  static_assert(!FILL || (alignof(Table) >= 16 && offsetof(Table, list) % 16 == 0), "the list is read 16 bytes at a time");
  const int lane = threadIdx.x & 63;
  int64_t start[S];
  int len[S];
  int tot = 0;
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const int32_t f = vol_face[v * S + k];
    start[k] = 0;
    len[k] = 0;
    if (f >= 0) {
      start[k] = row_ptr[f];
      len[k] = (int)(row_ptr[f + 1] - start[k]);
    }
    tot += len[k];
  }
  if (tot > kLapPad) {   // rows not from a build (a build has at most kMaxRows per face)
    if (lane == 0) {
      if (!FILL) count[v] = 0;
      if (too_long) atomicOr(too_long, 1);
    }
    return;
  }
  // the first 128 entries of every row at once
  int32_t c[S][2];
  double x[S][2];
#pragma unroll
  for (int k = 0; k < S; ++k)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int i = lane + 64 * u;
      c[k][u] = i < len[k] ? col[start[k] + i] : 0;
      x[k][u] = (FILL && i < len[k]) ? val[start[k] + i] : 0.0;
    }
  for (int i = lane; i < CAP; i += 64) {
    tb.key[i] = -1;
    if (FILL) tb.sum[i] = 0.0;
  }
  // (without this the loads move down to the insertions and wait there one after the other)
#pragma unroll
  for (int k = 0; k < S; ++k)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      asm volatile("" : "+v"(c[k][u]));
      if (FILL) asm volatile("" : "+v"(x[k][u]));
    }
  __syncthreads();
  int n = 0, n0 = 0;   // columns in the list, and those of the first row that has any
  const unsigned long long below = lanes_below(lane);
  auto add = [&](bool on, int32_t ci, double xi) {
    bool fresh;
    const int h = lap_insert<CAP>(tb.key, on, ci, &fresh);
    const unsigned long long m = __ballot(fresh);
    if (FILL) {
      if (on) __hip_atomic_fetch_add(&tb.sum[h], xi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (fresh) {
        const int p = min(n + __popcll(m & below), CAP + 7);
        tb.list[p] = ci;
        tb.slot[p] = (uint16_t)h;
      }
    }
    n += __popcll(m);
  };
#pragma unroll
  for (int k = 0; k < S; ++k) {
    const double sg = (k < 2 * D && (k & 1) == 0) ? -1.0 : 1.0;   // low faces point into v
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (64 * u < len[k]) add(lane + 64 * u < len[k], c[k][u], sg * x[k][u]);
    for (int i = 128; i < len[k]; i += 64) {
      const bool on = i + lane < len[k];
      add(on, on ? col[start[k] + i + lane] : 0, (FILL && on) ? sg * val[start[k] + i + lane] : 0.0);
    }
    if (n0 == 0) {
      n0 = n;
      if (FILL) {   // the columns that follow start at a multiple of four
        if (lane < 4) tb.list[n + lane] = 0x7fffffff;
        n = (n + 3) & ~3;
      }
    }
  }
  if constexpr (!FILL) {
    if (lane == 0) count[v] = n;
    return;
  } else {
    const int first = (n0 + 3) & ~3;
    n = min(n, CAP + 4);
    if (lane < 4) tb.list[n + lane] = 0x7fffffff;
    __syncthreads();
    const int64_t pos = lap_ptr[v];
    const double sc = vol_scale[v];
    for (int i0 = 0; i0 < n; i0 += 64) {
      const int i = i0 + lane;
      const bool in = i < n0 || (i >= first && i < n);
      const int32_t key = in ? tb.list[i] : 0;
      int rank = i;
      if (i0 + 64 > n0) {   // columns of later rows: their place among the first row's
        int lo = 0, hi = n0;
        while (__any(lo < hi)) {
          const int mid = (lo + hi) >> 1;
          if (lo < hi) {
            if (tb.list[mid] < key) lo = mid + 1;
            else hi = mid;
          }
        }
        rank = i < n0 ? i : lo;
      }
      for (int j = first; j < n; j += 4) {   // every lane reads the same four
        const int4 q = *reinterpret_cast<const int4*>(&tb.list[j]);
        rank += (q.x < key) + (q.y < key) + (q.z < key) + (q.w < key);
      }
      if (in) {
        lap_col[pos + rank] = key;
        lap_val[pos + rank] = sc * tb.sum[tb.slot[i]];
      }
    }
  }
}

template <int D>
__global__ __launch_bounds__(64) void k_lap_count(long long n_vol, const int32_t* __restrict__ vol_face,
                                                  const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                  int32_t* __restrict__ count, int32_t* too_long) {
  __shared__ LapTable<kLapPad, false> tb;
  merge_row<D, kLapPad, false>(tb, blockIdx.x, vol_face, nullptr, row_ptr, col, nullptr, count, nullptr, nullptr,
                               nullptr, too_long);
}

// Volumes whose merged rows fit the small table, one wave each: 9,264 bytes of shared memory
// leave 17 waves to a CU, the large table's 18,480 eight.
constexpr int kLapFastRows = kLapFast / 8 * 7;
template <int D>
__global__ __launch_bounds__(64) void k_lap_fill(long long n_vol, const int32_t* __restrict__ vol_face,
                                                 const double* __restrict__ vol_scale,
                                                 const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                 const double* __restrict__ val, const int64_t* __restrict__ lap_ptr,
                                                 int32_t* __restrict__ lap_col, double* __restrict__ lap_val) {
  __shared__ LapTable<kLapFast, true> tb;
  const long long v = blockIdx.x;
  if (lap_ptr[v + 1] - lap_ptr[v] > kLapFastRows) return;
  merge_row<D, kLapFast, true>(tb, v, vol_face, vol_scale, row_ptr, col, val, nullptr, lap_ptr, lap_col, lap_val,
                               nullptr);
}

// The others: a wave looks through 64 volumes.
template <int D>
__global__ __launch_bounds__(64) void k_lap_fill_long(long long n_vol, const int32_t* __restrict__ vol_face,
                                                      const double* __restrict__ vol_scale,
                                                      const int64_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ col, const double* __restrict__ val,
                                                      const int64_t* __restrict__ lap_ptr,
                                                      int32_t* __restrict__ lap_col, double* __restrict__ lap_val) {
  __shared__ LapTable<kLapPad, true> tb;
  const long long v0 = blockIdx.x * 64LL, v = v0 + threadIdx.x;
  for (unsigned long long m = __ballot(v < n_vol && lap_ptr[v + 1] - lap_ptr[v] > kLapFastRows); m != 0; m &= m - 1) {
    merge_row<D, kLapPad, true>(tb, v0 + __ffsll((long long)m) - 1, vol_face, vol_scale, row_ptr, col, val, nullptr,
                                lap_ptr, lap_col, lap_val, nullptr);
    __syncthreads();   // the next row reuses the table
  }
}

size_t laplacian_temp_bytes(long long n_vol) {
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  const long long n = std::max<long long>(n_vol, 1);
  return al(sizeof(int32_t) * n) + al(sizeof(int64_t) * (scan_tiles(n) + 1)) + al(sizeof(int32_t));
}

int laplacian_count(int D, long long n_vol, const int64_t* row_ptr, const int32_t* col, const double* val,
                    const int32_t* vol_face, const double* vol_scale, int64_t* lap_ptr, int64_t* nnz, char* ws,
                    size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < laplacian_temp_bytes(n_vol)) return fail(CUTCELL_E_WORKSPACE, "Laplacian workspace too small");
  auto al = [](size_t x) { return (x + 255) & ~size_t(255); };
  const long long n1 = std::max<long long>(n_vol, 1);
  int32_t* cnt = (int32_t*)ws;
  int64_t* tmp = (int64_t*)(ws + al(sizeof(int32_t) * n1));
  int32_t* too_long = (int32_t*)(ws + al(sizeof(int32_t) * n1) + al(sizeof(int64_t) * (scan_tiles(n1) + 1)));
  *nnz = 0;
  if (n_vol <= 0) {
    const int64_t zero = 0;
    CC_HIP(hipMemcpyAsync(lap_ptr, &zero, sizeof(int64_t), hipMemcpyHostToDevice, st));
    CC_HIP(hipStreamSynchronize(st));
    return CUTCELL_OK;
  }
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, too_long, 1LL, 0);
  if (D == 3)
    hipLaunchKernelGGL(k_lap_count<3>, dim3((unsigned)n_vol), dim3(64), 0, st, n_vol, vol_face, row_ptr, col, cnt,
                       too_long);
  else
    hipLaunchKernelGGL(k_lap_count<2>, dim3((unsigned)n_vol), dim3(64), 0, st, n_vol, vol_face, row_ptr, col, cnt,
                       too_long);
  int rc = exclusive_scan<int32_t, int64_t>(cnt, n_vol, n_vol, 1, lap_ptr, n_vol, lap_ptr + n_vol, tmp, st);
  if (rc) return rc;
  int32_t bad = 0;
  CC_HIP(hipMemcpyAsync(nnz, lap_ptr + n_vol, sizeof(int64_t), hipMemcpyDeviceToHost, st));
  CC_HIP(hipMemcpyAsync(&bad, too_long, sizeof(int32_t), hipMemcpyDeviceToHost, st));
  CC_HIP(hipStreamSynchronize(st));
  CC_HIP(hipGetLastError());
  if (bad) return fail(CUTCELL_E_UNSUPPORTED, "a volume's face rows hold more than 1024 entries");
  return CUTCELL_OK;
}

int laplacian_fill(int D, long long n_vol, const int64_t* row_ptr, const int32_t* col, const double* val,
                   const int32_t* vol_face, const double* vol_scale, const int64_t* lap_ptr, int32_t* lap_col,
                   double* lap_val, hipStream_t st) {
  if (n_vol <= 0) return CUTCELL_OK;
  const dim3 all((unsigned)n_vol), some((unsigned)((n_vol + 63) / 64)), block(64);
  if (D == 3) {
    hipLaunchKernelGGL(k_lap_fill<3>, all, block, 0, st, n_vol, vol_face, vol_scale, row_ptr, col, val, lap_ptr, lap_col,
                       lap_val);
    hipLaunchKernelGGL(k_lap_fill_long<3>, some, block, 0, st, n_vol, vol_face, vol_scale, row_ptr, col, val, lap_ptr,
                       lap_col, lap_val);
  } else {
    hipLaunchKernelGGL(k_lap_fill<2>, all, block, 0, st, n_vol, vol_face, vol_scale, row_ptr, col, val, lap_ptr, lap_col,
                       lap_val);
    hipLaunchKernelGGL(k_lap_fill_long<2>, some, block, 0, st, n_vol, vol_face, vol_scale, row_ptr, col, val, lap_ptr,
                       lap_col, lap_val);
  }
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

// L = lap Phi: one CSR gather over the volumes (F rows per wave, U rounds of 64 entries)
int apply_laplacian(int D, long long n_vol, const int64_t* lap_ptr, const int32_t* lap_col, const double* lap_val,
                    const double* phi, double* lphi, hipStream_t st) {
  if (n_vol <= 0) return CUTCELL_OK;
  const int T = 256;
  if (D == 3) {
    constexpr int F = 4, U = 10;  // ~129 entries per regular volume (the fastest shape measured)
    const long long waves = (n_vol + F - 1) / F;
    hipLaunchKernelGGL((k_flux<F, U>), dim3((unsigned)((waves * 64 + T - 1) / T)), dim3(T), 0, st, n_vol, lap_ptr,
                       lap_col, lap_val, phi, lphi);
  } else {
    constexpr int F = 8, U = 4;   // ~25-40 entries per volume
    const long long waves = (n_vol + F - 1) / F;
    hipLaunchKernelGGL((k_flux<F, U>), dim3((unsigned)((waves * 64 + T - 1) / T)), dim3(T), 0, st, n_vol, lap_ptr,
                       lap_col, lap_val, phi, lphi);
  }
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

}  // namespace cutcell
