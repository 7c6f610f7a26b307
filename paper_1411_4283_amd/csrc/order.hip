// Processing order of the faces (the permutation the stencil kernels walk).  Faces are
// grouped by bucket (16-row bins, then faces with fewer rows than monomials, then template
// copies), and inside that ordered by the cell they sit at -- a grid face's low-side
// cell (the last cell for faces on the high box side), an EB face's cut cell -- so that
// the faces of all directions around the same cells are solved together and share the
// rows' moments in one L2.  The stencils do not depend on the order.
//
// The faces of a cell are known from the enumeration's tables, so walking the cells gives
// them in order and only the buckets are left to separate: a count per tile of cells and
// bucket, a scan of those counts, and a second walk that writes each face to its place.  A
// thread's counts of the ten buckets share two 64-bit words, 12 bits each.  Bound by the
// launches and, from some 10^5 cells on, by the reads of the two walks; 64^3, path radius 3
// (724k faces): 240 us as a radix sort of 44-bit keys with the bucket counts and the most rows
// by atomics, 27 us like this.
#include "kernels.hpp"

namespace cutcell {

constexpr int kOrderThreads = 256;
constexpr int kFieldBits = 12, kFields = 5;   // counts in a word: at most 7 faces of each of 256 cells
static_assert(7 * kOrderThreads < (1 << kFieldBits) && kFields * kFieldBits <= 64 && 2 * kFields >= kNBuckets,
              "the counts of a tile step must fit in their fields");

struct OrderArgs {
  GridDims g;
  int G, M;
  int steps;          // steps of 256 cells of a workgroup
  int tiles;          // workgroups
  const int32_t* face_id;
  const int32_t* eb_id;
  const int64_t* counts;
  const int64_t* offs;
  const int32_t* nrows;
  const int32_t* tmpl;
};

struct Packed2 {
  unsigned long long w[2];
  __device__ __forceinline__ void add(int bucket) {
    const unsigned long long one = 1ULL << (kFieldBits * (bucket % kFields));
    w[0] += bucket < kFields ? one : 0;
    w[1] += bucket < kFields ? 0 : one;
  }
  __device__ __forceinline__ int get(int bucket) const {
    const unsigned long long v = bucket < kFields ? w[0] : w[1];
    return (int)(v >> (kFieldBits * (bucket % kFields))) & ((1 << kFieldBits) - 1);
  }
};

// the faces at cell i of the batch, in ascending order: at most two per direction and the EB face
template <class Fn>
__device__ __forceinline__ void faces_of_cell(const OrderArgs& A, long long i, Fn&& fn) {
  const GridDims& g = A.g;
  if (i >= A.G * g.ncell) return;
  const int gi = (int)(i / g.ncell);
  const int c = (int)(i - gi * g.ncell);
  int x[3];
  cell_coords(g, c, x);
  const long long F0 = A.offs[2 * (A.G + 1) + gi];
  const int32_t* fid = A.face_id + (long long)gi * g.NF;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    if (d >= g.D) break;
    const int m0 = g.n[0] + (d == 0), m1 = g.n[1] + (d == 1);
    const long long lf = g.foff[d] + x[0] + (long long)m0 * (x[1] + (long long)m1 * x[2]);
    const long long up = d == 0 ? 1 : d == 1 ? m0 : (long long)m0 * m1;
    const int32_t a = fid[lf];
    const int32_t b = x[d] == g.n[d] - 1 ? fid[lf + up] : -1;
    if (a >= 0) fn(F0 + a);
    if (b >= 0) fn(F0 + b);
  }
  const int32_t e = A.eb_id[i];
  if (e >= 0) fn(F0 + A.counts[4 * gi + 3] + e);
}

// hist[bucket][tile] and the most rows of a face of the tile
__global__ __launch_bounds__(kOrderThreads) void k_order_count(OrderArgs A, int32_t* __restrict__ hist,
                                                               int32_t* __restrict__ tile_max) {
  __shared__ int32_t part[kOrderThreads / 64][kNBuckets], pmax[kOrderThreads / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int mine = 0, mr = 0;   // lane b: the wave's faces of bucket b
  for (int s = 0; s < A.steps; ++s) {
    const long long i = ((long long)blockIdx.x * A.steps + s) * kOrderThreads + threadIdx.x;
    Packed2 p{{0, 0}};
    faces_of_cell(A, i, [&](long long F) {
      p.add(face_bucket(F, A.M, A.nrows, A.tmpl));
      mr = max(mr, A.nrows[F]);
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      p.w[0] += __shfl_xor(p.w[0], o, 64);
      p.w[1] += __shfl_xor(p.w[1], o, 64);
    }
    if (lane < kNBuckets) mine += p.get(lane);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mr = max(mr, __shfl_xor(mr, o, 64));
  if (lane < kNBuckets) part[wave][lane] = mine;
  if (lane == 0) pmax[wave] = mr;
  __syncthreads();
  if (threadIdx.x < kNBuckets) {
    int s = 0;
    for (int k = 0; k < kOrderThreads / 64; ++k) s += part[k][threadIdx.x];
    hist[threadIdx.x * A.tiles + blockIdx.x] = s;
  }
  if (threadIdx.x == 0) {
    int m = 0;
    for (int k = 0; k < kOrderThreads / 64; ++k) m = max(m, pmax[k]);
    tile_max[blockIdx.x] = m;
  }
}

// hist becomes its exclusive sums; bins: the buckets' counts, their starts, the most rows and
// the nonzeros
__global__ __launch_bounds__(1024) void k_order_scan(int tiles, int32_t* __restrict__ hist,
                                                     const int32_t* __restrict__ tile_max, int32_t* __restrict__ bins,
                                                     long long n_face, int64_t* __restrict__ row_ptr) {
  __shared__ int32_t wsum[16], wmax[16], start[kNBuckets + 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int n = kNBuckets * tiles, per = (n + 1023) / 1024;
  const int a = min(t * per, n), b = min(a + per, n);
  int s = 0, mr = 0;
  for (int i = a; i < b; ++i) s += hist[i];
  for (int i = t; i < tiles; i += 1024) mr = max(mr, tile_max[i]);
  int incl = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int v = __shfl_up(incl, o, 64);
    if (lane >= o) incl += v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) mr = max(mr, __shfl_xor(mr, o, 64));
  if (lane == 63) wsum[wave] = incl;
  if (lane == 0) wmax[wave] = mr;
  __syncthreads();
  int run = incl - s;
  for (int k = 0; k < wave; ++k) run += wsum[k];
  for (int i = a; i < b; ++i) {
    const int v = hist[i];
    hist[i] = run;
    if (i % tiles == 0) start[i / tiles] = run;
    run += v;
  }
  if (t == 1023) start[kNBuckets] = run;
  __syncthreads();
  if (t < kNBuckets) {
    bins[t] = start[t + 1] - start[t];
    bins[kNBuckets + t] = start[t];
  }
  if (t == 0) {
    int m = 0;
    for (int k = 0; k < 16; ++k) m = max(m, wmax[k]);
    bins[2 * kNBuckets] = m;
    if (row_ptr) {
      if (n_face == 0) row_ptr[0] = 0;
      *(int64_t*)(bins + 2 * kNBuckets + 2) = n_face == 0 ? 0 : row_ptr[n_face];
    }
  }
}

__global__ __launch_bounds__(kOrderThreads) void k_order_write(OrderArgs A, const int32_t* __restrict__ base,
                                                               int32_t* __restrict__ perm) {
  constexpr int NW = kOrderThreads / 64;
  __shared__ unsigned long long wtot[2][NW][2];
  __shared__ int32_t from[2 * kFields];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x < kNBuckets) from[threadIdx.x] = base[threadIdx.x * A.tiles + blockIdx.x];
  for (int s = 0; s < A.steps; ++s) {
    const long long i = ((long long)blockIdx.x * A.steps + s) * kOrderThreads + threadIdx.x;
    int32_t face[7];
    int bucket[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) bucket[k] = -1;
    Packed2 p{{0, 0}};
    int n = 0;
    faces_of_cell(A, i, [&](long long F) {
      const int b = face_bucket(F, A.M, A.nrows, A.tmpl);
      p.add(b);
#pragma unroll
      for (int k = 0; k < 7; ++k)
        if (k == n) {
          face[k] = (int32_t)F;
          bucket[k] = b;
        }
      ++n;
    });
    Packed2 q = p;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long u = __shfl_up(q.w[0], o, 64), v = __shfl_up(q.w[1], o, 64);
      if (lane >= o) {
        q.w[0] += u;
        q.w[1] += v;
      }
    }
    if (lane == 63) {
      wtot[s & 1][wave][0] = q.w[0];
      wtot[s & 1][wave][1] = q.w[1];
    }
    __syncthreads();
    Packed2 before{{q.w[0] - p.w[0], q.w[1] - p.w[1]}}, total{{0, 0}};
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const unsigned long long u = wtot[s & 1][k][0], v = wtot[s & 1][k][1];
      if (k < wave) {
        before.w[0] += u;
        before.w[1] += v;
      }
      total.w[0] += u;
      total.w[1] += v;
    }
#pragma unroll
    for (int k = 0; k < 7; ++k)
      if (bucket[k] >= 0) {
        perm[from[bucket[k]] + before.get(bucket[k])] = face[k];
        before.add(bucket[k]);
      }
    __syncthreads();
    if (threadIdx.x < kNBuckets) from[threadIdx.x] += total.get(threadIdx.x);
  }
}

// A workgroup takes one step of 256 cells, more where that would leave the single workgroup
// of the scan too much to do (beyond 2048 tiles, 20 counts per thread).
static int order_steps(long long cells) { return (int)((cells + kOrderThreads * 2048LL - 1) / (kOrderThreads * 2048LL)); }

int order_tiles(long long cells) {
  const long long step = (long long)kOrderThreads * order_steps(cells);
  return (int)((cells + step - 1) / step);
}

static OrderArgs order_args(const Work& w, int M, const int32_t* tmpl) {
  const long long cells = w.G * w.dims.ncell;
  return OrderArgs{w.dims,  w.G,      M,      order_steps(cells), order_tiles(cells), w.face_id,
                   w.eb_id, w.counts, w.offs, w.nrows,            tmpl};
}

int count_buckets(const Work& w, int M, const int32_t* tmpl, long long n_face, int64_t* row_ptr, hipStream_t st) {
  const OrderArgs A = order_args(w, M, tmpl);
  hipLaunchKernelGGL(k_order_count, dim3(A.tiles), dim3(kOrderThreads), 0, st, A, w.order_hist,
                     w.order_hist + kNBuckets * A.tiles);
  hipLaunchKernelGGL(k_order_scan, dim3(1), dim3(1024), 0, st, A.tiles, w.order_hist,
                     w.order_hist + kNBuckets * A.tiles, w.bins, n_face, row_ptr);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

int order_faces(const Work& w, int M, const int32_t* tmpl, hipStream_t st) {
  const OrderArgs A = order_args(w, M, tmpl);
  hipLaunchKernelGGL(k_order_write, dim3(A.tiles), dim3(kOrderThreads), 0, st, A, w.order_hist, w.perm);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

}  // namespace cutcell
