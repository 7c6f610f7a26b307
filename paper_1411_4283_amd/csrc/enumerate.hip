// Enumeration of volumes, boundary faces and flux faces (Sec. 2.1), path-radius
// neighbour rows (Sec. 2.4) and template faces.
#include "kernels.hpp"
#include "scan.hpp"

namespace cutcell {

__global__ void k_fill_i32(int32_t* p, long long n, int32_t v) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_f64(double* p, long long n, double v) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// row counts of an existing CSR, for binning the faces again (the adjoint)
__global__ void k_rows_per_face(long long n_face, const int64_t* __restrict__ row_ptr, int32_t* __restrict__ nrows) {
  long long f = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (f < n_face) {
    const int64_t n = row_ptr[f + 1] - row_ptr[f];
    nrows[f] = (n < 0 || n > (int64_t)kMaxRows) ? kMaxRows + 1 : (int32_t)n;
  }
}

static inline unsigned blocks_for(long long n, int t) { return (unsigned)((n + t - 1) / t); }

// lattice face lf (in the concatenated lattice) -> direction and coordinates
__device__ __forceinline__ int lattice_dir(const GridDims& g, long long lf) {
  return (lf >= g.foff[1]) + (lf >= g.foff[2]);
}

// (32-bit arithmetic: a geometry's lattice has fewer than 2^31 faces, checked on entry)
__device__ __forceinline__ void lattice_coords(const GridDims& g, int d, long long lf, int* j) {
  face_coords(g, d, (int)(lf - g.foff[d]), j);
}

__device__ __forceinline__ long long lattice_index(const GridDims& g, int d, const int* j) {
  int m0 = g.n[0] + (d == 0), m1 = g.n[1] + (d == 1);
  return g.foff[d] + j[0] + (long long)m0 * (j[1] + (long long)m1 * j[2]);
}

__device__ __forceinline__ long long cell_index(const GridDims& g, const int* i) {
  return i[0] + (long long)g.n[0] * (i[1] + (long long)g.n[1] * i[2]);
}

// box slot s (cells next to the box boundary, grouped by (d, side), ascending cell index
// inside a group) -> direction, side and the box face's lattice index
__device__ __forceinline__ long long box_slot_face(const GridDims& g, long long s, int* dd, int* side) {
  int k = 0;
  while (k < 5 && s >= g.boxoff[k + 1]) ++k;
  const int d = k / 2, sd = k % 2;
  long long t = s - g.boxoff[k];
  int a = (d == 0) ? 1 : 0;           // the two other directions, ascending
  int b = (d == 2) ? 1 : 2;
  int i[3] = {0, 0, 0};
  i[a] = (int)(t % g.n[a]);
  i[b] = (int)(t / g.n[a]);
  i[d] = sd ? g.n[d] : 0;             // lattice coordinate of the boundary face
  *dd = d;
  *side = sd;
  return lattice_index(g, d, i);
}

// Flags of cells, box slots and lattice faces; eb_id and box_id start at -1.  Past L, the EB
// cells are checked before anything indexes with them: strictly ascending, inside the grid
// and in volumes.
__global__ void k_enum_flags(GridDims g, int M, int Mf, const GeomPtrs* __restrict__ geoms, int32_t* flags,
                             long long L, int32_t* eb_id, int32_t* box_id, int32_t* bad) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int gi = blockIdx.y;
  const GeomPtrs gp = geoms[gi];
  if (i >= L) {
    const long long e = i - L;
    if (e >= gp.n_eb) return;
    const int32_t c = gp.eb_cell[e];
    bool ok = c >= 0 && c < g.ncell;
    if (ok && e > 0) ok = gp.eb_cell[e - 1] < c;
    if (ok) ok = gp.vol_mom[(long long)c * M] > 0.0;
    if (!ok) atomicOr(bad, 1);
    return;
  }
  int32_t f = 0;
  if (i < g.ncell) {
    f = gp.vol_mom[i * M] > 0.0;
    eb_id[gi * g.ncell + i] = -1;
  } else if (i < g.ncell + g.nboxslot) {
    int d, side;
    long long lf = box_slot_face(g, i - g.ncell, &d, &side);
    f = gp.face_mom[d][(lf - g.foff[d]) * Mf] > 0.0;
  } else {
    long long lf = i - g.ncell - g.nboxslot;
    int d = lattice_dir(g, lf);
    f = gp.face_mom[d][(lf - g.foff[d]) * Mf] > 0.0;
    box_id[gi * g.NF + lf] = -1;
  }
  flags[gi * L + i] = f;
}

__global__ void k_enum_counts(GridDims g, int G, long long L, const int32_t* __restrict__ excl,
                              const int32_t* __restrict__ seg_total, const GeomPtrs* __restrict__ geoms,
                              int64_t* counts, int64_t* offs) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int64_t* phi_off = offs;
  int64_t* vol_off = offs + (G + 1);
  int64_t* face_off = offs + 2 * (G + 1);
  phi_off[0] = vol_off[0] = face_off[0] = 0;
  for (int gi = 0; gi < G; ++gi) {
    const int32_t* e = excl + gi * L;
    int64_t n_vol = e[g.ncell];
    int64_t n_box = (int64_t)e[g.ncell + g.nboxslot] - e[g.ncell];
    int64_t n_gface = (int64_t)seg_total[gi] - e[g.ncell + g.nboxslot];
    int64_t n_eb = geoms[gi].n_eb;
    counts[4 * gi + 0] = n_vol;
    counts[4 * gi + 1] = n_eb;
    counts[4 * gi + 2] = n_box;
    counts[4 * gi + 3] = n_gface;
    phi_off[gi + 1] = phi_off[gi] + n_vol + n_eb + n_box;
    vol_off[gi + 1] = vol_off[gi] + n_vol;
    face_off[gi + 1] = face_off[gi] + n_gface + n_eb;
  }
}

__global__ void k_enum_maps(GridDims g, int G, long long L, const GeomPtrs* __restrict__ geoms,
                            const int32_t* __restrict__ flags, const int32_t* __restrict__ excl,
                            const int64_t* __restrict__ counts, const int64_t* __restrict__ offs, int32_t* vol_id,
                            int32_t* eb_id, int32_t* vol_cell, int32_t* box_id, int32_t* box_lf, int32_t* face_id,
                            int32_t* fcode, int32_t* fref) {
  long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  const int gi = blockIdx.y;
  if (i >= L) {   // EB faces
    const long long e = i - L;
    const GeomPtrs gp = geoms[gi];
    if (e >= gp.n_eb) return;
    const int32_t c = gp.eb_cell[e];
    if (c < 0 || c >= g.ncell) return;   // rejected by the argument check; never index with it
    eb_id[gi * g.ncell + c] = (int32_t)e;
    const long long F = offs[2 * (G + 1) + gi] + counts[4 * gi + 3] + e;
    fcode[F] = face_code(gi, 1, 0);
    fref[F] = (int32_t)e;
    return;
  }
  const int32_t f = flags[gi * L + i];
  const int32_t e = excl[gi * L + i];
  if (i < g.ncell) {
    vol_id[gi * g.ncell + i] = f ? e : -1;
    if (f) vol_cell[gi * g.ncell + e] = (int32_t)i;
  } else if (i < g.ncell + g.nboxslot) {
    if (!f) return;
    int d, side;
    long long lf = box_slot_face(g, i - g.ncell, &d, &side);
    int32_t b = e - excl[gi * L + g.ncell];
    box_id[gi * g.NF + lf] = b;
    box_lf[gi * g.nboxslot + b] = (int32_t)lf;
  } else {
    long long lf = i - g.ncell - g.nboxslot;
    int32_t loc = f ? e - excl[gi * L + g.ncell + g.nboxslot] : -1;
    face_id[gi * g.NF + lf] = loc;
    if (f) {
      long long F = offs[2 * (G + 1) + gi] + loc;
      fcode[F] = face_code(gi, 0, lattice_dir(g, lf));
      fref[F] = (int32_t)lf;
    }
  }
}

// one byte per cell for the neighbour search: bit 0 volume, bit 1 + 2d + s the grid face
// on side s (0 low, 1 high) of direction d has alpha > 0, bit 7 the cell has an EB face
__global__ void k_cellinfo(GridDims g, const int32_t* __restrict__ vol_id, const int32_t* __restrict__ eb_id,
                           const int32_t* __restrict__ face_id, uint8_t* __restrict__ info) {
  const int gi = blockIdx.y;
  long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (c >= g.ncell) return;
  const long long o = (long long)gi * g.ncell + c;
  unsigned v = vol_id[o] >= 0 ? 1u : 0u;
  if (v) {
    int x[3];
    cell_coords(g, (int)c, x);
    for (int d = 0; d < g.D; ++d)
      for (int s = 0; s < 2; ++s) {
        int j[3] = {x[0], x[1], x[2]};
        j[d] += s;
        if (face_id[(long long)gi * g.NF + lattice_index(g, d, j)] >= 0) v |= 1u << (1 + 2 * d + s);
      }
    if (eb_id[o] >= 0) v |= 0x80u;
  }
  info[o] = (uint8_t)v;
}

// Regular cells for the neighbour fast path: a volume without an EB face whose 2D faces are
// all flux faces and which does not touch the box boundary; reg(c) = 1 iff every cell within
// L1 distance R of c is one.  For such cells the path-distance ball of radius R is the L1 ball
// and touches no EB or box face.  A line of the ball is a run of at most 2R + 1 bytes of
// cellinfo, read eight at a time.  Bound by the latency of one round of loads; 64^3, R = 3:
// 17 us as a pass over the cells and R erosions, under 7 us like this.
template <int D, int R>
__global__ __launch_bounds__(256) void k_ball_regular(GridDims g, const uint8_t* __restrict__ info,
                                                      uint8_t* __restrict__ reg) {
  const int gi = blockIdx.y;
  const long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (c >= g.ncell) return;
  const long long o = (long long)gi * g.ncell + c;
  int x[3];
  cell_coords(g, (int)c, x);
  bool r = true;
#pragma unroll
  for (int d = 0; d < D; ++d) r = r && x[d] >= R + 1 && x[d] <= g.n[d] - 2 - R;
  if (r) {
    constexpr unsigned full = (1u << (1 + 2 * D)) - 1u;   // volume bit and all open-face bits
    constexpr unsigned long long all = 0x0101010101010101ULL * full;
    const long long line = g.n[0], plane = (long long)g.n[0] * g.n[1];
    unsigned long long differ = 0;
#pragma unroll
    for (int z = (D == 3 ? -R : 0); z <= (D == 3 ? R : 0); ++z)
#pragma unroll
      for (int y = -R; y <= R; ++y) {
        const int k = R - (y < 0 ? -y : y) - (z < 0 ? -z : z);
        if (k < 0) continue;
        const uint8_t* p = info + o + z * plane + y * line - k;
        unsigned long long v;
        __builtin_memcpy(&v, p, 8);
        const int bytes = 2 * k + 1;
        differ |= (v ^ all) & (bytes >= 8 ? ~0ULL : (1ULL << (8 * bytes)) - 1);
        if (bytes > 8) differ |= p[8] ^ full;
      }
    r = differ == 0;
  }
  reg[o] = r ? 1 : 0;
}

// out(c) = in(c) and in of its 2D neighbours: R of these keep the cells whose L1 ball of
// radius R is in the set
__global__ void k_erode(GridDims g, const uint8_t* __restrict__ in, uint8_t* __restrict__ out) {
  const int gi = blockIdx.y;
  long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (c >= g.ncell) return;
  const long long o = (long long)gi * g.ncell + c;
  bool r = in[o] != 0;   // a regular cell is interior, so its neighbours exist
  if (r) {
    const long long st[3] = {1, g.n[0], (long long)g.n[0] * g.n[1]};
    for (int d = 0; d < g.D; ++d) r = r && in[o - st[d]] && in[o + st[d]];
  }
  out[o] = r ? 1 : 0;
}

int enumerate_batch(const Work& w, const cutcell_opts& o, long long max_eb, hipStream_t st) {
  const GridDims& g = w.dims;
  const int D = o.dim, Q = o.order;
  const int M = binom(Q + D, D), Mf = binom(Q + D - 1, D - 1);
  const int T = 256;
  const dim3 all(blocks_for(w.L + max_eb, T), w.G), cells(blocks_for(g.ncell, T), w.G);
  hipLaunchKernelGGL(k_enum_flags, all, dim3(T), 0, st, g, M, Mf, w.geoms, w.flags, w.L, w.eb_id, w.box_id,
                     w.flagged + 1);
  int rc = exclusive_scan<int32_t, int32_t>(w.flags, w.L, w.L, w.G, w.excl, w.L, w.seg_total, w.scan_tmp, st);
  if (rc) return rc;
  hipLaunchKernelGGL(k_enum_counts, dim3(1), dim3(64), 0, st, g, w.G, w.L, w.excl, w.seg_total, w.geoms, w.counts,
                     w.offs);
  hipLaunchKernelGGL(k_enum_maps, all, dim3(T), 0, st, g, w.G, w.L, w.geoms, w.flags, w.excl, w.counts, w.offs,
                     w.vol_id, w.eb_id, w.vol_cell, w.box_id, w.box_lf, w.face_id, w.fcode, w.fref);
  hipLaunchKernelGGL(k_cellinfo, cells, dim3(T), 0, st, g, w.vol_id, w.eb_id, w.face_id, w.cellinfo);
#define CC_BR(DD, RR) \
  if (D == DD && o.path_radius == RR) \
    hipLaunchKernelGGL((k_ball_regular<DD, RR>), cells, dim3(T), 0, st, g, w.cellinfo, w.ballreg);
  CC_BR(2, 1) CC_BR(2, 2) CC_BR(2, 3) CC_BR(2, 4) CC_BR(3, 1) CC_BR(3, 2) CC_BR(3, 3) CC_BR(3, 4)
#undef CC_BR
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

// ---------------------------------------------------------------------------------------
// neighbours: breadth-first search by path distance inside a window around the face
//
// A lane holds lines of window cells along x as bit masks (volumes, open faces per side, EB
// faces), read as the line's bytes of cellinfo in one or two loads.  A step of the search is
// then a handful of bit operations on the lane's mask and its four neighbours' masks (y and
// z, through shared memory).  A window has (2R + 2)(2R + 1) lines in 3D and 2R + 2 in 2D, so
// 16, 32 or 64 lanes take a face; a wave takes a chunk of consecutive faces, answers the
// ones between ball-regular cells from the fixed offsets, and searches the others in turn.
// The fill pass searches again: that is cheaper than keeping the masks.  It is bound by the
// latency of the search's dependent steps.  64^3, path radius 3 (724k faces, half of them
// searched): count and fill 0.76 ms; with one cell per lane and step, a wave per face and the
// masks kept for the fill, 1.69 and 0.96 ms.

template <int D, int R>
struct Win {
  static constexpr int EN = 2 * R + 2;                       // extent along the face normal
  static constexpr int ET = 2 * R + 1;                       // transverse extent
  static constexpr int L = D == 3 ? EN * ET : EN;            // lines along x, at most
  static constexpr int LPF = L <= 16 ? 16 : (L <= 32 ? 32 : 64);   // lanes per face
  static constexpr int KL = (L + LPF - 1) / LPF;             // lines per lane
  static constexpr int FPW = 64 / LPF;                       // faces of a wave at a time
};

// Rows of a face between two ball-regular cells a (low) and a + e_d: the union of the L1
// balls of radius R around them, as offsets from a in ascending cell-index order (z, y, x).
template <int D, int R>
struct RegularRows {
  static constexpr int kMax = 2 * (2 * R + 2) * (2 * R + 1) * (D == 3 ? 2 * R + 1 : 1);
  int n = 0;
  int8_t off[3][kMax][3] = {};
  constexpr RegularRows() {
    for (int dn = 0; dn < D; ++dn) {
      int cnt = 0;
      const int zlo = (D == 3) ? -R : 0, zhi = (D == 3) ? R + (dn == 2) : 0;
      for (int z = zlo; z <= zhi; ++z)
        for (int y = -R; y <= R + (dn == 1); ++y)
          for (int x = -R; x <= R + (dn == 0); ++x) {
            const int o[3] = {x, y, z};
            int l0 = 0, l1 = 0;
            for (int ax = 0; ax < 3; ++ax) {
              const int v = o[ax], w = o[ax] - (ax == dn);
              l0 += v < 0 ? -v : v;
              l1 += w < 0 ? -w : w;
            }
            if (l0 <= R || l1 <= R) {
              off[dn][cnt][0] = (int8_t)x;
              off[dn][cnt][1] = (int8_t)y;
              off[dn][cnt][2] = (int8_t)z;
              ++cnt;
            }
          }
      n = cnt;
    }
  }
};

template <int D, int R>
inline constexpr RegularRows<D, R> kRegularRows{};

// bit i of the result: bit `b` of byte i of v
__device__ __forceinline__ unsigned byte_plane(uint2 v, int b) {
  const unsigned lo = (v.x >> b) & 0x01010101u, hi = (v.y >> b) & 0x01010101u;
  return __builtin_amdgcn_udot4(hi, 0x80402010u, __builtin_amdgcn_udot4(lo, 0x08040201u, 0u, false), false);
}

// sum of v over the lane's group of W lanes, and over the lanes of it before this one
template <int W>
__device__ __forceinline__ int group_sum(int v) {
#pragma unroll
  for (int o = W / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, W);
  return v;
}
template <int W>
__device__ __forceinline__ int group_before(int v) {
  const int l = threadIdx.x & (W - 1);
  int s = v;
#pragma unroll
  for (int o = 1; o < W; o <<= 1) {
    const int t = __shfl_up(s, o, W);
    if (l >= o) s += t;
  }
  return s - v;
}

struct NeighbourArgs {
  GridDims g;
  long long n_face;
  int chunk;                     // faces per wave, at most 64
  const int32_t* fcode;
  const int32_t* fref;
  const GeomPtrs* geoms;
  const int32_t* vol_id;
  const int32_t* eb_id;
  const int32_t* box_id;
  const int64_t* counts;
  const int64_t* offs;
  const uint8_t* cellinfo;       // readable kInfoPad bytes before and after
  const uint8_t* ballreg;
  int32_t* nrows;
  const int64_t* row_ptr;
  int32_t* col;
  int neumann;
};

template <int D, int R, bool FILL>
__global__ __launch_bounds__(64) void k_neighbours(NeighbourArgs A) {
  using W = Win<D, R>;
  constexpr int LPF = W::LPF, KL = W::KL, FPW = W::FPW;
  static_assert(W::EN <= 16 && W::EN <= kInfoPad, "a line's mask and its loads");
  __shared__ unsigned cur[FPW][KL * LPF];
  __shared__ int32_t stage[FILL ? FPW : 1][FILL ? kMaxRows : 1];
  __shared__ int8_t list[64];
  const GridDims& g = A.g;
  const int lane = threadIdx.x;
  const long long F0 = (long long)blockIdx.x * A.chunk;
  const long long st1 = g.n[0], st2 = (long long)g.n[0] * g.n[1];

  // ---- the chunk's faces, one per lane ------------------------------------------------------
  const bool have = lane < A.chunk && F0 + lane < A.n_face;
  int32_t code = 0, ref = 0;
  long long low = 0;               // regular faces: the low cell
  bool regular = false, search = false;
  int64_t pos0 = 0;
  if (have) {
    code = A.fcode[F0 + lane];
    ref = A.fref[F0 + lane];
    if (FILL) pos0 = A.row_ptr[F0 + lane];
    const int gi = code >> 4, kind = (code >> 2) & 3, dn = code & 3;
    search = true;
    if (kind == 1 && A.neumann) {
      // a Neumann EB face's flux is its data: one row, its own Phi entry
      if (!FILL) A.nrows[F0 + lane] = 1;
      else A.col[pos0] = (int32_t)(A.offs[gi] + A.counts[4 * gi + 0] + ref);
      search = false;
    } else if (kind == 0) {
      // a grid face between two ball-regular cells has the fixed L1-ball rows
      int j[3];
      lattice_coords(g, dn, ref, j);
      if (j[dn] >= 1 && j[dn] <= g.n[dn] - 1) {
        const long long b = cell_index(g, j);
        const uint8_t* reg = A.ballreg + (long long)gi * g.ncell;
        low = b - (dn == 0 ? 1 : (dn == 1 ? st1 : st2));
        regular = reg[low] && reg[b];
        search = !regular;
      }
    }
  }
  constexpr auto& P = kRegularRows<D, R>;
  if (!FILL) {
    if (regular) A.nrows[F0 + lane] = P.n;
  } else {
    // the wave writes one regular face at a time, an entry (or more) per lane
    constexpr int E = (P.n + 63) / 64;
    int off[D][E];
#pragma unroll
    for (int dn = 0; dn < D; ++dn)
#pragma unroll
      for (int i = 0; i < E; ++i) {
        const int k = lane + 64 * i < P.n ? lane + 64 * i : 0;
        off[dn][i] = (int)(P.off[dn][k][0] + st1 * P.off[dn][k][1] + st2 * P.off[dn][k][2]);
      }
    for (unsigned long long m = __ballot(regular); m != 0; m &= m - 1) {
      const int l = __ffsll((long long)m) - 1;
      const int cd = __builtin_amdgcn_readlane(code, l), dn = cd & 3, gi = cd >> 4;
      const long long a = __builtin_amdgcn_readlane((int)low, l);   // fewer than 2^31 cells
      const long long at = readlane_i64(pos0, l);
      const int32_t* vid = A.vol_id + (long long)gi * g.ncell + a;
      const int32_t phi0 = (int32_t)A.offs[gi];
#pragma unroll
      for (int i = 0; i < E; ++i) {
        int o = off[0][i];
        if (dn == 1) o = off[1][i];
        if (D == 3 && dn == 2) o = off[D - 1][i];
        if (lane + 64 * i < P.n) A.col[at + lane + 64 * i] = phi0 + vid[o];
      }
    }
  }

  // ---- the others, FPW at a time ---------------------------------------------------------------
  const unsigned long long todo = __ballot(search);
  const int ntodo = __popcll(todo);
  if (search) list[__popcll(todo & lanes_below(lane))] = (int8_t)lane;
  __syncthreads();
  const int grp = lane / LPF, gl = lane & (LPF - 1);
  for (int t0 = 0; t0 < ntodo; t0 += FPW) {
    const bool on = t0 + grp < ntodo;
    const int src = list[on ? t0 + grp : 0];
    const int cd = __shfl(code, src), rf = __shfl(ref, src);
    const int gi = cd >> 4, kind = (cd >> 2) & 3, dn = cd & 3;
    const int nrm = kind == 0 ? dn : 0;
    // window origin and extents; the adjacent cells sit at normal index R (and R + 1)
    int org[3] = {0, 0, 0}, ext[3] = {1, 1, 1};
    if (kind == 0) {
      int j[3];
      lattice_coords(g, dn, rf, j);
#pragma unroll
      for (int ax = 0; ax < D; ++ax) org[ax] = j[ax] - R - (ax == dn);
    } else {
      int x[3];
      cell_coords(g, A.geoms[gi].eb_cell[rf], x);
#pragma unroll
      for (int ax = 0; ax < D; ++ax) org[ax] = x[ax] - R;
    }
#pragma unroll
    for (int ax = 0; ax < D; ++ax) ext[ax] = ax == nrm ? W::EN : W::ET;
    const int nl = ext[1] * ext[2];
    const uint8_t* inf = A.cellinfo + (long long)gi * g.ncell;
    // bits of the line inside the box
    const int xlo = org[0] < 0 ? -org[0] : 0, xhi = min(ext[0], g.n[0] - org[0]);
    const unsigned xin = ((1u << xhi) - 1u) & ~((1u << xlo) - 1u);
    unsigned vol[KL], ol[KL][D], oh[KL][D], eb[KL], S[KL];
    int wy[KL], wz[KL];
    long long line[KL];
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      const int li = gl + LPF * k;
      wy[k] = li;
      wz[k] = 0;
      if (D == 3) {   // compile-time divisors: the long extent is along nrm
        wy[k] = nrm == 1 ? li % W::EN : li % W::ET;
        wz[k] = nrm == 1 ? li / W::EN : li / W::ET;
      }
      const int y = org[1] + wy[k], z = org[2] + wz[k];
      const bool in = on && li < nl && y >= 0 && y < g.n[1] && z >= 0 && z < g.n[2];
      line[k] = st2 * z + st1 * y + org[0];
      vol[k] = eb[k] = S[k] = 0;
#pragma unroll
      for (int ax = 0; ax < D; ++ax) ol[k][ax] = oh[k][ax] = 0;
      if (in) {
        uint2 v, w;
        __builtin_memcpy(&v, inf + line[k], 8);
        if (W::EN > 8) __builtin_memcpy(&w, inf + line[k] + 8, 8);
        auto plane = [&](int b) {
          unsigned m = byte_plane(v, b);
          if (W::EN > 8) m |= byte_plane(w, b) << 8;
          return m & xin;
        };
        vol[k] = plane(0);
        eb[k] = plane(7);
#pragma unroll
        for (int ax = 0; ax < D; ++ax) {
          ol[k][ax] = plane(1 + 2 * ax);
          oh[k][ax] = plane(2 + 2 * ax);
        }
        // the face's adjacent cells
        unsigned m = 0;
        if (nrm == 0) {
          if (wy[k] == R && (D == 2 || wz[k] == R)) m = kind == 0 ? 3u << R : 1u << R;
        } else if (nrm == 1) {
          if ((wy[k] == R || wy[k] == R + 1) && (D == 2 || wz[k] == R)) m = 1u << R;
        } else {
          if (wy[k] == R && (wz[k] == R || wz[k] == R + 1)) m = 1u << R;
        }
        S[k] = m & vol[k];
      }
    }
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
      __syncthreads();
#pragma unroll
      for (int k = 0; k < KL; ++k) cur[grp][gl + LPF * k] = S[k];
      __syncthreads();
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        // a cell is reached through its own open face from a reached neighbour in the window
        const int li = gl + LPF * k;
        unsigned m = ((S[k] << 1) & ol[k][0]) | ((S[k] >> 1) & oh[k][0]);
        if (wy[k] > 0 && li < nl) m |= cur[grp][li - 1] & ol[k][1];
        if (wy[k] + 1 < ext[1] && li < nl) m |= cur[grp][li + 1] & oh[k][1];
        if (D == 3) {
          if (wz[k] > 0 && li < nl) m |= cur[grp][li - ext[1]] & ol[k][D - 1];
          if (wz[k] + 1 < ext[2] && li < nl) m |= cur[grp][li + ext[1]] & oh[k][D - 1];
        }
        S[k] |= m;
      }
    }
    // box faces of the reached cells, by direction and side
    auto box_mask = [&](int k, int ax, int s) -> unsigned {
      const unsigned m = S[k] & (s ? oh[k][ax] : ol[k][ax]);
      const int at = s ? g.n[ax] - 1 : 0;
      if (ax == 0) {
        const int b = at - org[0];
        return (b >= 0 && b < ext[0]) ? m & (1u << b) : 0u;
      }
      return (ax == 1 ? org[1] + wy[k] : org[2] + wz[k]) == at ? m : 0u;
    };
    if (!FILL) {
      int c = 0;
#pragma unroll
      for (int k = 0; k < KL; ++k) {
        c += __popc(S[k]) + __popc(S[k] & eb[k]);
#pragma unroll
        for (int ax = 0; ax < D; ++ax) c += __popc(box_mask(k, ax, 0)) + __popc(box_mask(k, ax, 1));
      }
      c = group_sum<LPF>(c);
      if (on && gl == 0) A.nrows[F0 + src] = c;
      continue;
    }
    // rows in ascending Phi order: volumes, EB faces, box faces by (d, side).  The ids of a
    // line's volumes (and of its EB faces) are consecutive, so one load gives them all.
    const int64_t* cnt = A.counts + 4 * gi;
    const int32_t phi0 = (int32_t)A.offs[gi];
    const int32_t* vid = A.vol_id + (long long)gi * g.ncell;
    const int32_t* eid = A.eb_id + (long long)gi * g.ncell;
    const int32_t* bid = A.box_id + (long long)gi * g.NF;
    int n = 0;
    auto put = [&](int k, unsigned m, auto&& entry) {
      int p = n + group_before<LPF>(__popc(m));
      n += group_sum<LPF>(__popc(m));
      for (; m != 0; m &= m - 1) {
        if (p < kMaxRows) stage[FILL ? grp : 0][FILL ? p : 0] = entry(__ffs(m) - 1);
        ++p;
      }
    };
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      const int32_t v0 = vol[k] ? phi0 + vid[line[k] + __ffs(vol[k]) - 1] : 0;
      put(k, S[k], [&](int b) { return v0 + __popc(vol[k] & ((1u << b) - 1u)); });
    }
#pragma unroll
    for (int k = 0; k < KL; ++k) {
      const unsigned m = S[k] & eb[k];
      if (!__any(m != 0)) continue;
      const int32_t e0 = m ? phi0 + (int32_t)cnt[0] + eid[line[k] + __ffs(eb[k]) - 1] : 0;
      put(k, m, [&](int b) { return e0 + __popc(eb[k] & ((1u << b) - 1u)); });
    }
#pragma unroll
    for (int ax = 0; ax < D; ++ax)
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int k = 0; k < KL; ++k) {
          const unsigned m = box_mask(k, ax, s);
          if (!__any(m != 0)) continue;
          put(k, m, [&](int b) {
            int j[3] = {org[0] + b, org[1] + wy[k], org[2] + wz[k]};
            j[ax] += s;
            return phi0 + (int32_t)(cnt[0] + cnt[1]) + bid[lattice_index(g, ax, j)];
          });
        }
    __syncthreads();
    const long long at = __shfl(pos0, src);   // by every lane: one that is off gives nothing away
    if (on) {
      for (int i = gl; i < n; i += LPF) A.col[at + i] = stage[FILL ? grp : 0][FILL ? i : 0];
    }
    __syncthreads();
  }
}

template <int D, int R>
static void launch_neighbours(const Work& w, long long n_face, const int64_t* row_ptr, int32_t* col, bool fill,
                              int neumann, hipStream_t st) {
  NeighbourArgs A{w.dims, n_face, 64, w.fcode, w.fref, w.geoms, w.vol_id, w.eb_id, w.box_id, w.counts, w.offs,
                  w.cellinfo, w.ballreg, w.nrows, row_ptr, col, neumann};
  // a chunk of 64 faces hides most latency; smaller chunks where that would leave the chip
  // short of waves (8 per SIMD)
  while (A.chunk > Win<D, R>::FPW && n_face / A.chunk < 8192) A.chunk /= 2;
  const dim3 grid((unsigned)((n_face + A.chunk - 1) / A.chunk)), block(64);
  if (fill) hipLaunchKernelGGL((k_neighbours<D, R, true>), grid, block, 0, st, A);
  else hipLaunchKernelGGL((k_neighbours<D, R, false>), grid, block, 0, st, A);
}

int neighbour_rows(const Work& w, const cutcell_opts& o, long long n_face, const int64_t* row_ptr, int32_t* col,
                   bool fill, hipStream_t st) {
  if (n_face <= 0) return CUTCELL_OK;
  const int D = o.dim, R = o.path_radius;
  const int neumann = o.eb_bc == CUTCELL_BC_NEUMANN;
#define CC_NB(DD, RR) \
  if (D == DD && R == RR) { launch_neighbours<DD, RR>(w, n_face, row_ptr, col, fill, neumann, st); }
  CC_NB(2, 1) CC_NB(2, 2) CC_NB(2, 3) CC_NB(2, 4) CC_NB(3, 1) CC_NB(3, 2) CC_NB(3, 3) CC_NB(3, 4)
#undef CC_NB
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

// ---------------------------------------------------------------------------------------
// volume -> faces table and the 1/|V| scale of the divergence

__global__ void k_volume_tables(GridDims g, int G, int M, double hD, const GeomPtrs* __restrict__ geoms,
                                const int32_t* __restrict__ vol_id, const int32_t* __restrict__ eb_id,
                                const int32_t* __restrict__ face_id, const int64_t* __restrict__ counts,
                                const int64_t* __restrict__ offs, int32_t* vol_face, double* vol_scale,
                                int64_t* phi_off, int64_t* vol_off, int64_t* face_off) {
  const int gi = blockIdx.y;
  long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x <= (gi == 0 ? 1 : 0)) {   // offsets of geometry gi + 1, and of geometry 0
    const int i = threadIdx.x == 0 ? gi + 1 : 0;
    phi_off[i] = offs[i];
    vol_off[i] = offs[(G + 1) + i];
    face_off[i] = offs[2 * (G + 1) + i];
  }
  if (c >= g.ncell) return;
  const int32_t v = vol_id[gi * g.ncell + c];
  if (v < 0) return;
  const int D = g.D;
  const long long V = offs[(G + 1) + gi] + v;
  const long long F0 = offs[2 * (G + 1) + gi];
  int x[3];
  cell_coords(g, (int)c, x);
  const int S = 2 * D + 1;
  for (int d = 0; d < D; ++d)
    for (int s = 0; s < 2; ++s) {
      int j[3] = {x[0], x[1], x[2]};
      j[d] += s;
      int32_t f = face_id[gi * g.NF + lattice_index(g, d, j)];
      vol_face[V * S + 2 * d + s] = (f >= 0) ? (int32_t)(F0 + f) : -1;
    }
  int32_t e = eb_id[gi * g.ncell + c];
  vol_face[V * S + 2 * D] = (e >= 0) ? (int32_t)(F0 + counts[4 * gi + 3] + e) : -1;
  vol_scale[V] = 1.0 / (geoms[gi].vol_mom[c * M] * hD);
}

int volume_tables(const Work& w, const cutcell_opts& o, int32_t* vol_face, double* vol_scale, int64_t* phi_off,
                  int64_t* vol_off, int64_t* face_off, hipStream_t st) {
  const int M = binom(o.order + o.dim, o.dim);
  double hD = 1.0;
  for (int d = 0; d < o.dim; ++d) hD *= o.h;
  hipLaunchKernelGGL(k_volume_tables, dim3(blocks_for(w.dims.ncell, 256), w.G), dim3(256), 0, st, w.dims, w.G, M, hD,
                     w.geoms, w.vol_id, w.eb_id, w.face_id, w.counts, w.offs, vol_face, vol_scale, phi_off, vol_off,
                     face_off);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

int rows_per_face(const Work& w, long long n_face, const int64_t* row_ptr, hipStream_t st) {
  if (n_face > 0)
    hipLaunchKernelGGL(k_rows_per_face, dim3(blocks_for(n_face, 256)), dim3(256), 0, st, n_face, row_ptr, w.nrows);
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

// ---------------------------------------------------------------------------------------
// Template reuse.  A face between two cells whose every neighbour within the path radius
// is a plain interior volume has the fixed row pattern of the fast path above; if all of
// those cells and their faces also carry exactly the reference cell's moments, its system
// (rows about x0 -- the offsets are exact small half-integers --, weights and F) is bit
// for bit that of any other such face of the same direction, and so is its stencil.  One
// face per (geometry, direction) is solved; the others copy its values.

constexpr int32_t kNone = 0x7fffffff;

__global__ void k_ref_cell(GridDims g, const uint8_t* __restrict__ ballreg, int32_t* ref) {
  const int gi = blockIdx.y;
  const long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (c >= g.ncell) return;
  if (ballreg[(long long)gi * g.ncell + c]) atomicMin(&ref[gi], (int32_t)c);
}

__device__ __forceinline__ bool same_bits(const double* a, const double* b, int n) {
  bool s = true;
  for (int i = 0; i < n; ++i) s = s && (__double_as_longlong(a[i]) == __double_as_longlong(b[i]));
  return s;
}

// plain interior volume (as for ball regularity) whose volume moments and the moments of
// its 2D faces equal the reference cell's bit for bit
__global__ void k_canon0(GridDims g, int M, int Mf, const GeomPtrs* __restrict__ geoms,
                         const uint8_t* __restrict__ info, const int32_t* __restrict__ ref, uint8_t* __restrict__ out) {
  const int gi = blockIdx.y;
  const long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (c >= g.ncell) return;
  const long long o = (long long)gi * g.ncell + c;
  const unsigned full = (1u << (1 + 2 * g.D)) - 1u;
  bool r = info[o] == full;
  int x[3];
  cell_coords(g, (int)c, x);
  for (int d = 0; d < g.D; ++d) r = r && x[d] >= 1 && x[d] <= g.n[d] - 2;
  const int32_t rc = ref[gi];
  r = r && rc != kNone;
  if (r) {
    const GeomPtrs gp = geoms[gi];
    r = same_bits(gp.vol_mom + c * M, gp.vol_mom + (long long)rc * M, M);
    const int xr[3] = {(int)(rc % g.n[0]), (int)((rc / g.n[0]) % g.n[1]), (int)(rc / ((long long)g.n[0] * g.n[1]))};
    for (int d = 0; d < g.D && r; ++d)
      for (int s = 0; s < 2 && r; ++s) {
        int j[3] = {x[0], x[1], x[2]}, jr[3] = {xr[0], xr[1], xr[2]};
        j[d] += s;
        jr[d] += s;
        const long long lf = lattice_index(g, d, j) - g.foff[d], lr = lattice_index(g, d, jr) - g.foff[d];
        r = same_bits(gp.face_mom[d] + lf * Mf, gp.face_mom[d] + lr * Mf, Mf);
      }
  }
  out[o] = r ? 1 : 0;
}

// a grid face between two cells that are canonical out to the path radius
__device__ __forceinline__ bool template_face(const GridDims& g, const int32_t* fcode, const int32_t* fref,
                                             const uint8_t* canon, long long F, int* gi_out, int* dn_out) {
  const int32_t code = fcode[F];
  const int gi = code >> 4, kind = (code >> 2) & 3, dn = code & 3;
  *gi_out = gi;
  *dn_out = dn;
  if (kind != 0) return false;
  int j[3];
  lattice_coords(g, dn, fref[F], j);
  if (j[dn] < 1 || j[dn] > g.n[dn] - 1) return false;
  const long long b = cell_index(g, j);
  const long long st[3] = {1, g.n[0], (long long)g.n[0] * g.n[1]};
  const uint8_t* cn = canon + (long long)gi * g.ncell;
  return cn[b - st[dn]] && cn[b];
}

// The first template-able face of each (geometry, direction).  Faces of a wave are
// consecutive and nearly always of one (geometry, direction): the wave's lowest such lane
// stands for the lanes of its key (their minimum, faces ascending with the lane), and only
// lanes of another key add their own atomic -- one atomic per wave instead of one per
// face on three addresses per geometry.
__global__ void k_tmpl_pick(GridDims g, long long n_face, const int32_t* __restrict__ fcode,
                            const int32_t* __restrict__ fref, const uint8_t* __restrict__ canon, int32_t* tface) {
  const long long F = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  int gi = 0, dn = 0;
  const bool q = F < n_face && template_face(g, fcode, fref, canon, F, &gi, &dn);
  const unsigned long long m = __ballot(q);
  if (m == 0) return;
  const int lane = threadIdx.x & 63, leader = __ffsll((long long)m) - 1;
  const int key = 3 * gi + dn;
  const int lkey = __shfl(key, leader, 64);
  if (q && (lane == leader || key != lkey)) atomicMin(&tface[key], (int32_t)F);
}

__global__ void k_tmpl_assign(GridDims g, long long n_face, const int32_t* __restrict__ fcode,
                              const int32_t* __restrict__ fref, const uint8_t* __restrict__ canon,
                              const int32_t* __restrict__ tface, int32_t* __restrict__ tmpl) {
  const long long F = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (F >= n_face) return;
  int gi, dn;
  const bool q = template_face(g, fcode, fref, canon, F, &gi, &dn);
  const int32_t t = q ? tface[3 * gi + dn] : kNone;
  tmpl[F] = (q && t != (int32_t)F) ? t : -1;
}

int find_templates(const Work& w, const cutcell_opts& o, long long n_face, hipStream_t st) {
  const GridDims& g = w.dims;
  const int D = o.dim, Q = o.order;
  const int M = binom(Q + D, D), Mf = binom(Q + D - 1, D - 1);
  const int T = 256;
  hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, st, w.ref_cell, (long long)w.G, kNone);
  hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(3LL * w.G, 64)), dim3(64), 0, st, w.tface, 3LL * w.G, kNone);
  hipLaunchKernelGGL(k_ref_cell, dim3(blocks_for(g.ncell, T), w.G), dim3(T), 0, st, g, w.ballreg, w.ref_cell);
  // R erosions must leave the result in w.canon (ping-pong with ballreg_tmp)
  uint8_t* bufs[2] = {w.canon, w.ballreg_tmp};
  int cur = (o.path_radius % 2 == 0) ? 0 : 1;
  hipLaunchKernelGGL(k_canon0, dim3(blocks_for(g.ncell, T), w.G), dim3(T), 0, st, g, M, Mf, w.geoms, w.cellinfo,
                     w.ref_cell, bufs[cur]);
  for (int r = 0; r < o.path_radius; ++r) {
    hipLaunchKernelGGL(k_erode, dim3(blocks_for(g.ncell, T), w.G), dim3(T), 0, st, g, bufs[cur], bufs[1 - cur]);
    cur = 1 - cur;
  }
  if (n_face > 0) {
    hipLaunchKernelGGL(k_tmpl_pick, dim3(blocks_for(n_face, T)), dim3(T), 0, st, g, n_face, w.fcode, w.fref, w.canon,
                       w.tface);
    hipLaunchKernelGGL(k_tmpl_assign, dim3(blocks_for(n_face, T)), dim3(T), 0, st, g, n_face, w.fcode, w.fref,
                       w.canon, w.tface, w.tmpl);
  }
  CC_HIP(hipGetLastError());
  return CUTCELL_OK;
}

}  // namespace cutcell
