// Surface quadrature weights on the GPU (paper section 3.3, eqs. integral and
// functional_stencil): for every flat triangle E_j of a closed surface,
//   1. stencil S(E_j): the k nodes nearest to the centroid c_j;
//   2. projection point p_j (the origin for star-shaped surfaces; otherwise
//      the common point of the three cutting planes through E_j's edges);
//   3. stencil nodes pulled back along rays from p_j onto E_j's plane, with
//      the Jacobian of the central projection;
//   4. planar RBF-QF on E_j (phi = r^3 plus degree-2 polynomials): one
//      (k+6) x (k+6) saddle-point solve, right-hand side the exact integrals of
//      the basis over E_j;
//   5. q_i = sum of the scaled element weights of node i over all triangles,
//      added in increasing (triangle, slot) order.
// All arithmetic is FP64.  One wave per centroid group (k-nearest) and one
// wave per triangle (the solve); no float atomics, so q is reproducible.
#pragma once

#include "common.h"

namespace nfr {

// |p - c|^2 as (dx dx + dy dy) + dz dz with every operation rounded on its
// own (no fused multiply-add): stencil ranks are decided on this value.
__device__ inline double quad_sqdist(double px, double py, double pz, double cx, double cy, double cz) {
#pragma clang fp contract(off)
  const double dx = px - cx;
  const double dy = py - cy;
  const double dz = pz - cz;
  const double xy = dx * dx + dy * dy;
  return xy + dz * dz;
}

// Centroids (a + b + c) / 3 (summed in vertex order) and unit plane normals
// (b - a) x (c - a) / |.| of every triangle.
__global__ __launch_bounds__(kWG) void k_quad_centroids(const double* __restrict__ xyz, const int* __restrict__ tri,
                                                        int64_t ntri, double* __restrict__ cen,
                                                        double* __restrict__ nrm_tri) {
#pragma clang fp contract(off)
  const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (t >= ntri) return;
  const double* a = xyz + 3 * (int64_t)tri[3 * t];
  const double* b = xyz + 3 * (int64_t)tri[3 * t + 1];
  const double* c = xyz + 3 * (int64_t)tri[3 * t + 2];
  for (int d = 0; d < 3; ++d) cen[3 * t + d] = (a[d] + b[d] + c[d]) / 3.0;
  const double u0 = b[0] - a[0], u1 = b[1] - a[1], u2 = b[2] - a[2];
  const double v0 = c[0] - a[0], v1 = c[1] - a[1], v2 = c[2] - a[2];
  const double n0 = u1 * v2 - u2 * v1, n1 = u2 * v0 - u0 * v2, n2 = u0 * v1 - u1 * v0;
  const double len = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
  nrm_tri[3 * t] = n0 / len;
  nrm_tri[3 * t + 1] = n1 / len;
  nrm_tri[3 * t + 2] = n2 / len;
}

// ------------------------------------------------------------------ k nearest nodes

// Nodes are binned into a uniform grid of cubic cells; a centroid's search
// takes the cells within r = 1, 2, ... of its own, all at once by selection
// (quad_knn_select) or ring by ring (quad_knn_scan), and stops once its k-th
// key is below the squared distance from the centroid to the boundary of the
// cells visited (every node outside lies beyond it; a relative margin of 1e-12
// covers the rounding of the binning and of that bound).  The result is the exact k smallest (squared distance, index), the
// same as a full scan.

struct QuadGrid {
  double ox, oy, oz, h;   // origin (lower corner) and cell size
  int nx, ny, nz;
};

// One workgroup of kGridThreads threads (256 took 71 us at N = 65538, waiting for
// loads): bounding box of the nodes, then (thread 0) a
// grid with about 4 nodes per cell of the box's volume (a surface fills a
// small share of its box, so occupied cells hold a few tens of nodes), at most
// max_cells cells.
constexpr int kGridThreads = 1024;
__global__ __launch_bounds__(kGridThreads) void k_quad_grid(const double* __restrict__ xyz, int64_t n, int64_t max_cells,
                                                   QuadGrid* __restrict__ grid) {
  __shared__ double s_lo[3][kGridThreads], s_hi[3][kGridThreads];
  double lo[3] = {xyz[0], xyz[1], xyz[2]}, hi[3] = {xyz[0], xyz[1], xyz[2]};
  for (int64_t i = threadIdx.x; i < n; i += kGridThreads)
    for (int d = 0; d < 3; ++d) {
      lo[d] = fmin(lo[d], xyz[3 * i + d]);
      hi[d] = fmax(hi[d], xyz[3 * i + d]);
    }
  for (int d = 0; d < 3; ++d) {
    s_lo[d][threadIdx.x] = lo[d];
    s_hi[d][threadIdx.x] = hi[d];
  }
  __syncthreads();
  for (int w = kGridThreads / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int d = 0; d < 3; ++d) {
        s_lo[d][threadIdx.x] = fmin(s_lo[d][threadIdx.x], s_lo[d][threadIdx.x + w]);
        s_hi[d][threadIdx.x] = fmax(s_hi[d][threadIdx.x], s_hi[d][threadIdx.x + w]);
      }
    __syncthreads();
  }
  if (threadIdx.x != 0) return;
  double ext[3], emax = 0.0;
  for (int d = 0; d < 3; ++d) {
    ext[d] = s_hi[d][0] - s_lo[d][0];
    if (!(ext[d] < __builtin_inf())) ext[d] = 0.0;   // not finite: one layer of cells, as the search below ends for any
    emax = fmax(emax, ext[d]);
  }
  if (!(emax > 0.0)) emax = 1.0;
  // volume, with flat directions given a thousandth of the largest extent
  double h = cbrt(fmax(ext[0], emax * 1e-3) * fmax(ext[1], emax * 1e-3) * fmax(ext[2], emax * 1e-3) * 4.0 / (double)n);
  if (!(h > 0.0 && h < __builtin_inf())) h = emax;   // a volume beyond FP64's range: at most 8 cells
  int dim[3];
  for (;;) {
    int64_t cells = 1;
    for (int d = 0; d < 3; ++d) {
      dim[d] = (int)fmin(floor(ext[d] / h) + 1.0, 2048.0);
      cells *= dim[d];
    }
    if (cells <= max_cells) break;
    h *= 1.25;
  }
  grid->ox = s_lo[0][0];
  grid->oy = s_lo[1][0];
  grid->oz = s_lo[2][0];
  grid->h = h;
  grid->nx = dim[0];
  grid->ny = dim[1];
  grid->nz = dim[2];
}

__device__ inline int quad_cell_coord(double x, double o, double h, int dim) {
  const double c = floor((x - o) / h);
  return !(c > 0.0) ? 0 : (c >= (double)dim ? dim - 1 : (int)c);   // NaN: 0
}

__device__ inline int64_t quad_cell_of(const QuadGrid& g, double x, double y, double z) {
  const int cx = quad_cell_coord(x, g.ox, g.h, g.nx);
  const int cy = quad_cell_coord(y, g.oy, g.h, g.ny);
  const int cz = quad_cell_coord(z, g.oz, g.h, g.nz);
  return ((int64_t)cz * g.ny + cy) * g.nx + cx;
}

__global__ __launch_bounds__(kWG) void k_quad_bin_count(const double* __restrict__ xyz, int64_t n,
                                                        const QuadGrid* __restrict__ grid, int* __restrict__ cnt) {
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i >= n) return;
  atomicAdd(&cnt[quad_cell_of(*grid, xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2])], 1);
}

// Node i goes to a free place of its cell's list (order inside a cell is
// irrelevant: the ranking key is a total order).
__global__ __launch_bounds__(kWG) void k_quad_bin_fill(const double* __restrict__ xyz, int64_t n,
                                                       const QuadGrid* __restrict__ grid,
                                                       const int64_t* __restrict__ start, int* __restrict__ cursor,
                                                       int* __restrict__ nodes) {
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (i >= n) return;
  const int64_t c = quad_cell_of(*grid, xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]);
  nodes[start[c] + atomicAdd(&cursor[c], 1)] = (int)i;
}

__device__ inline bool key_less(double d, int i, double d2, int i2) { return d < d2 || (d == d2 && i < i2); }

// The k nodes with the smallest (squared distance, index) to the point c, in
// increasing order, entry r in lane r (one wave): rings of cells visited one
// cell after the other, the sorted list held one entry per lane; a candidate
// below the k-th key is inserted by a ballot (its rank) and a one-lane shift.
// Serves what quad_knn_select leaves (grids of few cells, clustered or
// coincident nodes).
__device__ inline int quad_knn_scan(const double* __restrict__ xyz, const QuadGrid& g, const int* __restrict__ cnt,
                                    const int64_t* __restrict__ start, const int* __restrict__ nodes, double cx,
                                    double cy, double cz, int k, int lane) {
  const int ix = quad_cell_coord(cx, g.ox, g.h, g.nx);
  const int iy = quad_cell_coord(cy, g.oy, g.h, g.ny);
  const int iz = quad_cell_coord(cz, g.oz, g.h, g.nz);
  double ld = __builtin_inf(), thr = __builtin_inf();
  int li = 0x7fffffff, thr_i = 0x7fffffff;
  const int rmax = max(max(g.nx, g.ny), g.nz);
  for (int r = 0; r <= rmax; ++r) {
    for (int dz = -r; dz <= r; ++dz) {
      const int z = iz + dz;
      if (z < 0 || z >= g.nz) continue;
      for (int dy = -r; dy <= r; ++dy) {
        const int y = iy + dy;
        if (y < 0 || y >= g.ny) continue;
        const bool face = dz == -r || dz == r || dy == -r || dy == r;
        for (int dx = -r; dx <= r; dx += (face || r == 0) ? 1 : 2 * r) {   // only the ring's shell
          const int x = ix + dx;
          if (x < 0 || x >= g.nx) continue;
          const int64_t c = ((int64_t)z * g.ny + y) * g.nx + x;
          const int64_t c0 = start[c];
          const int m = cnt[c];
          for (int b = 0; b < m; b += 64) {
            const bool valid = b + lane < m;
            const int j = valid ? nodes[c0 + b + lane] : 0;
            const double key = valid ? quad_sqdist(xyz[3 * (int64_t)j], xyz[3 * (int64_t)j + 1],
                                                   xyz[3 * (int64_t)j + 2], cx, cy, cz)
                                     : 0.0;
            uint64_t mask = __ballot(valid && key_less(key, j, thr, thr_i));
            while (mask) {
              const int src = __builtin_ctzll(mask);
              mask &= mask - 1;
              const double cd = __shfl(key, src);
              const int ci = __shfl(j, src);
              if (!key_less(cd, ci, thr, thr_i)) continue;
              const bool before = lane < k && key_less(ld, li, cd, ci);
              const int pos = __popcll(__ballot(before));
              const double up_d = __shfl_up(ld, 1);
              const int up_i = __shfl_up(li, 1);
              if (lane == pos) {
                ld = cd;
                li = ci;
              } else if (lane > pos && lane < k) {
                ld = up_d;
                li = up_i;
              }
              thr = __shfl(ld, k - 1);
              thr_i = __shfl(li, k - 1);
            }
          }
        }
      }
    }
    // distance from the centroid to the boundary of rings 0..r (sides with no
    // cells beyond them do not count)
    double bound = __builtin_inf();
    const double o[3] = {g.ox, g.oy, g.oz};
    const double p[3] = {cx, cy, cz};
    const int ic[3] = {ix, iy, iz};
    const int dims[3] = {g.nx, g.ny, g.nz};
    for (int d = 0; d < 3; ++d) {
      if (ic[d] - r > 0) bound = fmin(bound, p[d] - (o[d] + (double)(ic[d] - r) * g.h));
      if (ic[d] + r < dims[d] - 1) bound = fmin(bound, (o[d] + (double)(ic[d] + r + 1) * g.h) - p[d]);
    }
    if (bound == __builtin_inf()) break;                                   // every cell visited
    if (thr_i != 0x7fffffff && bound > 0.0 && thr < bound * bound * (1.0 - 1e-12)) break;
  }
  return li;
}

// The same by selection; returns false where it does not apply.  The nodes of
// the (2 r + 1)^2 rows of cells around c (a row's cells are consecutive in the
// cell order, so its nodes are one run of `nodes`) are flattened over the lanes,
// up to kKnnHeld per lane; when at least k keys lie below the squared distance
// to the rows' boundary, a threshold with k to 64 keys below it is found by
// counting ballots (keys of a surface's nodes are about evenly spread, so
// interpolation hits within a few tries), and those keys are sorted.
constexpr int kKnnHeld = 8;
struct KnnScratch {
  double key[64];
  int idx[64], pre[64], beg[64];
};

__device__ inline bool quad_knn_select(const double* __restrict__ xyz, const QuadGrid& g, const int* __restrict__ cnt,
                                       const int64_t* __restrict__ start, const int* __restrict__ nodes, double cx,
                                       double cy, double cz, int k, int lane, KnnScratch& s, int* out) {
  const int ix = quad_cell_coord(cx, g.ox, g.h, g.nx);
  const int iy = quad_cell_coord(cy, g.oy, g.h, g.ny);
  const int iz = quad_cell_coord(cz, g.oz, g.h, g.nz);
  for (int r = 1; r <= 3; ++r) {
    const int side = 2 * r + 1;
    int beg = 0, len = 0;
    {
      const int y = iy + lane % side - r, z = iz + lane / side - r;
      if (lane < side * side && y >= 0 && y < g.ny && z >= 0 && z < g.nz) {
        const int64_t c = ((int64_t)z * g.ny + y) * g.nx;
        const int x0 = max(ix - r, 0), x1 = min(ix + r, g.nx - 1);
        beg = (int)start[c + x0];
        len = (int)start[c + x1] + cnt[c + x1] - beg;
      }
    }
    int pre = len;   // inclusive prefix sum over the rows
    for (int o = 1; o < 64; o *= 2) {
      const int v = __shfl_up(pre, o);
      if (lane >= o) pre += v;
    }
    const int total = __builtin_amdgcn_readlane(pre, 63);
    if (total > 64 * kKnnHeld) return false;
    double bound = __builtin_inf();   // distance to the nearest side with cells beyond it
    const double o[3] = {g.ox, g.oy, g.oz};
    const double p[3] = {cx, cy, cz};
    const int ic[3] = {ix, iy, iz};
    const int dims[3] = {g.nx, g.ny, g.nz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      if (ic[d] - r > 0) bound = fmin(bound, p[d] - (o[d] + (double)(ic[d] - r) * g.h));
      if (ic[d] + r < dims[d] - 1) bound = fmin(bound, (o[d] + (double)(ic[d] + r + 1) * g.h) - p[d]);
    }
    if (bound == __builtin_inf()) return false;
    if (total < k || !(bound > 0.0)) continue;
    const double b2 = bound * bound * (1.0 - 1e-12);

    s.pre[lane] = pre;
    s.beg[lane] = beg - (pre - len);
    __builtin_amdgcn_wave_barrier();
    double key[kKnnHeld];
    int idx[kKnnHeld];
#pragma unroll
    for (int q = 0; q < kKnnHeld; ++q) {
      key[q] = __builtin_inf();
      idx[q] = 0;
      if (64 * q >= total) continue;
      const int e = 64 * q + lane;
      int row = 0;             // first row whose prefix exceeds e
#pragma unroll
      for (int w = 32; w > 0; w /= 2)
        if (s.pre[row + w - 1] <= e) row += w;
      if (e < total) {
        const int j = nodes[s.beg[row] + e];
        idx[q] = j;
        key[q] = quad_sqdist(xyz[3 * (int64_t)j], xyz[3 * (int64_t)j + 1], xyz[3 * (int64_t)j + 2], cx, cy, cz);
      }
    }
    auto below = [&](double t) {
      int c = 0;
#pragma unroll
      for (int q = 0; q < kKnnHeld; ++q)
        if (64 * q < total) c += __popcll(__ballot(key[q] < t));
      return c;
    };
    double t = b2, t_lo = 0.0;
    int c = below(t), c_lo = 0;
    if (c < k) continue;
    if (c > 64) {
      double t_hi = t;
      int c_hi = c, tries = 0;
      const double want = 0.5 * (k + 64);
      for (;; ++tries) {
        if (tries == 40) return false;        // equal keys
        const double f = tries < 8 ? (want - c_lo) / (double)(c_hi - c_lo) : 0.5;
        t = t_lo + (t_hi - t_lo) * f;
        c = below(t);
        if (c < k) {
          t_lo = t;
          c_lo = c;
        } else if (c > 64) {
          t_hi = t;
          c_hi = c;
        } else {
          break;
        }
      }
    }
    s.key[lane] = __builtin_inf();
    s.idx[lane] = 0x7fffffff;
    __builtin_amdgcn_wave_barrier();
    int base = 0;
#pragma unroll
    for (int q = 0; q < kKnnHeld; ++q) {
      if (64 * q >= total) continue;
      const bool in = key[q] < t;
      const uint64_t mask = __ballot(in);
      const int at = base + __popcll(mask & ((1ull << lane) - 1));
      if (in) {
        s.key[at] = key[q];
        s.idx[at] = idx[q];
      }
      base += __popcll(mask);
    }
    __builtin_amdgcn_wave_barrier();
    double d = s.key[lane];
    int i = s.idx[lane];
    __builtin_amdgcn_wave_barrier();
    for (int w = 2; w <= 64; w *= 2)          // bitonic sort of the 64 (key, index)
      for (int j = w / 2; j > 0; j /= 2) {
        const double pd = __shfl_xor(d, j);
        const int pi = __shfl_xor(i, j);
        const bool up = (lane & w) == 0, low = (lane & j) == 0;
        const bool take = key_less(pd, pi, d, i) == (up == low);
        d = take ? pd : d;
        i = take ? pi : i;
      }
    *out = i;
    return true;
  }
  return false;
}

// st[t*k + r], r < k: the stencil of triangle t (one wave); rank[t*k + r]: the
// entry's place among its node's entries, in the order in which they arrive.
// cnt / start: nodes per cell and their offsets into `nodes`.  Requires k <= 64
// and k <= n.  N = 65538, k = 32: 230 us; 930 us by quad_knn_scan alone, whose
// cells and insertions follow one another.
__global__ __launch_bounds__(kWG) void k_quad_knn(const double* __restrict__ xyz, const QuadGrid* __restrict__ grid_p,
                                                  const int* __restrict__ cnt, const int64_t* __restrict__ start,
                                                  const int* __restrict__ nodes, const double* __restrict__ cen,
                                                  int64_t n, int64_t ntri, int k, int* __restrict__ st,
                                                  int* __restrict__ node_cnt, int* __restrict__ rank) {
  __shared__ KnnScratch scratch[kWG / 64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t = (int64_t)blockIdx.x * (kWG / 64) + wave;
  if (t >= ntri) return;
  const QuadGrid g = *grid_p;
  const double cx = cen[3 * t], cy = cen[3 * t + 1], cz = cen[3 * t + 2];
  int li;
  if (!quad_knn_select(xyz, g, cnt, start, nodes, cx, cy, cz, k, lane, scratch[wave], &li))
    li = quad_knn_scan(xyz, g, cnt, start, nodes, cx, cy, cz, k, lane);
  if (lane >= k) return;
  st[t * k + lane] = li;
  if (li >= 0 && li < n) rank[t * k + lane] = atomicAdd(&node_cnt[li], 1);
}

// ------------------------------------------------------------------ projection points

// Singular values of a 3 x 3 matrix (rows m[0..2]) by one-sided Jacobi
// rotations of its columns; returns sigma_max / sigma_min (inf if singular).
__device__ inline double cond3(const double m[3][3]) {
  double a[3][3];
  for (int r = 0; r < 3; ++r)
    for (int c = 0; c < 3; ++c) a[r][c] = m[r][c];
  for (int sweep = 0; sweep < 30; ++sweep) {
    bool rotated = false;
    for (int i = 0; i < 2; ++i)
      for (int j = i + 1; j < 3; ++j) {
        double al = 0.0, be = 0.0, ga = 0.0;
        for (int r = 0; r < 3; ++r) {
          al += a[r][i] * a[r][i];
          be += a[r][j] * a[r][j];
          ga += a[r][i] * a[r][j];
        }
        if (fabs(ga) <= 1e-15 * sqrt(al * be)) continue;
        rotated = true;
        const double zeta = (be - al) / (2.0 * ga);
        const double tn = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
        const double cs = 1.0 / sqrt(1.0 + tn * tn);
        const double sn = cs * tn;
        for (int r = 0; r < 3; ++r) {
          const double x = a[r][i], y = a[r][j];
          a[r][i] = cs * x - sn * y;
          a[r][j] = sn * x + cs * y;
        }
      }
    if (!rotated) break;
  }
  double smax = 0.0, smin = __builtin_inf();
  for (int c = 0; c < 3; ++c) {
    const double s = sqrt(a[0][c] * a[0][c] + a[1][c] * a[1][c] + a[2][c] * a[2][c]);
    smax = fmax(smax, s);
    smin = fmin(smin, s);
  }
  return smin > 0.0 ? smax / smin : __builtin_inf();
}

// p_j for every triangle (written to proj[3*t]; a NaN row means "orthogonal
// projection onto E_j's plane").  mode 1 (origin): p_j = 0; mode 2
// (orthogonal): a NaN row for every triangle.  Mode 0 (planes): row e of the
// 3 x 3 system is the unit normal of the cutting plane through edge e
// (vertex e to vertex e+1), n_j - n_{neighbour across e} normalised, with
// right-hand side its product with (vertex e - c_j); p_j = c_j + solution.
// A system with condition number above cond_max (or a zero row) falls back
// to orthogonal projection.
__global__ __launch_bounds__(kWG) void k_quad_proj(const double* __restrict__ xyz, const int* __restrict__ tri,
                                                   const int* __restrict__ nbr, const double* __restrict__ cen,
                                                   const double* __restrict__ nrm_tri, int64_t ntri, int mode,
                                                   double cond_max, double* __restrict__ proj) {
  const int64_t t = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (t >= ntri) return;
  if (mode == 1) {
    proj[3 * t] = proj[3 * t + 1] = proj[3 * t + 2] = 0.0;
    return;
  }
  if (mode == 2) {
    const double nan = __builtin_nan("");
    proj[3 * t] = proj[3 * t + 1] = proj[3 * t + 2] = nan;
    return;
  }
  double m[3][3], rhs[3];
  bool ok = true;
  for (int e = 0; e < 3; ++e) {
    const int64_t o = nbr[3 * t + e];
    double row[3], len2 = 0.0;
    for (int d = 0; d < 3; ++d) {
      row[d] = nrm_tri[3 * t + d] - nrm_tri[3 * o + d];
      len2 += row[d] * row[d];
    }
    const double len = sqrt(len2);
    if (!(len > 0.0)) ok = false;
    double r = 0.0;
    const double* v = xyz + 3 * (int64_t)tri[3 * t + e];
    for (int d = 0; d < 3; ++d) {
      m[e][d] = row[d] / len;
      r += m[e][d] * (v[d] - cen[3 * t + d]);
    }
    rhs[e] = r;
  }
  if (ok && !(cond3(m) <= cond_max)) ok = false;
  if (!ok) {
    const double nan = __builtin_nan("");
    proj[3 * t] = proj[3 * t + 1] = proj[3 * t + 2] = nan;
    return;
  }
  // Gaussian elimination with partial pivoting on [m | rhs]
  int perm[3] = {0, 1, 2};
  for (int c = 0; c < 3; ++c) {
    int piv = c;
    for (int r = c + 1; r < 3; ++r)
      if (fabs(m[perm[r]][c]) > fabs(m[perm[piv]][c])) piv = r;
    const int tmp = perm[c];
    perm[c] = perm[piv];
    perm[piv] = tmp;
    for (int r = c + 1; r < 3; ++r) {
      const double f = m[perm[r]][c] / m[perm[c]][c];
      for (int cc = c; cc < 3; ++cc) m[perm[r]][cc] -= f * m[perm[c]][cc];
      rhs[perm[r]] -= f * rhs[perm[c]];
    }
  }
  double x[3];
  for (int c = 2; c >= 0; --c) {
    double s = rhs[perm[c]];
    for (int cc = c + 1; cc < 3; ++cc) s -= m[perm[c]][cc] * x[cc];
    x[c] = s / m[perm[c]][c];
  }
  for (int d = 0; d < 3; ++d) proj[3 * t + d] = cen[3 * t + d] + x[d];
}

// ------------------------------------------------------------------ element weights

// Integral of |s - P|^3 over the triangle (P, p, q) (2-D, unsigned).  In
// polar coordinates about P it is (d^5 / 5) times the antiderivative of
// sec^5 between the angles of p and q, d the distance from P to the line pq;
// with rho = d sec(alpha) and l = d tan(alpha) (l measured along p -> q from
// the foot of the perpendicular) the antiderivative times d^4 reads
//   rho^3 l / 4 + 3 d^2 rho l / 8 + 3 d^4 log(rho + l) / 8.
// For l < 0, rho + l = d^2 / (rho - l) (no cancellation); the difference of the
// two logarithms is taken as the logarithm of one quotient.
__device__ inline double r3_apex(double Px, double Py, double px, double py, double qx, double qy) {
  const double ex = qx - px, ey = qy - py;
  const double len = sqrt(ex * ex + ey * ey);
  const double ux = ex / len, uy = ey / len;
  const double wx = px - Px, wy = py - Py;
  const double lp = wx * ux + wy * uy;
  const double lq = lp + len;
  const double d = fabs(wx * uy - wy * ux);
  const double d2 = d * d;
  const double rp = sqrt(d2 + lp * lp);
  const double rq = sqrt(d2 + lq * lq);
  double val = 0.25 * (rq * rq * rq * lq - rp * rp * rp * lp) + 0.375 * d2 * (rq * lq - rp * lp);
  if (d > 0.0) {
    const double num = lp >= 0.0 ? rq + lq : rp - lp;
    const double den = lp >= 0.0 ? rp + lp : rq - lq;
    // lp < 0 <= lq: the two sides of the foot, log(rq + lq) + log(rp - lp) - 2 log d
    const double L = (lp < 0.0 && lq >= 0.0) ? log((rq + lq) / d) + log(num / d) : log(num / den);
    val += 0.375 * d2 * d2 * L;
  }
  return d * val / 5.0;
}

__device__ inline double cross2(double ax, double ay, double bx, double by) { return ax * by - ay * bx; }

__device__ inline double sgn(double x) { return x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0); }

// Integral of |s - P|^3 over the triangle (v0, v1, v2): the three triangles
// with apex P, each signed by its orientation relative to the triangle's.
__device__ inline double r3_triangle(double Px, double Py, const double v[3][2]) {
  const double o = sgn(cross2(v[1][0] - v[0][0], v[1][1] - v[0][1], v[2][0] - v[0][0], v[2][1] - v[0][1]));
  double total = 0.0;
  for (int e = 0; e < 3; ++e) {
    const double* p = v[e];
    const double* q = v[(e + 1) % 3];
    const double s = sgn(cross2(p[0] - Px, p[1] - Py, q[0] - Px, q[1] - Py)) * o;
    if (s != 0.0) total += s * r3_apex(Px, Py, p[0], p[1], q[0], q[1]);
  }
  return total;
}

__device__ inline double mono2(int m, double x, double y) {
  switch (m) {
    case 0: return 1.0;
    case 1: return x;
    case 2: return y;
    case 3: return x * x;
    case 4: return x * y;
    default: return y * y;
  }
}

constexpr int kQuadMaxK = 57;   // k + 7 <= 64: one lane per column of the system and its right-hand side

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Maximum over the 64 lanes of a wave (DPP moves fused into the maximum; lane 63 holds it).
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  auto step = [&](auto ctrl, auto rows) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xF, false);
    v = v > o ? v : o;
  };
  using std::integral_constant;
  step(integral_constant<int, 0xB1>{}, integral_constant<int, 0xF>{});    // quad_perm [1, 0, 3, 2]
  step(integral_constant<int, 0x4E>{}, integral_constant<int, 0xF>{});    // quad_perm [2, 3, 0, 1]
  step(integral_constant<int, 0x141>{}, integral_constant<int, 0xF>{});   // row_half_mirror
  step(integral_constant<int, 0x140>{}, integral_constant<int, 0xF>{});   // row_mirror
  step(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});   // row_bcast15 into rows 1 and 3
  step(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});   // row_bcast31 into rows 2 and 3
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// One wave per triangle t: pull-back, Jacobian, planar system, LU with partial
// pivoting, back substitution; entry e = t*k + r gives w_r h_t^2 J_r to its node's
// list (place off[node] + rank[e]).
//
// Lane r holds row r of the (k+6) x (k+6) system and its right-hand side in
// registers, with the kernel columns at 0 .. k-1 and the polynomial columns at
// KP .. KP+5 (KP >= k, the size the registers are cut for; the columns between
// are skipped).  Rows are not moved: a step takes the pivot among the lanes
// still available, and every other available lane subtracts its multiple of
// the pivot lane's row, whose elements reach the wave as scalars (two lane
// reads per multiply-add).  Pivots are compared by the upper 32 bits of their
// magnitude (20 of 52 mantissa bits), the lowest lane among equals.  Bound by
// instruction issue: about 750 multiply-adds, 1500 lane reads and 32 square
// roots per lane at k = 32 (2, 3 or 4 waves per SIMD: the same time).
// N = 65538, k = 32 (131072 triangles): 2.02 ms; 4.73 ms with the matrix in LDS
// and a lane per column (barriers and LDS latency in every step).
template <int KP>
__global__ __launch_bounds__(64) void k_quad_elements(const double* __restrict__ xyz, const double* __restrict__ nrm,
                                                      const int* __restrict__ tri, const double* __restrict__ cen,
                                                      const double* __restrict__ nrm_tri,
                                                      const double* __restrict__ proj, const int* __restrict__ st,
                                                      int64_t n, int64_t ntri, int k, const int64_t* __restrict__ off,
                                                      const int* __restrict__ rank, double* __restrict__ val,
                                                      int* __restrict__ list) {
  constexpr int D = KP + 6;
  __shared__ double s_poly[6][KP];     // polynomial rows (the transposed polynomial columns)
  const int dim = k + 6;
  const int64_t t = blockIdx.x;
  const int lane = threadIdx.x;
  if (t >= ntri) return;

  double A[3], B[3], C[3], nj[3], cj[3], p[3];
  for (int d = 0; d < 3; ++d) {
    A[d] = xyz[3 * (int64_t)tri[3 * t] + d];
    B[d] = xyz[3 * (int64_t)tri[3 * t + 1] + d];
    C[d] = xyz[3 * (int64_t)tri[3 * t + 2] + d];
    nj[d] = nrm_tri[3 * t + d];
    cj[d] = cen[3 * t + d];
    p[d] = proj[3 * t + d];
  }
  const bool orth = p[0] != p[0];
  // frame of E_j: e1 along B - A, e2 = n_j x e1
  double e1[3] = {B[0] - A[0], B[1] - A[1], B[2] - A[2]};
  {
    const double l = sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
    for (int d = 0; d < 3; ++d) e1[d] /= l;
  }
  const double e2[3] = {nj[1] * e1[2] - nj[2] * e1[1], nj[2] * e1[0] - nj[0] * e1[2], nj[0] * e1[1] - nj[1] * e1[0]};

  // lane r < k: stencil node, its pre-image xi on E_j's plane and the Jacobian
  double J = 0.0, rel1 = 0.0, rel2 = 0.0, rlen = 0.0;
  if (lane < k) {
    const int64_t s = st[t * k + lane];
    const bool in_range = s >= 0 && s < n;   // a stencil slot left unfilled (non-finite coordinates) gives NaN
    double X[3], Ns[3], xi[3];
    for (int d = 0; d < 3; ++d) {
      X[d] = in_range ? xyz[3 * s + d] : __builtin_nan("");
      Ns[d] = in_range ? nrm[3 * s + d] : __builtin_nan("");
    }
    if (!orth) {
      double dxp[3], num = 0.0, den = 0.0, nx = 0.0;
      for (int d = 0; d < 3; ++d) {
        dxp[d] = X[d] - p[d];
        num += nj[d] * (A[d] - p[d]);
        den += nj[d] * dxp[d];
        nx += dxp[d] * dxp[d];
      }
      const double tt = num / den;
      double nxi = 0.0, cp = 0.0, cs = 0.0;
      nx = sqrt(nx);
      for (int d = 0; d < 3; ++d) {
        xi[d] = p[d] + tt * dxp[d];
        const double diff = xi[d] - p[d];
        nxi += diff * diff;
        cp += nj[d] * dxp[d] / nx;
        cs += Ns[d] * dxp[d] / nx;
      }
      const double ratio = nx / sqrt(nxi);
      J = ratio * ratio * fabs(cp) / fabs(cs);
    } else {
      double h = 0.0, c = 0.0;
      for (int d = 0; d < 3; ++d) {
        h += nj[d] * (X[d] - A[d]);
        c += Ns[d] * nj[d];
      }
      for (int d = 0; d < 3; ++d) xi[d] = X[d] - h * nj[d];
      J = 1.0 / fabs(c);
    }
    double rel[3];
    for (int d = 0; d < 3; ++d) rel[d] = xi[d] - cj[d];
    rel1 = rel[0] * e1[0] + rel[1] * e1[1] + rel[2] * e1[2];
    rel2 = rel[0] * e2[0] + rel[1] * e2[1] + rel[2] * e2[2];
    rlen = sqrt(rel[0] * rel[0] + rel[1] * rel[1] + rel[2] * rel[2]);
  }
  // h_t = largest stencil radius (wave maximum)
  double h = rlen;
  for (int off = 32; off > 0; off >>= 1) h = fmax(h, __shfl_xor(h, off));
  double v[3][2];
  {
    const double* V[3] = {A, B, C};
    for (int i = 0; i < 3; ++i) {
      double r0 = 0.0, r1 = 0.0;
      for (int d = 0; d < 3; ++d) {
        r0 += (V[i][d] - cj[d]) * e1[d];
        r1 += (V[i][d] - cj[d]) * e2[d];
      }
      v[i][0] = r0 / h;
      v[i][1] = r1 / h;
    }
  }
  const double sx = rel1 / h, sy = rel2 / h;

  // rows r < k: [|s_r - s_c|^3 (c < k) | pi_m(s_r) | int_E |s - s_r|^3]
  // rows k + m: [pi_m(s_c) (c < k) | 0 | int_E pi_m]
  double a[D], rhs = 0.0;
#pragma unroll
  for (int c = 0; c < KP; ++c) {
    a[c] = 0.0;
    if (c < k) {
      const double dx = sx - readlane_f64(sx, c), dy = sy - readlane_f64(sy, c);
      const double r2 = dx * dx + dy * dy;
      a[c] = r2 * sqrt(r2);
    }
  }
#pragma unroll
  for (int m = 0; m < 6; ++m) {
    a[KP + m] = mono2(m, sx, sy);
    if (lane < k) s_poly[m][lane] = a[KP + m];
  }
  __syncthreads();
  if (lane < k) {
    rhs = r3_triangle(sx, sy, v);
  } else if (lane < dim) {
    const int m = lane - k;
#pragma unroll
    for (int c = 0; c < KP; ++c) a[c] = c < k ? s_poly[m][c] : 0.0;
#pragma unroll
    for (int c = KP; c < D; ++c) a[c] = 0.0;
    // exact for degree 2: area / 3 times the sum over the edge midpoints
    const double area = 0.5 * fabs(cross2(v[1][0] - v[0][0], v[1][1] - v[0][1], v[2][0] - v[0][0], v[2][1] - v[0][1]));
    double acc = 0.0;
    for (int e = 0; e < 3; ++e) {
      const int f = (e + 1) % 3;
      acc += mono2(m, 0.5 * (v[e][0] + v[f][0]), 0.5 * (v[e][1] + v[f][1]));
    }
    rhs = acc * (area / 3.0);
  }

  uint64_t avail = dim < 64 ? (1ull << dim) - 1 : ~0ull;   // rows that have not been pivots
  int row_of = 0;                                           // lane c: the pivot row of column c
  double diag = 1.0;                                        // this row's pivot
#pragma unroll
  for (int col = 0; col < D; ++col) {
    if (col < KP && col >= k) continue;
    const bool mine = (avail >> lane) & 1;
    const uint32_t mag = mine ? (uint32_t)(__builtin_bit_cast(uint64_t, a[col]) >> 32) & 0x7fffffffu : 0u;
    const uint32_t top = wave_max_u32(mag);
    const int p = __builtin_ctzll(__ballot(mine && mag == top));
    avail &= ~(1ull << p);
    row_of = lane == col ? p : row_of;
    const double pv = readlane_f64(a[col], p);
    diag = lane == p ? pv : diag;
    const double l = (mine && lane != p) ? a[col] / pv : 0.0;
#pragma unroll
    for (int c = col + 1; c < D; ++c) a[c] = fma(-l, readlane_f64(a[c], p), a[c]);
    rhs = fma(-l, readlane_f64(rhs, p), rhs);
  }
  // back substitution: every lane subtracts, only rows still to be solved matter
  const double rdiag = 1.0 / diag;
  double w = 0.0;
#pragma unroll
  for (int col = D - 1; col >= 0; --col) {
    if (col < KP && col >= k) continue;
    const int p = __builtin_amdgcn_readlane(row_of, col);
    double x = rhs * rdiag;
    x = fma(fma(-diag, x, rhs), rdiag, x);
    const double xc = readlane_f64(x, p);
    rhs = fma(-a[col], xc, rhs);
    w = lane == col ? xc : w;
  }
  if (lane < k) {
    const int64_t e = t * k + lane;
    const int i = st[e];
    if (i >= 0 && i < n) {
      const int64_t at = off[i] + rank[e];
      val[at] = w * h * h * J;
      list[at] = (int)e;
    }
  }
}

// ------------------------------------------------------------------ accumulation

// Exclusive prefix sums in three passes: block totals, a single-workgroup
// scan of the totals, then each block's own scan plus its offset.
__global__ __launch_bounds__(kWG) void k_scan_blocks(const int* __restrict__ cnt, int64_t n,
                                                     int64_t* __restrict__ bsum) {
  __shared__ int64_t s[kWG];
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  s[threadIdx.x] = i < n ? cnt[i] : 0;
  __syncthreads();
  for (int w = kWG / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) bsum[blockIdx.x] = s[0];
}

__global__ __launch_bounds__(kWG) void k_scan_totals(int64_t* __restrict__ bsum, int64_t nb) {
  __shared__ int64_t s[kWG];
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kWG) {
    const int64_t b = b0 + threadIdx.x;
    const int64_t v = b < nb ? bsum[b] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int w = 1; w < kWG; w <<= 1) {
      const int64_t add = threadIdx.x >= w ? s[threadIdx.x - w] : 0;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    if (b < nb) bsum[b] = carry + s[threadIdx.x] - v;
    carry += s[kWG - 1];
    __syncthreads();
  }
}

__global__ __launch_bounds__(kWG) void k_scan_apply(const int* __restrict__ cnt, int64_t n,
                                                    const int64_t* __restrict__ bsum, int64_t* __restrict__ off) {
  __shared__ int64_t s[kWG];
  const int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x;
  const int64_t v = i < n ? cnt[i] : 0;
  s[threadIdx.x] = v;
  __syncthreads();
  for (int w = 1; w < kWG; w <<= 1) {
    const int64_t add = threadIdx.x >= w ? s[threadIdx.x - w] : 0;
    __syncthreads();
    s[threadIdx.x] += add;
    __syncthreads();
  }
  if (i < n) off[i] = bsum[blockIdx.x] + s[threadIdx.x] - v;
}

// q_i = sum of node i's entries in increasing order of their numbers, one after
// the other from 0, one wave per node: up to kSumHeld entries are put in that
// order through LDS by their rank among the others (every lane then adds the
// same broadcasts); longer lists (never a mesh of bounded valence) are searched
// for the next entry each time.  A thread per
// node sorting its list in memory took 490 us at N = 65538, a wave 66 (60 with its
// lanes adding strided parts, in another order).
constexpr int kSumHeld = 256;
__global__ __launch_bounds__(kWG) void k_quad_sum(const int64_t* __restrict__ off, const int* __restrict__ cnt,
                                                  int64_t n, const int* __restrict__ list,
                                                  const double* __restrict__ val, double* __restrict__ q) {
  __shared__ double s_val[kWG / 64][kSumHeld];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t i = (int64_t)blockIdx.x * (kWG / 64) + wave;
  if (i >= n) return;
  const int len = __builtin_amdgcn_readfirstlane(cnt[i]);
  const int* const seg = list + off[i];
  const double* const v = val + off[i];
  double acc = 0.0;
  if (len <= kSumHeld) {
    int e[kSumHeld / 64];
#pragma unroll
    for (int c = 0; c < kSumHeld / 64; ++c) e[c] = 64 * c + lane < len ? seg[64 * c + lane] : 0x7fffffff;
    for (int c = 0; 64 * c < len; ++c) {
      const int mine = 64 * c + lane < len ? seg[64 * c + lane] : 0x7fffffff;
      int r = 0;
#pragma unroll
      for (int d = 0; d < kSumHeld / 64; ++d)
        for (int b = 0; b < 64 && 64 * d + b < len; ++b) r += __builtin_amdgcn_readlane(e[d], b) < mine ? 1 : 0;
      if (64 * c + lane < len) s_val[wave][r] = v[64 * c + lane];
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 8
    for (int c = 0; c < len; ++c) acc += s_val[wave][c];
  } else {
    int last = -1;
    for (int a = 0; a < len; ++a) {
      int best = 0x7fffffff, at = 0;
      for (int c = lane; c < len; c += 64)
        if (seg[c] > last && seg[c] < best) {
          best = seg[c];
          at = c;
        }
      for (int o = 32; o > 0; o >>= 1) {
        const int ob = __shfl_xor(best, o), oa = __shfl_xor(at, o);
        if (ob < best) {
          best = ob;
          at = oa;
        }
      }
      acc += v[at];
      last = best;
    }
  }
  if (lane == 0) q[i] = acc;
}

}  // namespace nfr
