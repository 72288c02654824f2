// Tile order of a problem's nodes.
//
// The fused split kernel evaluates the normalised kernel
// u = exp2(-t) + kappa exp2(-rho t) of a Gaussian Mexican hat (rho < 1: the
// excitatory exponential is the steeper one).  Where (1 - rho) t exceeds
// 25 - log2|kappa| the first term is below half a unit in the last place of
// the second, so the FP32 sum equals the second term alone and the first
// exponential need not be evaluated.  Whether a whole block of entries lies
// in that range follows from bounding spheres of its target and source
// nodes, which is useful only when consecutive nodes are close in space.
// The tile order is a permutation of the nodes that makes them so (a k-d
// tree, below).  Problems keep their own node order at the boundary; the
// fused form gathers states into the tile order at the start of a call and
// scatters them back at the end.
#pragma once

#include "common.h"

namespace nfr {

constexpr int kTileRowBlock = 32;   // target rows per wave of the fused kernel
constexpr int kTileColBlock = 16;   // source columns per MFMA step of the fused kernel

// The order is built by recursive bisection (a k-d tree): level l cuts the
// slots into 2^l segments of whole 16-slot blocks, segment s holding blocks
// [floor(s nb / 2^l), floor((s + 1) nb / 2^l)) of the nb = ceil(n / 16) blocks
// (the last one may be partial); each segment is ordered along the longest
// axis of its nodes' bounding box, so that its halves at the next level are
// the nodes below and above its median.  After the last level every segment
// is one block of 16 nodes, and blocks of 32 are two sibling leaves.  Nodes of
// a segment are ranked by the key coordinate along the axis quantised to 24
// bits over the segment's extent | node index (22 bits); keys are unique, so
// the order is deterministic.  On the ellipsoid of 65536 nodes 75 % of the
// 32 x 16 blocks of one application are far with this order (a Morton order
// gave 69 %, a Hilbert order 72 %).
//
// A level needs only the two sets, not their order, until the last one: the
// levels whose segments exceed kTileLocal slots select the median key and
// partition (k_tile_split, one workgroup per segment, one launch per level);
// the levels below run in LDS, all in one launch (k_tile_local).  Selection
// by digit histograms reads a segment a few times, where bitonic sorts of the
// whole array went over it once per compare-exchange pass and launch: problem
// creation at N = 2000 / 20000 / 65536 / 262144 takes 92 / 168 / 289 / 875 us
// in 7 to 14 launches, against 1176 / 3292 / 3904 / 6660 us in 475 to 3460.
constexpr int kTileLeaf = 16;
constexpr int kTileNodeBits = 22, kTileCoordBits = 24;
// Slots of a segment that k_tile_local takes: its counting is quadratic in
// them (N = 2000: 323 us with 2048 slots; with 512, 35 us and two more split
// levels of 13 us each).
constexpr int kTileLocal = 512;
constexpr int kTileThreads = 1024;        // of k_tile_split

inline int tile_levels(int64_t n) {
  const int64_t nb = ceil_div(n, kTileLeaf);
  int L = 0;
  while ((int64_t(1) << L) < nb) ++L;
  return L;
}

// Levels that k_tile_split handles: the first whose segments all fit k_tile_local.
inline int tile_split_levels(int64_t n) {
  const int64_t nb = ceil_div(n, kTileLeaf);
  int l = 0;
  while (ceil_div(nb, int64_t(1) << l) * kTileLeaf > kTileLocal) ++l;
  return l;
}

// First slot of segment s at level l (s = 2^l: n), nb blocks.
__device__ inline int64_t tile_seg_start(int64_t s, int l, int64_t nb, int64_t n) {
  const int64_t v = ((s * nb) >> l) * kTileLeaf;
  return v < n ? v : n;
}

// Floats as unsigned integers in the same order, so that box sides are exact
// integer minima and maxima; NaN coordinates are left out of the box.
__device__ inline uint32_t tile_enc(float x) {
  const uint32_t b = __builtin_bit_cast(uint32_t, x);
  return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}
__device__ inline float tile_dec(uint32_t e) {
  return __builtin_bit_cast(float, e ^ ((e >> 31) ? 0x80000000u : 0xffffffffu));
}

// Axis, origin and extent of a segment's key from its encoded box (lo[3], hi[3]);
// a box of no finite node has lo > hi and gets extent <= 0 (every coordinate 0).
struct TileAxis {
  int ax;
  double lo, ext;
};
__device__ inline TileAxis tile_axis(const uint32_t* lo, const uint32_t* hi) {
  TileAxis a{0, 0.0, -1.0};
  for (int d = 0; d < 3; ++d) {
    if (lo[d] > hi[d]) continue;
    const double l = tile_dec(lo[d]), e = (double)tile_dec(hi[d]) - l;
    if (a.ext < 0.0 || e > a.ext) a = TileAxis{d, l, e};
  }
  return a;
}

// Key of a node within its segment.
__device__ inline uint64_t tile_key(const TileAxis& a, float c, int node) {
  const double qmax = (double)((1u << kTileCoordBits) - 1);
  const uint64_t q = a.ext > 0.0 ? (uint64_t)fmin(fmax(((double)c - a.lo) / a.ext * qmax, 0.0), qmax) : 0;
  return (q << kTileNodeBits) | (uint64_t)node;
}

// One level of the bisection for segments larger than kTileLocal: workgroup s
// puts the nodes of segment s whose keys are among the m smallest (m = slots
// of its left half) into the left half of perm, the others into the right.
// Four passes over the segment, bound by one compute unit's loads (one
// workgroup per segment; 70 us for 65536 slots with 8 loads in flight per
// thread, 106 us with the loads left to the loop, 14 us for 1024): bounding box, keys with a histogram of their top digit, the
// candidates of the median's digit, partition.  The median is then ranked
// among the candidates in LDS; a digit that more than kTileCand keys share
// (many equal coordinates) is refined by the next one, down to the node index.
// keys: n entries of scratch.  first: perm is still the identity (level 0).
constexpr int kTileCand = 1024;
__global__ __launch_bounds__(kTileThreads) void k_tile_split(const float4* __restrict__ src, int64_t n, int l, int first,
                                                             uint64_t* __restrict__ keys, int* __restrict__ perm) {
  constexpr int kBins = 4096;
  constexpr int kBatch = 8;      // loads in flight per thread
  // digits of the 46-bit key from the top: their low bits and widths
  constexpr int kDigits = 4;
  constexpr int kLow[kDigits] = {34, 22, 11, 0}, kWidth[kDigits] = {12, 12, 11, 11};
  __shared__ uint32_t lo[3], hi[3];
  __shared__ uint32_t hist[kBins];
  __shared__ uint64_t cand[kTileCand];
  __shared__ uint32_t wsum[kTileThreads / 64];
  __shared__ uint32_t sel_bin, sel_below, count, left, right;
  __shared__ uint64_t median;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t nb = ceil_div(n, kTileLeaf);
  const int64_t seg = blockIdx.x;
  const int64_t s0 = tile_seg_start(seg, l, nb, n), s1 = tile_seg_start(seg + 1, l, nb, n);
  const int64_t mid = tile_seg_start(2 * seg + 1, l + 1, nb, n);
  if (tid < 3) {
    lo[tid] = 0xffffffffu;
    hi[tid] = 0u;
  }
  if (tid == 0) left = right = count = 0;
  __syncthreads();
  {
    uint32_t bl[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, bh[3] = {0u, 0u, 0u};
    for (int64_t b0 = s0 + tid; b0 < s1; b0 += kBatch * kTileThreads) {
      float4 p[kBatch];
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const int64_t s = min(b0 + e * kTileThreads, s1 - 1);   // past the end: the last node again
        p[e] = src[first ? s : perm[s]];
      }
#pragma unroll
      for (int e = 0; e < kBatch; ++e) {
        const float c[3] = {p[e].x, p[e].y, p[e].z};
#pragma unroll
        for (int d = 0; d < 3; ++d)
          if (c[d] == c[d]) {
            const uint32_t v = tile_enc(c[d]);
            bl[d] = min(bl[d], v);
            bh[d] = max(bh[d], v);
          }
      }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      for (int off = 32; off > 0; off >>= 1) {
        bl[d] = min(bl[d], (uint32_t)__shfl_xor((int)bl[d], off));
        bh[d] = max(bh[d], (uint32_t)__shfl_xor((int)bh[d], off));
      }
      if (lane == 0) {
        atomicMin(&lo[d], bl[d]);
        atomicMax(&hi[d], bh[d]);
      }
    }
  }
  for (int b = tid; b < kBins; b += kTileThreads) hist[b] = 0;
  __syncthreads();
  const TileAxis ax = tile_axis(lo, hi);
  const float* const axis = reinterpret_cast<const float*>(src) + ax.ax;
  for (int64_t b0 = s0 + tid; b0 < s1; b0 += kBatch * kTileThreads) {
    int nd[kBatch];
    float c[kBatch];
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      const int64_t s = min(b0 + e * kTileThreads, s1 - 1);
      nd[e] = first ? (int)s : perm[s];
      c[e] = axis[4 * (int64_t)nd[e]];
    }
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      const int64_t s = b0 + e * kTileThreads;
      if (s < s1) {
        const uint64_t k = tile_key(ax, c[e], nd[e]);
        keys[s] = k;
        atomicAdd(&hist[k >> kLow[0]], 1u);
      }
    }
  }
  // digit by digit: `prefix` holds the digits chosen so far, `rank` the
  // median's rank among the keys that share them
  uint64_t prefix = 0;
  uint32_t rank = (uint32_t)(mid - s0) - 1;
  int d = 0;
  for (;; ++d) {
    __syncthreads();
    // the bin that holds `rank`: each thread sums kBins / kTileThreads bins
    constexpr int kPer = kBins / kTileThreads;
    uint32_t mine[kPer], sum = 0;
#pragma unroll
    for (int b = 0; b < kPer; ++b) {
      mine[b] = hist[tid * kPer + b];
      sum += mine[b];
    }
    uint32_t inc = sum;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t up = (uint32_t)__shfl_up((int)inc, off);
      if (lane >= off) inc += up;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t below = inc - sum;
    for (int w = 0; w < wave; ++w) below += wsum[w];
#pragma unroll
    for (int b = 0; b < kPer; ++b) {
      if (rank >= below && rank < below + mine[b]) {
        sel_bin = (uint32_t)(tid * kPer + b);
        sel_below = below;
        count = mine[b];
      }
      below += mine[b];
    }
    __syncthreads();
    prefix = (prefix << kWidth[d]) | sel_bin;
    rank -= sel_below;
    const uint32_t c = count;
    if (c <= (uint32_t)kTileCand) break;   // the last digit leaves one key: keys are unique
    __syncthreads();
    for (int b = tid; b < kBins; b += kTileThreads) hist[b] = 0;
    __syncthreads();
    for (int64_t s = s0 + tid; s < s1; s += kTileThreads) {
      const uint64_t k = keys[s];
      if ((k >> kLow[d]) == prefix) atomicAdd(&hist[(k >> kLow[d + 1]) & ((1u << kWidth[d + 1]) - 1)], 1u);
    }
  }
  __syncthreads();
  const int ncand = (int)count;
  __syncthreads();
  if (tid == 0) count = 0;
  __syncthreads();
  for (int64_t b0 = s0 + tid; b0 < s1; b0 += kBatch * kTileThreads) {
    uint64_t k[kBatch];
#pragma unroll
    for (int e = 0; e < kBatch; ++e) k[e] = keys[min(b0 + e * kTileThreads, s1 - 1)];
#pragma unroll
    for (int e = 0; e < kBatch; ++e)
      if (b0 + e * kTileThreads < s1 && (k[e] >> kLow[d]) == prefix) cand[atomicAdd(&count, 1u)] = k[e];
  }
  __syncthreads();
  if (tid < ncand) {
    const uint64_t k = cand[tid];
    uint32_t r = 0;
    for (int j = 0; j < ncand; ++j) r += cand[j] < k ? 1u : 0u;
    if (r == rank) median = k;
  }
  __syncthreads();
  const uint64_t med = median;
  // partition; the order inside a half does not matter.  Every wave runs the
  // same number of rounds, its lanes beyond the segment masked.
  for (int64_t r0 = s0; r0 < s1; r0 += kBatch * kTileThreads) {
    uint64_t k[kBatch], ml[kBatch], mr[kBatch];
#pragma unroll
    for (int e = 0; e < kBatch; ++e) k[e] = keys[min(r0 + tid + e * kTileThreads, s1 - 1)];
    uint32_t nl = 0, nr = 0;
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      const bool in = r0 + tid + e * kTileThreads < s1;
      ml[e] = __ballot(in && k[e] <= med);
      mr[e] = __ballot(in && k[e] > med);
      nl += (uint32_t)__popcll(ml[e]);
      nr += (uint32_t)__popcll(mr[e]);
    }
    uint32_t bl = 0, br = 0;
    if (lane == 0) {
      bl = atomicAdd(&left, nl);
      br = atomicAdd(&right, nr);
    }
    bl = (uint32_t)__shfl((int)bl, 0);
    br = (uint32_t)__shfl((int)br, 0);
    const uint64_t bit = 1ull << lane;
#pragma unroll
    for (int e = 0; e < kBatch; ++e) {
      const int node = (int)(k[e] & ((1ull << kTileNodeBits) - 1));
      if (ml[e] & bit) perm[s0 + bl + __popcll(ml[e] & (bit - 1))] = node;
      if (mr[e] & bit) perm[mid + br + __popcll(mr[e] & (bit - 1))] = node;
      bl += (uint32_t)__popcll(ml[e]);
      br += (uint32_t)__popcll(mr[e]);
    }
  }
}

// The remaining levels l0 .. L - 1 of the segment `blockIdx.x` of level l0 (at
// most kTileLocal slots), in LDS: per level the boxes of its subsegments, the
// keys, and every node's place by counting the smaller keys of its subsegment
// (the lanes of a wave read the same key at once).
// first: no split level ran, perm is the identity.
__global__ __launch_bounds__(kTileLocal) void k_tile_local(const float4* __restrict__ src, int64_t n, int l0, int L,
                                                           int first, int* __restrict__ perm) {
  constexpr int kSub = kTileLocal / kTileLeaf;      // bounds the subsegments of the last level
  __shared__ float co[3][kTileLocal];               // coordinates by first place
  __shared__ int node[kTileLocal];
  __shared__ uint16_t at[2][kTileLocal];            // slot -> local index
  __shared__ uint64_t key[kTileLocal];
  __shared__ uint32_t lo[3][kSub], hi[3][kSub];
  const int64_t nb = ceil_div(n, kTileLeaf);
  const int64_t seg = blockIdx.x;
  const int64_t s0 = tile_seg_start(seg, l0, nb, n), s1 = tile_seg_start(seg + 1, l0, nb, n);
  const int m = (int)(s1 - s0);
  const int i = threadIdx.x;                        // this thread's slot
  if (i < m) {
    const int nd = first ? (int)(s0 + i) : perm[s0 + i];
    const float4 p = src[nd];
    node[i] = nd;
    co[0][i] = p.x;
    co[1][i] = p.y;
    co[2][i] = p.z;
    at[0][i] = (uint16_t)i;
  }
  int cur = 0;
  for (int l = l0; l < L; ++l) {
    const int nsub = 1 << (l - l0);                 // subsegments of this level inside the segment
    const int64_t sub0 = seg << (l - l0);
    if (i < 3 * nsub) {
      lo[i / nsub][i % nsub] = 0xffffffffu;
      hi[i / nsub][i % nsub] = 0u;
    }
    __syncthreads();
    // subsegment of slot i: block (s0 + i) / 16 lies in the largest s with floor(s nb / 2^l) <= block
    const int sb = (int)((((((s0 + i) / kTileLeaf) + 1) << l) - 1) / nb - sub0);
    const int j = i < m ? at[cur][i] : 0;
    if (i < m) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const float c = co[d][j];
        if (c == c) {
          atomicMin(&lo[d][sb], tile_enc(c));
          atomicMax(&hi[d][sb], tile_enc(c));
        }
      }
    }
    __syncthreads();
    if (i < m) {
      const uint32_t bl[3] = {lo[0][sb], lo[1][sb], lo[2][sb]}, bh[3] = {hi[0][sb], hi[1][sb], hi[2][sb]};
      const TileAxis ax = tile_axis(bl, bh);
      key[i] = tile_key(ax, co[ax.ax][j], node[j]);
    }
    __syncthreads();
    if (i < m) {
      const int a = (int)(tile_seg_start(sub0 + sb, l, nb, n) - s0), b = (int)(tile_seg_start(sub0 + sb + 1, l, nb, n) - s0);
      const uint64_t k = key[i];
      int r = 0;
#pragma unroll 8
      for (int o = a; o < b; ++o) r += key[o] < k ? 1 : 0;
      at[cur ^ 1][a + r] = (uint16_t)j;
    }
    __syncthreads();
    cur ^= 1;
  }
  if (i < m) perm[s0 + i] = node[at[cur][i]];
}

// The slots' packed coordinates and weights (padding slots keep their index).
__global__ __launch_bounds__(kWG) void k_tile_build(int64_t n, int64_t npad, const float4* __restrict__ src,
                                                    const double* __restrict__ q, int* __restrict__ perm,
                                                    float4* __restrict__ src_t, double* __restrict__ q_t) {
  const int64_t s = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (s >= npad) return;
  int64_t i = s;
  if (s < n)
    i = perm[s];
  else
    perm[s] = (int)s;
  src_t[s] = src[i];
  q_t[s] = q[i];
}

// Bounding spheres of the blocks of 32 and of 16 slots of the tile order (one
// thread each): centre (mean of
// its nodes) and a radius rounded up past every node's FP32 distance from the
// FP32 centre; blocks holding no node get radius -1.
__global__ __launch_bounds__(64) void k_tile_bounds(const float4* __restrict__ src_t, int64_t n, int64_t nb32,
                                                    int64_t nb16, float4* __restrict__ bnd32,
                                                    float4* __restrict__ bnd16) {
  int64_t b = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (b >= nb32 + nb16) return;
  const bool rows = b < nb32;
  if (!rows) b -= nb32;
  const int bs = rows ? kTileRowBlock : kTileColBlock;
  float4* const bnd = rows ? bnd32 : bnd16;
  const int64_t s0 = b * bs;
  int64_t s1 = s0 + bs;
  if (s1 > n) s1 = n;
  if (s1 <= s0) {
    bnd[b] = make_float4(0.0f, 0.0f, 0.0f, -1.0f);
    return;
  }
  double cx = 0.0, cy = 0.0, cz = 0.0;
  for (int64_t s = s0; s < s1; ++s) {
    const float4 p = src_t[s];
    cx += p.x;
    cy += p.y;
    cz += p.z;
  }
  const double inv = 1.0 / (double)(s1 - s0);
  const float fx = (float)(cx * inv), fy = (float)(cy * inv), fz = (float)(cz * inv);
  double r2 = 0.0;
  for (int64_t s = s0; s < s1; ++s) {
    const float4 p = src_t[s];
    const double dx = (double)p.x - fx, dy = (double)p.y - fy, dz = (double)p.z - fz;
    r2 = fmax(r2, dx * dx + dy * dy + dz * dz);
  }
  // relative margin covers the FP32 rounding of the centre and of the test's
  // own arithmetic
  const double r = sqrt(r2) * (1.0 + 1e-6) + 1e-6 * (1.0 + fabs((double)fx) + fabs((double)fy) + fabs((double)fz));
  bnd[b] = make_float4(fx, fy, fz, (float)r * (1.0f + 1e-6f));
}

// ut[b n + s] = u[b n + perm[s]] (states into the tile order).
__global__ __launch_bounds__(kWG) void k_tile_gather(const double* __restrict__ u, const int* __restrict__ perm,
                                                     int64_t n, int64_t total, double* __restrict__ ut) {
  const int64_t idx = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (idx >= total) return;
  const int64_t b = idx / n, s = idx - b * n;
  ut[idx] = u[b * n + perm[s]];
}

// u[b n + perm[s]] = ut[b n + s] (states back into the problem's order).
__global__ __launch_bounds__(kWG) void k_tile_scatter(const double* __restrict__ ut, const int* __restrict__ perm,
                                                      int64_t n, int64_t total, double* __restrict__ u) {
  const int64_t idx = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (idx >= total) return;
  const int64_t b = idx / n, s = idx - b * n;
  u[b * n + perm[s]] = ut[idx];
}

// Far test of the fused kernel for a target block (centre, radius) and a
// source block: every pair at distance^2 > d2far, or the source block empty.
__device__ inline bool tile_far(float4 rb, float4 cb, float d2far) {
  if (cb.w < 0.0f || rb.w < 0.0f) return true;
  const float dx = rb.x - cb.x, dy = rb.y - cb.y, dz = rb.z - cb.z;
  const float d = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx))) - rb.w - cb.w;
  return d > 0.0f && d * d > d2far;
}

// Count of (target block of kTileRowBlock, source block of kTileColBlock)
// pairs that the far test passes, over all npad / 32 x npad / 16 pairs; one
// thread per target block, counts[target block] (exact integers).
__global__ __launch_bounds__(kWG) void k_tile_far_count(const float4* __restrict__ bnd32,
                                                        const float4* __restrict__ bnd16, int64_t nrow, int64_t ncol,
                                                        float d2far, int64_t* __restrict__ counts) {
  const int64_t r = (int64_t)blockIdx.x * kWG + threadIdx.x;
  if (r >= nrow) return;
  const float4 rb = bnd32[r];
  int64_t c = 0;
  for (int64_t j = 0; j < ncol; ++j) c += tile_far(rb, bnd16[j], d2far) ? 1 : 0;
  counts[r] = c;
}

}  // namespace nfr
