// knn.hip — exact k nearest neighbours of isosurface points (the plain
// initialisation sets each Gaussian's scale from its 3 nearest neighbours;
// the learned initialisation reads 16-NN features).
//
// Device pipeline (sizes that depend on the data stay on the device):
//   k_bbox_partial / k_grid_params   bounding box -> uniform grid whose cell
//                                    edge suits the points' occupancy
//   k_cell_zero, k_cell_count        cell of each point, its rank there and
//                                    the per-cell counts
//   k_knn_scan_*                     exclusive scan of the counts
//   k_cell_scatter                   points grouped by cell (float4 x,y,z,id)
//   k_query                          one thread per point, in cell order for
//                                    cache locality: the 3x3x3 box around the
//                                    point's cell, then growing Chebyshev
//                                    shells of cells, until the k-th best
//                                    distance is within the distance to the
//                                    searched box (exact); the K best
//                                    (distance^2, index) pairs stay sorted in
//                                    registers, ties broken by index.
//   k_query_far                      a wave for each point whose neighbours
//                                    are beyond those shells: shells of blocks
//                                    of cells.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "gs_device.h"

namespace gsmi {

constexpr int kKnnThreads = 256;
constexpr int kKnnScanPer = 8;
constexpr int kBlockShift = 2, kBlock = 1 << kBlockShift;   // cells per block edge
constexpr int kKnnScanItems = kKnnThreads * kKnnScanPer;

struct GridParams {
  float lo[3];
  float h, inv_h;
  int g[3];
  int bg[3];            // blocks of kBlock^3 cells per axis
  int64_t n_cells, n_blocks;
  uint32_t n_far;       // points left to k_query_far
};

static inline size_t a256(size_t x) { return (x + 255) & ~size_t(255); }

// Sample points for the choice of the grid: of the array's 256-point spans
// every `span`-th gives those of its points whose place is a multiple of
// 1 << shift, at most kSample in all.  Written together by the blocks that
// read them (a work-group gathering them afterwards took 35 us).
constexpr int kSample = 8192;

struct KnnSample {
  uint32_t span;
  int shift;
};

static KnnSample knn_sample(int64_t nb_pts) {
  KnnSample S{1u, 8};
  if (nb_pts >= kSample) S.span = (uint32_t)ceil_div(nb_pts, kSample);
  else
    while (S.shift > 0 && nb_pts << (8 - S.shift + 1) <= kSample) --S.shift;
  return S;
}

// Cells per point that the grid may have.  Isosurface points fill few of a
// volume's cells: with one cell per point 4M points of a closed surface put
// 60 into each occupied cell, and a query compared some 600 of them.  16
// cells per point (64 bytes of counts) leave 10 there: the 16-NN search of
// those points took 22.2 ms, and takes 1.48 ms (250 us more for the larger
// table); 1M points of a volume 5.4 -> 0.67 ms.
constexpr int64_t kCellsPerPoint = 16;
constexpr int64_t kMaxBboxBlocks = 1024;

struct KnnLayout {
  int64_t max_cells, nb_pts, nb_bbox, nb_scan;
  size_t off_part, off_sample, off_params, off_cell, off_rank, off_count, off_block, off_sorted, off_bsum,
      total;
};

static KnnLayout knn_layout(int64_t n) {
  KnnLayout L;
  const int64_t m = n > 0 ? n : 1;
  L.max_cells = std::min<int64_t>(kCellsPerPoint * m + 1024, int64_t(1) << 31);
  L.nb_pts = ceil_div(m, kKnnThreads);
  L.nb_bbox = std::min(L.nb_pts, kMaxBboxBlocks);
  L.nb_scan = ceil_div(L.max_cells + 1, kKnnScanItems);
  size_t o = 0;
  L.off_part = o; o += a256(sizeof(float) * 6 * (size_t)L.nb_bbox);
  L.off_sample = o; o += a256(sizeof(float) * 3 * kSample);
  L.off_params = o; o += a256(sizeof(GridParams));
  L.off_cell = o; o += a256(sizeof(uint32_t) * (size_t)m);
  L.off_rank = o; o += a256(sizeof(uint32_t) * (size_t)m);
  L.off_count = o; o += a256(sizeof(uint32_t) * (size_t)(L.max_cells + 1));
  // (thin grids have up to a block per kBlock cells)
  L.off_block = o; o += a256((size_t)(L.max_cells / kBlock + 1024));
  L.off_sorted = o; o += a256(sizeof(float4) * (size_t)m);
  L.off_bsum = o; o += a256(sizeof(uint32_t) * (size_t)L.nb_scan);
  L.total = o;
  return L;
}

// Block bounding boxes part[block][6] and the sample [3][kSample] (NaN past
// the last point).
__global__ __launch_bounds__(kKnnThreads) void k_bbox_partial(const float* __restrict__ pts,
                                                              int64_t n, KnnSample smp,
                                                              float* __restrict__ part,
                                                              float* __restrict__ sample) {
  __shared__ float sm[6][kKnnThreads / 64];
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int64_t u = blockIdx.x; u * kKnnThreads < n; u += gridDim.x) {
    const int64_t i = u * kKnnThreads + threadIdx.x;
    const uint32_t su = (uint32_t)u / smp.span;
    const bool take = su * smp.span == (uint32_t)u && (threadIdx.x & ((1u << smp.shift) - 1)) == 0;
    const uint32_t slot = (su << (8 - smp.shift)) + (threadIdx.x >> smp.shift);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float x = i < n ? pts[a * n + i] : __builtin_nanf("");
      v[a] = fminf(v[a], x);
      v[3 + a] = fmaxf(v[3 + a], x);
      if (take) sample[a * kSample + slot] = x;
    }
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], __shfl_xor(v[a], d, 64));
      v[3 + a] = fmaxf(v[3 + a], __shfl_xor(v[3 + a], d, 64));
    }
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int a = 0; a < 6; ++a) sm[a][threadIdx.x >> 6] = v[a];
  __syncthreads();
  if (threadIdx.x < 6) {
    const int a = threadIdx.x;
    float r = sm[a][0];
    for (int w = 1; w < kKnnThreads / 64; ++w) r = a < 3 ? fminf(r, sm[a][w]) : fmaxf(r, sm[a][w]);
    part[(int64_t)blockIdx.x * 6 + a] = r;
  }
}

__device__ __forceinline__ int cell_coord(float x, float lo, float inv_h, int g) {
  return min(max((int)floorf((x - lo) * inv_h), 0), g - 1);
}

// Sets the grid's edge and dimensions (at most max_cells cells) for a wanted
// edge h.
__device__ __forceinline__ void grid_dims(const float (&ext)[3], float h, int64_t max_cells,
                                          GridParams& G) {
  for (int it = 0; it < 64; ++it) {
    int64_t cells = 1;
    for (int a = 0; a < 3; ++a) {
      G.g[a] = max(1, (int)ceilf(ext[a] / h) + 1);
      cells *= G.g[a];
    }
    if (cells <= max_cells) break;
    h *= 1.25f;
  }
  G.h = h;
  G.inv_h = 1.0f / h;
  G.n_cells = (int64_t)G.g[0] * G.g[1] * G.g[2];
  for (int a = 0; a < 3; ++a) G.bg[a] = ((G.g[a] - 1) >> kBlockShift) + 1;
  G.n_blocks = (int64_t)G.bg[0] * G.bg[1] * G.bg[2];
}

// One work-group: bounding box of the block boxes, then the grid.  A grid of
// one cell per point suits points that fill the volume.  How the points lie
// is measured on the sample (ns points, NaN ones aside): with h0 the edge of a
// grid of one cell per sample point, N2 and N4 cells of edge 2 h0 and 4 h0
// hold points.  In a volume N2 / N4 is near 8; where it is near 4 the points
// lie on a surface, the number of occupied cells grows as 1 / h^2, and the
// edge is taken that gives `per_cell` points of all n to an occupied cell.
// (The search is exact for any edge.)
constexpr float kSurfaceRatio = 5.5f;
constexpr int kParamThreads = 1024;

__global__ __launch_bounds__(kParamThreads) void k_grid_params(
    const float* __restrict__ part, int64_t nb, const float* __restrict__ sample, int ns, int64_t n,
    int64_t max_cells, float per_cell, GridParams* __restrict__ P) {
  constexpr int kWords = (kSample + 1024) / 32;
  __shared__ float sm[6][kParamThreads / 64];
  __shared__ uint32_t bits[2][kWords];
  __shared__ GridParams G;
  __shared__ float s_ext[3];
  __shared__ int occupied[2];
  const int t = threadIdx.x;
  float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
  for (int64_t b = t; b < nb; b += kParamThreads)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], part[b * 6 + a]);
      v[3 + a] = fmaxf(v[3 + a], part[b * 6 + 3 + a]);
    }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = fminf(v[a], __shfl_xor(v[a], d, 64));
      v[3 + a] = fmaxf(v[3 + a], __shfl_xor(v[3 + a], d, 64));
    }
  if ((t & 63) == 0)
#pragma unroll
    for (int a = 0; a < 6; ++a) sm[a][t >> 6] = v[a];
  for (int i = t; i < kWords; i += kParamThreads) bits[0][i] = bits[1][i] = 0u;
  constexpr int kPer = kSample / kParamThreads;
  float sx[kPer], sy[kPer], sz[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int k = min(t + q * kParamThreads, ns - 1);
    sx[q] = sample[k];
    sy[q] = sample[kSample + k];
    sz[q] = sample[2 * kSample + k];
  }
  __syncthreads();
  float vol = 1.0f, emax = 0.0f;
  if (t == 0) {
    for (int a = 0; a < 3; ++a) {
      float lo = sm[a][0], hi = sm[3 + a][0];
      for (int w = 1; w < kParamThreads / 64; ++w) {
        lo = fminf(lo, sm[a][w]);
        hi = fmaxf(hi, sm[3 + a][w]);
      }
      G.lo[a] = lo;
      s_ext[a] = fmaxf(hi - lo, 0.0f);
      emax = fmaxf(emax, s_ext[a]);
    }
    if (!(emax > 0.0f)) emax = 1.0f;
    for (int a = 0; a < 3; ++a) vol *= fmaxf(s_ext[a], emax * 1e-3f);
    const float ext[3] = {s_ext[0], s_ext[1], s_ext[2]};
    grid_dims(ext, fmaxf(cbrtf(vol / (float)ns), emax * 1e-6f), kSample, G);
    occupied[0] = occupied[1] = 0;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    if (t + q * kParamThreads >= ns || !(sx[q] == sx[q])) continue;
    const int cx = cell_coord(sx[q], G.lo[0], G.inv_h, G.g[0]);
    const int cy = cell_coord(sy[q], G.lo[1], G.inv_h, G.g[1]);
    const int cz = cell_coord(sz[q], G.lo[2], G.inv_h, G.g[2]);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int s = e + 1, gx = ((G.g[0] - 1) >> s) + 1, gy = ((G.g[1] - 1) >> s) + 1;
      const int c = ((cz >> s) * gy + (cy >> s)) * gx + (cx >> s);
      atomicOr(&bits[e][c >> 5], 1u << (c & 31));
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    int occ = 0;
    for (int i = t; i < kWords; i += kParamThreads) occ += __popc(bits[e][i]);
    if (occ) atomicAdd(&occupied[e], occ);
  }
  __syncthreads();
  if (t == 0) {
    const float ext[3] = {s_ext[0], s_ext[1], s_ext[2]};
    const float n2 = (float)occupied[0], n4 = (float)occupied[1];
    float h = cbrtf(vol / (float)n);                            // one cell per point
    if (n2 < kSurfaceRatio * n4)
      h = fminf(h, fmaxf(2.0f * G.h * sqrtf(per_cell * n2 / (float)n),
                         cbrtf(vol / ((float)max_cells * 0.8f))));
    grid_dims(ext, fmaxf(h, emax * 1e-6f), max_cells, G);
    G.n_far = 0;
    *P = G;
  }
}

// Clears the counts of the grid's cells and the entry that closes the last
// one, and the blocks' marks.
__global__ __launch_bounds__(kKnnThreads) void k_cell_zero(const GridParams* __restrict__ P,
                                                           uint4* __restrict__ count,
                                                           uint4* __restrict__ block) {
  const int64_t words = (P->n_cells + 1 + 3) / 4, bwords = (P->n_blocks + 15) / 16;
  const int64_t i0 = (int64_t)blockIdx.x * kKnnThreads + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * kKnnThreads;
  for (int64_t i = i0; i < words; i += step) count[i] = make_uint4(0u, 0u, 0u, 0u);
  for (int64_t i = i0; i < bwords; i += step) block[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(kKnnThreads) void k_cell_count(const float* __restrict__ pts, int64_t n,
                                                            const GridParams* __restrict__ P,
                                                            uint32_t* __restrict__ cell,
                                                            uint32_t* __restrict__ rank,
                                                            uint32_t* __restrict__ count,
                                                            uint8_t* __restrict__ block) {
  const int64_t i = (int64_t)blockIdx.x * kKnnThreads + threadIdx.x;
  if (i >= n) return;
  const GridParams G = *P;
  const int cx = cell_coord(pts[i], G.lo[0], G.inv_h, G.g[0]);
  const int cy = cell_coord(pts[n + i], G.lo[1], G.inv_h, G.g[1]);
  const int cz = cell_coord(pts[2 * n + i], G.lo[2], G.inv_h, G.g[2]);
  const uint32_t c = (uint32_t)(((int64_t)cz * G.g[1] + cy) * G.g[0] + cx);
  cell[i] = c;
  const uint32_t r = atomicAdd(&count[c], 1u);
  rank[i] = r;
  // (the first point of a cell marks its block; equal stores may race)
  if (r == 0u)
    block[((int64_t)(cz >> kBlockShift) * G.bg[1] + (cy >> kBlockShift)) * G.bg[0] +
          (cx >> kBlockShift)] = 1;
}

// exclusive scan of count[0 .. n_cells] (n_cells read from P) in place; the
// extra entry (zero before the scan) becomes n and closes the last cell.
// Blocks past the grid's cells return at once.
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = __shfl_up(v, d, 64);
    if ((int)(threadIdx.x & 63) >= d) v += u;
  }
  return v;
}

// Exclusive prefix over the block's threads; total in every thread.
template <int THREADS>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* sm, uint32_t& total) {
  const int w = threadIdx.x >> 6;
  const uint32_t inc = wave_scan(v);
  if ((threadIdx.x & 63) == 63) sm[w] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < THREADS / 64; ++k) {
    if (k < w) base += sm[k];
    tot += sm[k];
  }
  __syncthreads();
  total = tot;
  return base + inc - v;
}

// A thread's kKnnScanPer consecutive counts (0 past nc), as 16-byte words.
__device__ __forceinline__ void load_counts(const uint32_t* __restrict__ count, int64_t i0,
                                            int64_t nc, uint32_t (&v)[kKnnScanPer]) {
#pragma unroll
  for (int q = 0; q < kKnnScanPer / 4; ++q) {
    uint4 w = make_uint4(0u, 0u, 0u, 0u);
    if (i0 + 4 * q < nc) w = *reinterpret_cast<const uint4*>(count + i0 + 4 * q);
    v[4 * q] = w.x;
    v[4 * q + 1] = w.y;
    v[4 * q + 2] = w.z;
    v[4 * q + 3] = w.w;
  }
#pragma unroll
  for (int k = 0; k < kKnnScanPer; ++k)
    if (i0 + k >= nc) v[k] = 0u;
}

__global__ __launch_bounds__(kKnnThreads) void k_knn_scan_reduce(const uint32_t* __restrict__ count,
                                                                 const GridParams* __restrict__ P,
                                                                 uint32_t* __restrict__ bsum) {
  __shared__ uint32_t sm[kKnnThreads / 64];
  const int64_t nc = P->n_cells + 1;
  const int64_t base = (int64_t)blockIdx.x * kKnnScanItems;
  if (base >= nc) return;
  uint32_t v[kKnnScanPer], s = 0, total;
  load_counts(count, base + threadIdx.x * kKnnScanPer, nc, v);
#pragma unroll
  for (int k = 0; k < kKnnScanPer; ++k) s += v[k];
  block_scan<kKnnThreads>(s, sm, total);
  if (threadIdx.x == 0) bsum[blockIdx.x] = total;
}

constexpr int kTopThreads = 1024;

__global__ __launch_bounds__(kTopThreads) void k_knn_scan_top(const GridParams* __restrict__ P,
                                                              uint32_t* __restrict__ bsum) {
  __shared__ uint32_t sm[kTopThreads / 64];
  const int64_t nb = (P->n_cells + 1 + kKnnScanItems - 1) / kKnnScanItems;
  uint32_t carry = 0;
  for (int64_t b0 = 0; b0 < nb; b0 += kTopThreads) {
    const int64_t b = b0 + threadIdx.x;
    const uint32_t x = b < nb ? bsum[b] : 0u;
    uint32_t total;
    const uint32_t ex = block_scan<kTopThreads>(x, sm, total);
    if (b < nb) bsum[b] = carry + ex;
    carry += total;
  }
}

__global__ __launch_bounds__(kKnnThreads) void k_knn_scan_down(uint32_t* __restrict__ count,
                                                               const GridParams* __restrict__ P,
                                                               const uint32_t* __restrict__ bsum) {
  __shared__ uint32_t sm[kKnnThreads / 64];
  const int64_t nc = P->n_cells + 1;
  const int64_t base = (int64_t)blockIdx.x * kKnnScanItems;
  if (base >= nc) return;
  const int64_t i0 = base + threadIdx.x * kKnnScanPer;
  uint32_t v[kKnnScanPer], s = 0, total;
  load_counts(count, i0, nc, v);
#pragma unroll
  for (int k = 0; k < kKnnScanPer; ++k) s += v[k];
  uint32_t run = bsum[blockIdx.x] + block_scan<kKnnThreads>(s, sm, total);
#pragma unroll
  for (int k = 0; k < kKnnScanPer; ++k) {
    const uint32_t x = v[k];
    v[k] = run;
    run += x;
  }
  // (the words past nc lie inside the 256-byte padded array)
#pragma unroll
  for (int q = 0; q < kKnnScanPer / 4; ++q)
    if (i0 + 4 * q < nc)
      *reinterpret_cast<uint4*>(count + i0 + 4 * q) =
          make_uint4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
}

__global__ __launch_bounds__(kKnnThreads) void k_cell_scatter(const float* __restrict__ pts, int64_t n,
                                                              const uint32_t* __restrict__ cell,
                                                              const uint32_t* __restrict__ rank,
                                                              const uint32_t* __restrict__ start,
                                                              float4* __restrict__ sorted) {
  const int64_t i = (int64_t)blockIdx.x * kKnnThreads + threadIdx.x;
  if (i >= n) return;
  sorted[start[cell[i]] + rank[i]] = make_float4(pts[i], pts[n + i], pts[2 * n + i], __int_as_float((int)i));
}

// The K best (distance^2, index) pairs, ascending, as 64-bit keys: distances
// are not negative, so their bits order as they do.
__device__ __forceinline__ uint64_t knn_key(float d2, int j) {
  return ((uint64_t)__float_as_uint(d2) << 32) | (uint32_t)j;
}
constexpr uint64_t kNoNeighbour = ((uint64_t)0x7f800000u << 32) | 0x7fffffffu;

// Puts a key that beats the K-th into place: entry s becomes the median of
// its predecessor, itself and the key (a compare and four selects; swapping
// pairs of distances and indices took twice that).
template <int K>
__device__ __forceinline__ void knn_insert(uint64_t (&best)[K], uint64_t key) {
  if (!(key < best[K - 1])) return;
  bool below = true;                                // key < best[s]
#pragma unroll
  for (int s = K - 1; s > 0; --s) {
    const bool below_prev = key < best[s - 1];
    best[s] = below_prev ? best[s - 1] : (below ? key : best[s]);
    below = below_prev;
  }
  best[0] = below ? key : best[0];
}

// Distance^2 of the K-th neighbour found so far.
template <int K>
__device__ __forceinline__ float knn_bound(const uint64_t (&best)[K]) {
  return __uint_as_float((uint32_t)(best[K - 1] >> 32));
}

// The points of sorted positions j .. end - 1 against query q of index qi.
template <int K>
__device__ __forceinline__ void knn_scan(uint64_t (&best)[K], const float4& q, int qi,
                                         const float4* __restrict__ sorted, uint32_t j,
                                         uint32_t end) {
  for (; j < end; ++j) {
    const float4 p = sorted[j];
    const int pj = __float_as_int(p.w);
    const float dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
    const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    if (d2 <= knn_bound(best) && pj != qi) knn_insert<K>(best, knn_key(d2, pj));
  }
}

// Distance of x to the nearer of the faces of cells c0 .. c1 that have cells
// beyond them.
__device__ __forceinline__ float knn_wall(float x, float lo, float h, int g, int c0, int c1) {
  float wall = INFINITY;
  if (c0 > 0) wall = fminf(wall, x - (lo + c0 * h));
  if (c1 < g - 1) wall = fminf(wall, lo + (c1 + 1) * h - x);
  return wall;
}

// Whether the k-th distance is within `wall`, the distance to the faces of
// the searched cells: every unsearched point is beyond them.
template <int K>
__device__ __forceinline__ bool knn_done(const uint64_t (&best)[K], int k, float wall) {
  wall = fmaxf(wall, 0.0f);
  // (the k-th as the largest of the first k: a choice by k would put the
  // array in memory)
  uint32_t kth = 0;
#pragma unroll
  for (int t = 0; t < K; ++t) kth = max(kth, t < k ? (uint32_t)(best[t] >> 32) : 0u);
  return __uint_as_float(kth) <= wall * wall * 0.9999f || wall == INFINITY;
}

template <int K>
__device__ __forceinline__ void knn_write(const uint64_t (&best)[K], int qi, int k,
                                          int32_t* __restrict__ idx, float* __restrict__ dist,
                                          float* __restrict__ mean_dist) {
  float d[K], dsum = 0.0f;
  int bi[K], found = 0;
#pragma unroll
  for (int t = 0; t < K; ++t) {
    const bool has = best[t] != kNoNeighbour;
    bi[t] = has ? (int)(uint32_t)best[t] : -1;
    d[t] = sqrtf(__uint_as_float((uint32_t)(best[t] >> 32)));
    if (t < k && has) {
      dsum += d[t];
      ++found;
    }
  }
  // whole rows of 16-byte words where they fit, else one value at a time
  const int64_t o = (int64_t)qi * k;
  const bool wide = K % 4 == 0 && k == K && (((uintptr_t)idx | (uintptr_t)dist) & 15) == 0;
  if (wide) {
#pragma unroll
    for (int t = 0; t < K; t += 4) {
      if (idx)
        *reinterpret_cast<int4*>(idx + o + t) = make_int4(bi[t], bi[t + 1], bi[t + 2], bi[t + 3]);
      if (dist)
        *reinterpret_cast<float4*>(dist + o + t) = make_float4(d[t], d[t + 1], d[t + 2], d[t + 3]);
    }
  } else {
#pragma unroll
    for (int t = 0; t < K; ++t)
      if (t < k) {
        if (idx) idx[o + t] = bi[t];
        if (dist) dist[o + t] = d[t];
      }
  }
  // mean over the neighbours found, in ascending order of distance
  if (mean_dist) mean_dist[qi] = found ? dsum / (float)found : 0.0f;
}

// The rows of cells around a point, nearest first: 4 bits a row, dy + 1 and
// dz + 1.
constexpr uint64_t kRowOrder = 0xa82091645ull;

// Shells of cells searched here; a point of a surface or a volume is done by
// the second.  A point far from its neighbours would visit (2 r + 1)^3 mostly
// empty cells: it goes to the list far[0 .. P->n_far) for k_query_far.
constexpr int kFineShells = 4;

template <int K>
__global__ __launch_bounds__(kKnnThreads) void k_query(const float4* __restrict__ sorted, int64_t n,
                                                       int k, GridParams* __restrict__ P,
                                                       const uint32_t* __restrict__ start,
                                                       uint32_t* __restrict__ far,
                                                       int32_t* __restrict__ idx,
                                                       float* __restrict__ dist,
                                                       float* __restrict__ mean_dist) {
  const int64_t s = (int64_t)blockIdx.x * kKnnThreads + threadIdx.x;
  if (s >= n) return;
  const GridParams G = *P;
  const float4 q = sorted[s];
  const int qi = __float_as_int(q.w);
  const int cx = cell_coord(q.x, G.lo[0], G.inv_h, G.g[0]);
  const int cy = cell_coord(q.y, G.lo[1], G.inv_h, G.g[1]);
  const int cz = cell_coord(q.z, G.lo[2], G.inv_h, G.g[2]);
  uint64_t best[K];
#pragma unroll
  for (int t = 0; t < K; ++t) best[t] = kNoNeighbour;
  // distance from the point to its cell's faces, less the rounding of both
  // sides of a cell boundary; a row of cells beyond a face is at least that
  // far away
  auto face = [&](float x, float lo, int c, int d) {
    if (d == 0) return 0.0f;
    const float edge = lo + (float)(d < 0 ? c : c + 1) * G.h;
    return fmaxf((d < 0 ? x - edge : edge - x) - (1e-3f * G.h + 1e-6f * fabsf(edge)), 0.0f);
  };
  // the 3x3 rows of cells around the point, its own first, so that the K-th
  // distance is small when the others are reached; rows that are farther than
  // it are left out
#pragma unroll 1
  for (int i = 0; i < 9; ++i) {
    const int dy = (int)(kRowOrder >> (4 * i) & 3) - 1;
    const int dz = (int)(kRowOrder >> (4 * i + 2) & 3) - 1;
    const int y = cy + dy, z = cz + dz;
    if (y < 0 || y >= G.g[1] || z < 0 || z >= G.g[2]) continue;
    const float fy = face(q.y, G.lo[1], cy, dy), fz = face(q.z, G.lo[2], cz, dz);
    if (fmaf(fy, fy, fz * fz) * 0.9999f > knn_bound(best)) continue;
    const int64_t row = ((int64_t)z * G.g[1] + y) * G.g[0];
    knn_scan(best, q, qi, sorted, start[row + max(cx - 1, 0)],
             start[row + min(cx + 1, G.g[0] - 1) + 1]);
  }
#pragma unroll 1
  for (int r = 1;; ++r) {
    if (r > 1) {
      for (int z = max(cz - r, 0); z <= min(cz + r, G.g[2] - 1); ++z)
        for (int y = max(cy - r, 0); y <= min(cy + r, G.g[1] - 1); ++y) {
          const int64_t row = ((int64_t)z * G.g[1] + y) * G.g[0];
          // interior rows of the shell only contribute their two end cells
          const bool whole = abs(z - cz) == r || abs(y - cy) == r;
          const int w = whole ? 2 * r : 0;
          for (int x = cx - r; x <= cx + r; x += whole ? 2 * r + 1 : 2 * r)
            if (x + w >= 0 && x < G.g[0])
              knn_scan(best, q, qi, sorted, start[row + max(x, 0)],
                       start[row + min(x + w, G.g[0] - 1) + 1]);
        }
    }
    const float wall = fminf(knn_wall(q.x, G.lo[0], G.h, G.g[0], cx - r, cx + r),
                             fminf(knn_wall(q.y, G.lo[1], G.h, G.g[1], cy - r, cy + r),
                                   knn_wall(q.z, G.lo[2], G.h, G.g[2], cz - r, cz + r)));
    if (knn_done(best, k, wall)) break;
    if (r == kFineShells) {
      far[atomicAdd(&P->n_far, 1u)] = (uint32_t)s;
      return;
    }
  }
  knn_write(best, qi, k, idx, dist, mean_dist);
}

// The points that k_query left: a wave each, over shells of blocks of cells.
// The lanes test a shell's blocks together (the empty ones and those beyond
// the k-th distance are passed over), then the points of a block, and lane t
// holds the t-th best key, which a better one moves up by a lane.  Bound by a
// point's chain of loads, some 2000 blocks for an outlier.  A thread per point
// and a wave per point, whole call: 30,000 points of a normal distribution,
// k = 3 939 -> 218 us, k = 16 1720 -> 432; 300,007 of a long-tailed one, k = 16
// 253 -> 87 ms; but where tens of thousands of points are left, a thread each
// fills the chip (300,007 of a square, k = 32 732 -> 1019 us).
__global__ __launch_bounds__(kKnnThreads) void k_query_far(
    const float4* __restrict__ sorted, int k, const GridParams* __restrict__ P,
    const uint32_t* __restrict__ start, const uint8_t* __restrict__ block,
    const uint32_t* __restrict__ far, int32_t* __restrict__ idx, float* __restrict__ dist,
    float* __restrict__ mean_dist) {
  const GridParams G = *P;
  const int lane = threadIdx.x & 63;
  auto slab = [&](float x, float lo, int b) {
    const float e0 = lo + (float)(b * kBlock) * G.h, e1 = e0 + (float)kBlock * G.h;
    const float d = fmaxf(e0 - x, x - e1);
    return fmaxf(d - (1e-3f * G.h + 1e-6f * (fabsf(e0) + fabsf(e1))), 0.0f);
  };
  const uint32_t waves = gridDim.x * (kKnnThreads / 64);
  for (uint32_t i = blockIdx.x * (kKnnThreads / 64) + (threadIdx.x >> 6); i < G.n_far; i += waves) {
    const float4 q = sorted[far[i]];
    const int qi = __float_as_int(q.w);
    const int bx = cell_coord(q.x, G.lo[0], G.inv_h, G.g[0]) >> kBlockShift;
    const int by = cell_coord(q.y, G.lo[1], G.inv_h, G.g[1]) >> kBlockShift;
    const int bz = cell_coord(q.z, G.lo[2], G.inv_h, G.g[2]) >> kBlockShift;
    uint64_t best = kNoNeighbour;
    uint64_t kth = kNoNeighbour;              // lane k - 1's
    auto visit = [&](int x, int y, int z) {   // the points of a block
      const int x0 = x * kBlock, x1 = min(x0 + kBlock, G.g[0]);
      // the start and end of row l of its kBlock^2 rows of cells, in lane l
      const int cy = y * kBlock + (lane & (kBlock - 1)), cz = z * kBlock + (lane >> kBlockShift);
      uint32_t r0 = 0, r1 = 0;
      if (lane < kBlock * kBlock && cy < G.g[1] && cz < G.g[2]) {
        const int64_t row = ((int64_t)cz * G.g[1] + cy) * G.g[0];
        r0 = start[row + x0];
        r1 = start[row + x1];
      }
      for (uint64_t rows = __ballot(r1 > r0); rows; rows &= rows - 1) {
        const int l = (int)__builtin_ctzll(rows);
        const uint32_t j0 = __builtin_amdgcn_readlane(r0, l), j1 = __builtin_amdgcn_readlane(r1, l);
        for (uint32_t j = j0; j < j1; j += 64) {
          uint64_t key = kNoNeighbour;
          if (j + lane < j1) {
            const float4 p = sorted[j + lane];
            const int pj = __float_as_int(p.w);
            const float dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
            const float d2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
            if (d2 <= INFINITY && pj != qi) key = knn_key(d2, pj);
          }
          for (uint64_t todo = __ballot(key < kth); todo; todo &= todo - 1) {
            const int c = (int)__builtin_ctzll(todo);
            const uint64_t n = __shfl(key, c, 64);
            if (n >= kth) continue;           // one before it moved the k-th below it
            const uint64_t below = __shfl_up(best, 1, 64);
            if (n < best) best = lane > 0 && n < below ? below : n;
            kth = __shfl(best, k - 1, 64);
          }
        }
      }
    };
    // the blocks [xa, xb] x [ya, yb] x [za, zb] of the grid, one of the three
    // ranges a single block
    auto face = [&](int xa, int xb, int ya, int yb, int za, int zb) {
      const int nx = xb - xa + 1, ny = yb - ya + 1, nz = zb - za + 1;
      if (nx <= 0 || ny <= 0 || nz <= 0) return;
      const int64_t blocks = (int64_t)nx * ny * nz;
      for (int64_t b0 = 0; b0 < blocks; b0 += 64) {
        const uint32_t f = (uint32_t)min(b0 + lane, blocks - 1);
        const int x = xa + (int)(f % nx), y = ya + (int)(f / nx % ny), z = za + (int)(f / nx / ny);
        const bool hit = b0 + lane < blocks &&
                         block[((int64_t)z * G.bg[1] + y) * G.bg[0] + x] != 0;
        const float fx = slab(q.x, G.lo[0], x), fy = slab(q.y, G.lo[1], y),
                    fz = slab(q.z, G.lo[2], z);
        const float reach = fmaf(fx, fx, fmaf(fy, fy, fz * fz)) * 0.9999f;
        for (uint64_t todo = __ballot(hit); todo; todo &= todo - 1) {
          const int c = (int)__builtin_ctzll(todo);
          if (__shfl(reach, c, 64) > __uint_as_float((uint32_t)(kth >> 32))) continue;
          visit(__builtin_amdgcn_readlane(x, c), __builtin_amdgcn_readlane(y, c),
                __builtin_amdgcn_readlane(z, c));
        }
      }
    };
#pragma unroll 1
    for (int r = 0;; ++r) {
      // the shell of blocks at Chebyshev distance r, face by face
      const int x0 = max(bx - r, 0), x1 = min(bx + r, G.bg[0] - 1);
      const int y0 = max(by - r, 0), y1 = min(by + r, G.bg[1] - 1);
      const int yi0 = max(by - r + 1, 0), yi1 = min(by + r - 1, G.bg[1] - 1);
      const int zi0 = max(bz - r + 1, 0), zi1 = min(bz + r - 1, G.bg[2] - 1);
#pragma unroll 1
      for (int f = 0; f < (r ? 6 : 1); ++f) {
        const int d = f & 1 ? r : -r;
        const bool fz = f < 2, fy = f >= 2 && f < 4, fx = f >= 4;
        const int at = fz ? bz + d : (fy ? by + d : bx + d);
        if (at < 0 || at >= (fz ? G.bg[2] : (fy ? G.bg[1] : G.bg[0]))) continue;
        face(fx ? at : x0, fx ? at : x1, fy ? at : (fx ? yi0 : y0), fy ? at : (fx ? yi1 : y1),
             fz ? at : zi0, fz ? at : zi1);
      }
      const int r1 = r + 1;
      const float wall = fmaxf(fminf(
          knn_wall(q.x, G.lo[0], G.h, G.g[0], (bx - r) * kBlock, (bx + r1) * kBlock - 1),
          fminf(knn_wall(q.y, G.lo[1], G.h, G.g[1], (by - r) * kBlock, (by + r1) * kBlock - 1),
                knn_wall(q.z, G.lo[2], G.h, G.g[2], (bz - r) * kBlock, (bz + r1) * kBlock - 1))), 0.0f);
      // (true once the whole grid is searched)
      if (__uint_as_float((uint32_t)(kth >> 32)) <= wall * wall * 0.9999f || wall == INFINITY) break;
    }
    const bool has = best != kNoNeighbour;
    const float d = sqrtf(__uint_as_float((uint32_t)(best >> 32)));
    if (lane < k) {
      const int64_t o = (int64_t)qi * k + lane;
      if (idx) idx[o] = has ? (int)(uint32_t)best : -1;
      if (dist) dist[o] = d;
    }
    if (mean_dist) {                          // nearest first
      const int found = (int)__builtin_popcountll(__ballot(lane < k && has));
      float sum = 0.0f;
      for (int t = 0; t < found; ++t) sum += lane_f(d, t);
      if (lane == 0) mean_dist[qi] = found ? sum / (float)found : 0.0f;
    }
  }
}

// Plain initialisation of the Gaussians of surface points (one thread per
// point): mean = point, colour coefficient sqrt(pi) n (so that the degree-0
// colour max(0, C0 f + 1/2) is (n + 1)/2), and, when the k-NN mean distances
// d are given, an isotropic log-scale log(max(d, 1e-6)), the identity
// rotation and a fixed opacity logit.
__global__ __launch_bounds__(kKnnThreads) void k_plain_init(
    const float* __restrict__ pts, const float* __restrict__ nrm, int64_t n,
    const float* __restrict__ d, float logit, float* __restrict__ mean,
    float* __restrict__ log_scale, float* __restrict__ quat, float* __restrict__ opacity_logit,
    float* __restrict__ color) {
  const int64_t i = (int64_t)blockIdx.x * kKnnThreads + threadIdx.x;
  if (i >= n) return;
  const float kSqrtPi = 1.7724538509055160f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    mean[a * n + i] = pts[a * n + i];
    color[a * n + i] = kSqrtPi * nrm[a * n + i];
  }
  if (!d) return;
  const float ls = logf(fmaxf(d[i], 1e-6f));
#pragma unroll
  for (int a = 0; a < 3; ++a) log_scale[a * n + i] = ls;
  quat[i] = 1.0f;
  quat[n + i] = quat[2 * n + i] = quat[3 * n + i] = 0.0f;
  opacity_logit[i] = logit;
}

}  // namespace gsmi

using namespace gsmi;

extern "C" {

size_t gs_knn_workspace_bytes(int64_t n, int32_t k) {
  (void)k;
  if (n < 0) return 0;
  return knn_layout(n).total;
}

gs_status gs_knn(const float* pts, int64_t n, int32_t k, void* ws, size_t ws_bytes, int32_t* idx,
                 float* dist, float* mean_dist, void* stream) {
  clear_error();
  GS_REQUIRE(k >= 1 && k <= 32, "gs_knn: k=%d outside [1, 32]", k);
  GS_REQUIRE(n >= 0 && n < (int64_t(1) << 31), "gs_knn: n=%lld outside [0, 2^31)", (long long)n);
  if (n == 0) return GS_OK;
  GS_REQUIRE(pts && ws, "gs_knn: NULL points or workspace");
  GS_REQUIRE(idx || dist || mean_dist, "gs_knn: no output requested");
  const KnnLayout L = knn_layout(n);
  GS_REQUIRE(ws_bytes >= L.total, "gs_knn: workspace %zu < required %zu", ws_bytes, L.total);
  GS_REQUIRE(((uintptr_t)ws & 255) == 0, "gs_knn: workspace must be 256-byte aligned");
  char* w = (char*)ws;
  float* part = (float*)(w + L.off_part);
  float* sample = (float*)(w + L.off_sample);
  GridParams* P = (GridParams*)(w + L.off_params);
  uint32_t* cell = (uint32_t*)(w + L.off_cell);
  uint32_t* count = (uint32_t*)(w + L.off_count);
  uint32_t* rank = (uint32_t*)(w + L.off_rank);
  uint8_t* block = (uint8_t*)(w + L.off_block);
  float4* sorted = (float4*)(w + L.off_sorted);
  uint32_t* bsum = (uint32_t*)(w + L.off_bsum);
  hipStream_t s = as_stream(stream);
  const unsigned nb = (unsigned)L.nb_pts;
  const KnnSample smp = knn_sample(L.nb_pts);
  const int ns = (int)(ceil_div(L.nb_pts, smp.span) << (8 - smp.shift));
  hipLaunchKernelGGL(k_bbox_partial, dim3((unsigned)L.nb_bbox), dim3(kKnnThreads), 0, s, pts, n,
                     smp, part, sample);
  GS_LAUNCH_CHECK("gs_knn/bbox");
  // points wanted in an occupied cell: the 3x3 cells around a surface point
  // then hold its k nearest (a disc of k points has a radius of
  // sqrt(k / (pi per_cell)) cell edges)
  const float per_cell = std::max(2.0f, (float)k / 3.0f);
  hipLaunchKernelGGL(k_grid_params, dim3(1), dim3(kParamThreads), 0, s, part, L.nb_bbox, sample,
                     ns, n, L.max_cells, per_cell, P);
  GS_LAUNCH_CHECK("gs_knn/grid");
  hipLaunchKernelGGL(k_cell_zero,
                     dim3((unsigned)std::min<int64_t>(ceil_div(L.max_cells + 4, 4 * kKnnThreads),
                                                      8 * (int64_t)device_cu_count())),
                     dim3(kKnnThreads), 0, s, P, (uint4*)count, (uint4*)block);
  GS_LAUNCH_CHECK("gs_knn/zero");
  hipLaunchKernelGGL(k_cell_count, dim3(nb), dim3(kKnnThreads), 0, s, pts, n, P, cell, rank, count,
                     block);
  GS_LAUNCH_CHECK("gs_knn/count");
  // scan n_cells + 1 entries so that start[n_cells] = n closes the last cell
  hipLaunchKernelGGL(k_knn_scan_reduce, dim3((unsigned)L.nb_scan), dim3(kKnnThreads), 0, s, count,
                     P, bsum);
  GS_LAUNCH_CHECK("gs_knn/scan_reduce");
  hipLaunchKernelGGL(k_knn_scan_top, dim3(1), dim3(kTopThreads), 0, s, P, bsum);
  GS_LAUNCH_CHECK("gs_knn/scan_top");
  hipLaunchKernelGGL(k_knn_scan_down, dim3((unsigned)L.nb_scan), dim3(kKnnThreads), 0, s, count, P,
                     bsum);
  GS_LAUNCH_CHECK("gs_knn/scan_down");
  hipLaunchKernelGGL(k_cell_scatter, dim3(nb), dim3(kKnnThreads), 0, s, pts, n, cell, rank, count,
                     sorted);
  GS_LAUNCH_CHECK("gs_knn/scatter");
  // (the cells of the points are not needed any more: their array takes the
  // list of far points)
  uint32_t* far = cell;
  const unsigned nb_far =
      (unsigned)std::min<int64_t>(ceil_div(n, kKnnThreads / 64), 8 * (int64_t)device_cu_count());
  auto query = [&](auto KK) {
    constexpr int K = decltype(KK)::value;
    hipLaunchKernelGGL(k_query<K>, dim3(nb), dim3(kKnnThreads), 0, s, sorted, n, k, P, count, far,
                       idx, dist, mean_dist);
  };
  if (k <= 4) query(std::integral_constant<int, 4>{});
  else if (k <= 8) query(std::integral_constant<int, 8>{});
  else if (k <= 16) query(std::integral_constant<int, 16>{});
  else query(std::integral_constant<int, 32>{});
  GS_LAUNCH_CHECK("gs_knn/query");
  hipLaunchKernelGGL(k_query_far, dim3(nb_far), dim3(kKnnThreads), 0, s, sorted, k, P, count,
                     block, far, idx, dist, mean_dist);
  GS_LAUNCH_CHECK("gs_knn/far");
  return GS_OK;
}

size_t gs_plain_init_workspace_bytes(int64_t n) {
  if (n < 0) return 0;
  return a256(knn_layout(n).total) + a256(sizeof(float) * (size_t)(n > 0 ? n : 1));
}

gs_status gs_plain_init(const float* pts, const float* normals, int64_t n, float opacity,
                        void* ws, size_t ws_bytes, float* mean, float* log_scale, float* quat,
                        float* opacity_logit, float* color, void* stream) {
  clear_error();
  GS_REQUIRE(n >= 0 && n < (int64_t(1) << 31), "gs_plain_init: n=%lld outside [0, 2^31)",
             (long long)n);
  if (n == 0) return GS_OK;
  GS_REQUIRE(pts && normals && mean && color, "gs_plain_init: NULL points, normals, mean or colour");
  const bool shape = log_scale != nullptr;
  GS_REQUIRE(!shape || (quat && opacity_logit && ws),
             "gs_plain_init: log_scale given without quat, opacity_logit or workspace");
  GS_REQUIRE(!shape || (opacity > 0.f && opacity < 1.f), "gs_plain_init: opacity %f outside (0, 1)",
             (double)opacity);
  float* d = nullptr;
  if (shape) {
    const size_t need = gs_plain_init_workspace_bytes(n);
    GS_REQUIRE(ws_bytes >= need, "gs_plain_init: workspace %zu < required %zu", ws_bytes, need);
    GS_REQUIRE(((uintptr_t)ws & 255) == 0, "gs_plain_init: workspace must be 256-byte aligned");
    const size_t off = a256(knn_layout(n).total);
    d = (float*)((char*)ws + off);
    gs_status st = gs_knn(pts, n, 3, ws, off, nullptr, nullptr, d, stream);
    if (st != GS_OK) return st;
  }
  const float logit = shape ? logf(opacity / (1.0f - opacity)) : 0.0f;
  hipLaunchKernelGGL(k_plain_init, dim3((unsigned)ceil_div(n, kKnnThreads)), dim3(kKnnThreads), 0,
                     as_stream(stream), pts, normals, n, d, logit, mean, log_scale, quat,
                     opacity_logit, color);
  GS_LAUNCH_CHECK("gs_plain_init");
  return GS_OK;
}

}  // extern "C"
