// Per-frame projection: grid-cell frustum culling, 1x1-pixel splat into a
// 64-bit z-buffer, and RGBDA resolve.
//
// Method, "Point Cloud Projection" and Fig. 1: the space-partitioned cloud is
// culled against the view frustum per grid cell; every surviving point is
// rasterised to a single pixel; a z-buffer resolves collisions; the result is
// RGB, depth D and a binary fill mask A.
//
// Exactness: the per-point arithmetic is float32 in a fixed order with no
// fused multiply-add (the library is built with -ffp-contract=off) and a
// correctly rounded division; the z-buffer keeps min(depth bits << 32 | index),
// which is order independent, so the image does not depend on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "lnr_internal.h"

#pragma clang fp contract(off)

namespace lnr {
namespace {

constexpr int kThreads = 256;

// Per-frame reset: the key buffer (npix words), n_counters words of the render
// counters and n_tiles words of per-tile segment counts (may be 0).
__global__ __launch_bounds__(kThreads) void clear_kernel(uint64_t *__restrict__ key, uint32_t npix,
                                                         uint32_t *__restrict__ counters, uint32_t n_counters,
                                                         uint32_t *__restrict__ tile_nseg, uint32_t n_tiles) {
  const uint32_t stride = gridDim.x * kThreads;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < npix; i += stride) key[i] = ~0ull;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n_tiles; i += stride) tile_nseg[i] = 0u;
  if (blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < n_counters; i += kThreads) counters[i] = 0;
}

// Conservative visibility of a cell's box [lo, hi] for one camera: the box is
// visible unless some half-space's maximum over it is below -slack (all in
// double, in the order below).  If visible, *bucket is the depth bucket of the
// box centre.
__device__ __attribute__((always_inline)) inline bool cell_visible(const CullParams &prm, double lo0, double lo1, double lo2, double hi0,
                                    double hi1, double hi2, int *bucket) {
  bool vis = true;
  if (!prm.no_cull) {
    const double mx0 = fmax(fabs(lo0), fabs(hi0));
    const double mx1 = fmax(fabs(lo1), fabs(hi1));
    const double mx2 = fmax(fabs(lo2), fabs(hi2));
    double S[3];
    for (int r = 0; r < 3; ++r)
      S[r] = ((prm.absP[r][0] * mx0 + prm.absP[r][1] * mx1) + prm.absP[r][2] * mx2) + prm.absP[r][3];
    const double slack = 0x1p-20 * ((S[0] + S[1]) + prm.wh1 * S[2]);
    for (int h = 0; h < 6; ++h) {
      const double *k = prm.hs[h];
      const double m =
          ((fmax(k[0] * lo0, k[0] * hi0) + fmax(k[1] * lo1, k[1] * hi1)) + fmax(k[2] * lo2, k[2] * hi2)) + k[3];
      if (m < -slack) vis = false;
    }
  }
  if (vis) {
    // camera depth of the box centre -> bucket
    const double cw = ((prm.wrow[0] * (0.5 * (lo0 + hi0)) + prm.wrow[1] * (0.5 * (lo1 + hi1))) +
                       prm.wrow[2] * (0.5 * (lo2 + hi2))) + prm.wrow[3];
    const float q = cw > prm.z_near ? kBucketsPerOctave * __log2f((float)(cw / prm.z_near)) : 0.f;
    *bucket = q >= (float)(kDepthBuckets - 1) ? kDepthBuckets - 1 : (int)q;
  }
  return vis;
}

// Queue places for this lane's nch work items in queue `bucket`: the first
// one's place within that queue.  Compaction without LDS atomics: per depth
// bucket present in the wave, a wave-wide exclusive prefix of the lanes'
// work-item counts (a ballot and a count of the set lanes below when every
// cell has at most one work item, else a shuffle scan) places each cell
// within the wave's run; the
// runs of the block's waves follow each other in wave order through LDS, and
// one global atomic per bucket and block reserves the block's run.  Every
// thread of the block calls it (block barriers).
__device__ __attribute__((always_inline)) inline uint32_t reserve_places(uint32_t nch, int bucket, uint32_t *__restrict__ counters) {
  constexpr int kWaves = kThreads / 64;
  __shared__ uint32_t s_wave[kWaves][kDepthBuckets], s_base[kDepthBuckets];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t present = nch ? (1u << bucket) : 0u;  // buckets of this wave's visible cells
  for (int off = 32; off > 0; off >>= 1) present |= __shfl_xor(present, off, 64);
  // lanes whose cell has more than one work item: with none in the wave (the
  // common case), a bucket's prefix is a ballot and a count of the lanes below
  const bool multi = __ballot(nch > 1) != 0;
  const uint64_t below = (1ull << lane) - 1ull;
  uint32_t local = 0;
  if (lane < kDepthBuckets) s_wave[wave][lane] = 0u;  // buckets absent from the wave
  // one pass per bucket present in the wave (the set is the same for every
  // lane; the loop stays rolled, which keeps this short-lived kernel small)
#pragma unroll 1
  for (uint32_t m = __builtin_amdgcn_readfirstlane(present); m; m &= m - 1) {
    const int b = __builtin_ctz(m);
    const uint32_t v = bucket == b ? nch : 0u;
    uint32_t tot;
    if (!multi) {
      const uint64_t bal = __ballot(v != 0);
      if (v) local = (uint32_t)__popcll(bal & below);
      tot = (uint32_t)__popcll(bal);
    } else {
      uint32_t incl = v;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
      }
      if (v) local = incl - v;
      tot = __shfl(incl, 63, 64);
    }
    if (lane == 0) s_wave[wave][b] = tot;
  }
  __syncthreads();
  if (threadIdx.x < kDepthBuckets) {
    uint32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += s_wave[w][threadIdx.x];
    s_base[threadIdx.x] = sum ? atomicAdd(&counters[4 + threadIdx.x], sum) : 0u;
  }
  __syncthreads();
  uint32_t pos = 0;
  if (nch) {
    pos = s_base[bucket] + local;
    for (int w = 0; w < wave; ++w) pos += s_wave[w][bucket];
  }
  return pos;
}

// Frame totals: work items, visible cells and their points, reduced per wave
// with one atomic per wave.
__device__ __attribute__((always_inline)) inline void add_totals(bool vis, uint32_t nch, uint32_t cnt, uint32_t *__restrict__ counters) {
  uint32_t wave_chunks = nch;
  for (int off = 32; off > 0; off >>= 1) wave_chunks += __shfl_xor(wave_chunks, off, 64);
  const uint64_t vis_mask = __ballot(vis);
  uint32_t pts = vis ? cnt : 0u;
  for (int off = 32; off > 0; off >>= 1) pts += __shfl_xor(pts, off, 64);
  if ((threadIdx.x & 63) == 0 && wave_chunks) {
    atomicAdd(&counters[0], wave_chunks);
    atomicAdd(&counters[1], (uint32_t)__popcll(vis_mask));
    atomicAdd(reinterpret_cast<unsigned long long *>(&counters[2]), (unsigned long long)pts);
  }
}

// One lane per cell.  A visible non-empty cell is cut into splat work items
// of at most `chunk` points, queued in the depth bucket of the cell's
// centre.  DEV: the camera's parameters are read from device memory (prm_dev)
// instead of the kernel arguments, so that a captured graph can be replayed
// for new cameras.
template <bool DEV>
__global__ __launch_bounds__(kThreads) void cull_kernel(const float *__restrict__ aabb,
                                                        const uint32_t *__restrict__ cell_start, uint32_t n_cells,
                                                        CullParams prm_val, const CullParams *__restrict__ prm_dev,
                                                        uint8_t *__restrict__ flags, uint2 *__restrict__ chunks,
                                                        uint32_t cap, uint32_t chunk, uint32_t *__restrict__ counters) {
  const CullParams &prm = DEV ? *prm_dev : prm_val;
  const uint32_t c = blockIdx.x * kThreads + threadIdx.x;
  uint32_t start = 0, cnt = 0;
  bool vis = false;
  int bucket = 0;
  if (c < n_cells) {
    start = cell_start[c];
    cnt = cell_start[c + 1] - start;
    if (cnt > 0)
      vis = cell_visible(prm, aabb[6ull * c + 0], aabb[6ull * c + 1], aabb[6ull * c + 2], aabb[6ull * c + 3],
                         aabb[6ull * c + 4], aabb[6ull * c + 5], &bucket);
    flags[c] = vis ? 1 : 0;
  }
  const uint32_t nch = vis ? (cnt + chunk - 1) / chunk : 0u;
  const uint32_t pos = reserve_places(nch, bucket, counters);
  for (uint32_t k = 0; k < nch; ++k) {
    const uint32_t off = k * chunk;
    chunks[(size_t)bucket * cap + pos + k] = make_uint2(start + off, min(chunk, cnt - off));
  }
  add_totals(vis, nch, cnt, counters);
}

// Several views at once (dev: their cameras in device memory, or nullptr): a
// cell is tested against every view's frustum, and
// its work items carry the mask of the views that see it (bit v = view v) and
// go to the queue of the nearest of those views' depth buckets.
__global__ __launch_bounds__(kThreads) void cull_views_kernel(const float *__restrict__ aabb,
                                                              const uint32_t *__restrict__ cell_start,
                                                              uint32_t n_cells, ViewsCull prm,
                                                              const DevCam *__restrict__ dev,
                                                              uint8_t *__restrict__ flags, uint4 *__restrict__ items,
                                                              uint32_t cap, uint32_t chunk,
                                                              uint32_t *__restrict__ counters) {
  const uint32_t c = blockIdx.x * kThreads + threadIdx.x;
  uint32_t start = 0, cnt = 0, mask = 0;
  int bucket = kDepthBuckets - 1;
  if (c < n_cells) {
    start = cell_start[c];
    cnt = cell_start[c + 1] - start;
    if (cnt > 0) {
      const double lo0 = aabb[6ull * c + 0], lo1 = aabb[6ull * c + 1], lo2 = aabb[6ull * c + 2];
      const double hi0 = aabb[6ull * c + 3], hi1 = aabb[6ull * c + 4], hi2 = aabb[6ull * c + 5];
      for (int v = 0; v < prm.n; ++v) {
        int b = 0;
        if (cell_visible(dev ? dev[v].cull : prm.v[v], lo0, lo1, lo2, hi0, hi1, hi2, &b)) {
          mask |= 1u << v;
          bucket = min(bucket, b);
        }
      }
    }
    flags[c] = mask ? 1 : 0;
  }
  const bool vis = mask != 0;
  const uint32_t nch = vis ? (cnt + chunk - 1) / chunk : 0u;
  const uint32_t pos = reserve_places(nch, bucket, counters);
  for (uint32_t k = 0; k < nch; ++k) {
    const uint32_t off = k * chunk;
    items[(size_t)bucket * cap + pos + k] = make_uint4(start + off, min(chunk, cnt - off), mask, 0u);
  }
  add_totals(vis, nch, cnt, counters);
}

// Work item `i` of the frame, walking the depth-bucket queues nearest first
// (counters[4 + b] items in bucket b); false past the last item.
template <typename Item>
__device__ inline bool work_item(uint32_t i, const uint32_t *__restrict__ counters, const Item *__restrict__ chunks,
                                 uint32_t cap, Item *ch) {
  if (i >= counters[0]) return false;
  for (int b = 0; b < kDepthBuckets; ++b) {
    const uint32_t nb = counters[4 + b];
    if (i < nb) {
      *ch = chunks[(size_t)b * cap + i];
      return true;
    }
    i -= nb;
  }
  return false;
}

// One block per work item.  Keys only ever decrease, so a (possibly stale)
// relaxed read of the pixel's key is an upper bound of its current value and
// the atomic can be skipped when the new key is not smaller.
//
// When the work item's points fall in a screen rectangle of at most
// kDedupPx pixels, they first meet in an LDS z-buffer over that rectangle
// (LDS 64-bit atomicMin), and only the nearest point of each pixel goes on to
// the global z-buffer, in row order: dense surfaces (many points per pixel)
// then cost one coalesced early-out read, and at most one atomic, per pixel
// instead of per point.  A work item spread over a larger rectangle (a near
// surface, few points per pixel) takes the per-point path.  The minimum is the
// same either way.
//
// COUNT adds the number of global atomics issued to counters[kAtomicWord]
// (one add per wave), for measurement; the keys written are the same.
constexpr int kDedupPx = 4096;
constexpr int kPtsPerThread = kSplatChunk / kThreads;
static_assert(kSplatChunk % kThreads == 0, "work items must split evenly over the threads");

template <bool COUNT>
__device__ inline void global_min(uint64_t *dst, uint64_t k, uint32_t &issued) {
  // relaxed atomic read: other blocks lower the word concurrently
  if (k < __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    atomicMin(reinterpret_cast<unsigned long long *>(dst), (unsigned long long)k);
    if constexpr (COUNT) ++issued;
  }
}

// floor(p / w) for 0 <= p < 4096 and 1 <= w <= 4096, by a float reciprocal:
// the quotient of p + 1/2 is at least 1/(2w) from an integer, and the two
// float roundings move it by at most (4096/w) 2^-23, which is less, so the
// truncation lands on the same integer.  inv_w = 1.0f / w.
__device__ inline uint32_t small_div(uint32_t p, float inv_w) {
  return (uint32_t)(((float)p + 0.5f) * inv_w);
}

// Point j at (x, y, z) through the camera: true if drawn, with its key
// (depth bits << 32 | j) and pixel.
__device__ __attribute__((always_inline)) inline bool project_point(float x, float y, float z, uint32_t j, const SplatCam &cam, uint64_t &k,
                                     uint32_t &px, uint32_t &py) {
  const float *P = cam.P;
  const float a = ((P[0] * x + P[1] * y) + P[2] * z) + P[3];
  const float b = ((P[4] * x + P[5] * y) + P[6] * z) + P[7];
  const float w = ((P[8] * x + P[9] * y) + P[10] * z) + P[11];
  if (w >= cam.z_near && w <= cam.z_far) {
    const float u = a / w;
    const float v = b / w;
    if (u >= 0.f && u < cam.Wf && v >= 0.f && v < cam.Hf) {
      px = (uint32_t)u;
      py = (uint32_t)v;
      k = ((uint64_t)__float_as_uint(w) << 32) | j;
      return true;
    }
  }
  return false;
}

// floor(RN(a / w)) for w > 0 and whether it lies in [0, lim): the quotient by the
// reciprocal decides unless it is within its error (below 2^-22 of its size, and
// rounding a / w moves it by half an ulp) of an integer, where the correctly
// rounded division does.  Non-finite values take the division too.
__device__ __attribute__((always_inline)) inline bool pixel_coord(float a, float w, float rw, float lim, uint32_t *p) {
  const float q = a * rw;
  float f = floorf(q);
  const float r = q - f, m = fmaxf(fabsf(q), 1.0f) * 0x1p-21f;
  if (!(r > m && r < 1.0f - m)) f = a / w;
  *p = (uint32_t)f;
  return f >= 0.f && f < lim;
}
// As project_point: the depth's bits and the pixel of a drawn point.
__device__ __attribute__((always_inline)) inline bool project_pixel(float x, float y, float z, const SplatCam &cam,
                                                                    uint32_t *wbits, uint32_t *px, uint32_t *py) {
  const float *P = cam.P;
  const float a = ((P[0] * x + P[1] * y) + P[2] * z) + P[3];
  const float b = ((P[4] * x + P[5] * y) + P[6] * z) + P[7];
  const float w = ((P[8] * x + P[9] * y) + P[10] * z) + P[11];
  *wbits = __float_as_uint(w);
  const bool in = w >= cam.z_near && w <= cam.z_far;
  const float rw = __builtin_amdgcn_rcpf(w);
  const bool inx = pixel_coord(a, w, rw, cam.Wf, px), iny = pixel_coord(b, w, rw, cam.Hf, py);
  return in & inx & iny;
}

// The block-wide rectangle of the lanes' rectangles [x0, x1] x [y0, y1]
// (x0 > x1 if none).  Contains block barriers.
__device__ __attribute__((always_inline)) inline void block_rect(uint32_t x0, uint32_t y0, uint32_t x1, uint32_t y1, uint32_t *s_bb, uint32_t *rx0,
                                  uint32_t *ry0, uint32_t *rx1, uint32_t *ry1) {
  for (int off = 32; off > 0; off >>= 1) {
    x0 = min(x0, (uint32_t)__shfl_xor(x0, off, 64));
    y0 = min(y0, (uint32_t)__shfl_xor(y0, off, 64));
    x1 = max(x1, (uint32_t)__shfl_xor(x1, off, 64));
    y1 = max(y1, (uint32_t)__shfl_xor(y1, off, 64));
  }
  if (threadIdx.x == 0) {
    s_bb[0] = ~0u;
    s_bb[1] = ~0u;
    s_bb[2] = 0;
    s_bb[3] = 0;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    atomicMin(&s_bb[0], x0);
    atomicMin(&s_bb[1], y0);
    atomicMax(&s_bb[2], x1);
    atomicMax(&s_bb[3], y1);
  }
  __syncthreads();
  *rx0 = s_bb[0];
  *ry0 = s_bb[1];
  *rx1 = s_bb[2];
  *ry1 = s_bb[3];
}

// Project the work item's points (thread t takes points t, t + 256, ...):
// kk = key, (px, py) = pixel, px = ~0u if the point is not drawn; and the
// screen rectangle [x0, x1] x [y0, y1] of the drawn points over the whole
// block (x0 > x1 if none).  Contains block barriers.
__device__ inline void project_work_item(const float *__restrict__ xs, const float *__restrict__ ys,
                                         const float *__restrict__ zs, uint2 ch, const SplatCam &cam,
                                         uint64_t (&kk)[kPtsPerThread], uint32_t (&px)[kPtsPerThread],
                                         uint32_t (&py)[kPtsPerThread], uint32_t *s_bb, uint32_t *rx0, uint32_t *ry0,
                                         uint32_t *rx1, uint32_t *ry1) {
  const int tid = threadIdx.x;
  uint32_t x0 = ~0u, y0 = ~0u, x1 = 0, y1 = 0;
#pragma unroll
  for (int q = 0; q < kPtsPerThread; ++q) {
    const uint32_t i = tid + q * kThreads;
    uint64_t k = 0;
    uint32_t ux = ~0u, uy = 0;
    if (i < ch.y) {
      const uint32_t j = ch.x + i;
      if (project_point(xs[j], ys[j], zs[j], j, cam, k, ux, uy)) {
        x0 = min(x0, ux);
        x1 = max(x1, ux);
        y0 = min(y0, uy);
        y1 = max(y1, uy);
      } else {
        ux = ~0u;
      }
    }
    kk[q] = k;
    px[q] = ux;
    py[q] = uy;
  }
  block_rect(x0, y0, x1, y1, s_bb, rx0, ry0, rx1, ry1);
}

// Lower the global z-buffer (row length W) by the block's projected points,
// whose rectangle [x0, x1] x [y0, y1] is not empty: through the LDS z-buffer
// zb over the rectangle when it has at most kDedupPx pixels, else point by
// point.  Contains block barriers.
template <bool COUNT>
__device__ __attribute__((always_inline)) inline void splat_block(const uint64_t (&kk)[kPtsPerThread], const uint32_t (&px)[kPtsPerThread],
                                   const uint32_t (&py)[kPtsPerThread], uint32_t x0, uint32_t y0, uint32_t x1,
                                   uint32_t y1, uint32_t W, uint64_t *__restrict__ key, unsigned long long *zb,
                                   uint32_t &issued) {
  const int tid = threadIdx.x;
  const uint32_t bw = x1 - x0 + 1;
  const uint64_t a64 = (uint64_t)bw * (uint64_t)(y1 - y0 + 1);
  if (a64 <= (uint64_t)kDedupPx) {
    const uint32_t area = (uint32_t)a64;
    for (uint32_t p = tid; p < area; p += kThreads) zb[p] = ~0ull;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPtsPerThread; ++q)
      if (px[q] != ~0u) atomicMin(&zb[(py[q] - y0) * bw + (px[q] - x0)], (unsigned long long)kk[q]);
    __syncthreads();
    const float inv_bw = 1.0f / (float)bw;
    for (uint32_t p = tid; p < area; p += kThreads) {
      const uint64_t k = zb[p];
      if (k == ~0ull) continue;
      const uint32_t ry = small_div(p, inv_bw), rx = p - ry * bw;
      global_min<COUNT>(key + (size_t)(y0 + ry) * W + (x0 + rx), k, issued);
    }
  } else {
#pragma unroll
    for (int q = 0; q < kPtsPerThread; ++q)
      if (px[q] != ~0u) global_min<COUNT>(key + (size_t)py[q] * W + px[q], kk[q], issued);
  }
}

template <bool COUNT>
__global__ __launch_bounds__(kThreads) void splat_kernel(const float *__restrict__ xs, const float *__restrict__ ys,
                                                         const float *__restrict__ zs, const uint2 *__restrict__ chunks,
                                                         uint32_t cap, uint32_t *__restrict__ counters,
                                                         SplatCam cam, uint64_t *__restrict__ key) {
  __shared__ unsigned long long zb[kDedupPx];
  __shared__ uint32_t s_bb[4];
  uint2 ch;
  if (!work_item(blockIdx.x, counters, chunks, cap, &ch)) return;
  uint32_t issued = 0;
  uint64_t kk[kPtsPerThread];
  uint32_t px[kPtsPerThread], py[kPtsPerThread];
  uint32_t x0, y0, x1, y1;
  project_work_item(xs, ys, zs, ch, cam, kk, px, py, s_bb, &x0, &y0, &x1, &y1);
  if (x0 > x1) return;  // nothing drawn (the same for the whole block)
  splat_block<COUNT>(kk, px, py, x0, y0, x1, y1, cam.W, key, zb, issued);
  if constexpr (COUNT) {
    for (int off = 32; off > 0; off >>= 1) issued += __shfl_xor(issued, off, 64);
    if ((threadIdx.x & 63) == 0 && issued) atomicAdd(&counters[kAtomicWord], issued);
  }
}

// Several views at once: the work item's points are read from memory once,
// kept in registers, and projected and splatted into each view of its mask
// in turn, as splat_kernel does for one view.
__global__ __launch_bounds__(kThreads) void splat_views_kernel(const float *__restrict__ xs,
                                                               const float *__restrict__ ys,
                                                               const float *__restrict__ zs,
                                                               const uint4 *__restrict__ items, uint32_t cap,
                                                               const uint32_t *__restrict__ counters, ViewsSplat vs) {
  __shared__ unsigned long long zb[kDedupPx];
  __shared__ uint32_t s_bb[4];
  uint4 it;
  if (!work_item(blockIdx.x, counters, items, cap, &it)) return;
  const int tid = threadIdx.x;
  float x[kPtsPerThread], y[kPtsPerThread], z[kPtsPerThread];
#pragma unroll
  for (int q = 0; q < kPtsPerThread; ++q) {
    const uint32_t i = tid + q * kThreads;
    x[q] = y[q] = z[q] = 0.f;
    if (i < it.y) {
      x[q] = xs[it.x + i];
      y[q] = ys[it.x + i];
      z[q] = zs[it.x + i];
    }
  }
  uint32_t issued = 0;
  // the mask is the same for every lane: keep it (and the view index) scalar
  for (uint32_t m = __builtin_amdgcn_readfirstlane(it.z); m; m &= m - 1) {
    const int v = __builtin_ctz(m);
    const SplatCam &cam = vs.cam[v];
    uint64_t kk[kPtsPerThread];
    uint32_t px[kPtsPerThread], py[kPtsPerThread];
    uint32_t x0 = ~0u, y0 = ~0u, x1 = 0, y1 = 0;
#pragma unroll
    for (int q = 0; q < kPtsPerThread; ++q) {
      const uint32_t i = tid + q * kThreads;
      uint64_t k = 0;
      uint32_t ux = ~0u, uy = 0;
      if (i < it.y && project_point(x[q], y[q], z[q], it.x + i, cam, k, ux, uy)) {
        x0 = min(x0, ux);
        x1 = max(x1, ux);
        y0 = min(y0, uy);
        y1 = max(y1, uy);
      } else {
        ux = ~0u;
      }
      kk[q] = k;
      px[q] = ux;
      py[q] = uy;
    }
    block_rect(x0, y0, x1, y1, s_bb, &x0, &y0, &x1, &y1);
    if (x0 <= x1) splat_block<false>(kk, px, py, x0, y0, x1, y1, cam.W, vs.key[v], zb, issued);
    __syncthreads();  // s_bb and zb are reused by the next view
  }
}

// ---------------------------------------------------------------------------
// Screen-tiled splat (the default): no global atomic per point or pixel.
//
//   bin       one workgroup per work item: project the points; if they fall
//             in few enough 8 x 8 pixel blocks, keep only the nearest of each
//             pixel (LDS z-buffer); write the entries, grouped by 32 x 32
//             screen tile, as 8-byte records at the work item's own place in
//             the record array.  Each (work item, tile) group is a segment.
//   tilescan  one workgroup: per-tile segment offsets, and the units of work
//             of the tile kernel: up to kSegsPerUnit segments, or a few
//             thousand records, of one tile.
//   segsort   groups the segment ids by tile, and empties the keys of the
//             tiles of more than one unit (the only keys not written whole).
//             Up to kMaxScanTiles tiles, segscan_kernel does both in one
//             launch (every workgroup repeats the scan in LDS).
//   tile      one workgroup per unit: LDS z-buffer of the tile over the
//             unit's records.  A tile of one unit owns its pixels and writes
//             key, depth and rgba (the resolve) with plain stores; the units
//             of a busier tile merge their minima into the key buffer with
//             atomicMin (one per pixel and unit), and
//   tileres   resolves those tiles afterwards.
//
// The soft z-buffer takes the same launches with every drawn point an entry:
// the tile kernel sums the colours of a tile of one unit too, and
//   soft      sums those of the busier tiles once their nearest depths have met.
//
// A record is (float32 depth bits << 32) | (pixel within the tile << 14) |
// (point index - work item start); the tile kernel rebuilds the key
// (depth bits << 32) | sorted index, so the image equals the atomic splat's.
// ---------------------------------------------------------------------------
constexpr int kTileShift = 5;  // 32 x 32 pixel tiles
constexpr int kTileSide = 1 << kTileShift;
constexpr int kTilePx = kTileSide * kTileSide;
constexpr int kHistBins = 1024;  // tiles one binning pass can address
constexpr int kSegsPerUnit = 32;
// Records per unit, about (see units_of).  Up to kFewTiles tiles (fewer
// workgroups than the chip takes at once) the smaller: soft z-buffer of 2.8 M
// points at 604 x 604: 139 us by segments alone, 92 with 4096, 85 with 2048.  Above
// it the merging of more units costs more than it evens out: 100 M points at
// 2560 x 1440: 340 us with 2048, 323 with 4096.
constexpr uint32_t kFewTiles = 1024, kRecsPerUnitFew = 2048, kRecsPerUnitMany = 4096;
__host__ __device__ inline uint32_t recs_per_unit(uint32_t n_tiles) {
  return n_tiles <= kFewTiles ? kRecsPerUnitFew : kRecsPerUnitMany;
}
constexpr int kRecOffsetBits = 14;  // of a record: the point's offset in its work item
static_assert(kBinDense <= 1u << kRecOffsetBits, "a record keeps the point offset within its work item");

// exclusive prefix over the block (blockDim.x = NT): each thread passes its
// value and gets the sum of the values of lower threads; *total receives the
// sum over the block
template <int NT>
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t *s_tmp /* [NT / 64] */, uint32_t *total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(incl, off, 64);
    if (lane >= off) incl += o;
  }
  if (lane == 63) s_tmp[wave] = incl;
  __syncthreads();
  uint32_t wbase = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    const uint32_t x = s_tmp[w];
    if (w < wave) wbase += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return wbase + incl - v;
}

struct TileGrid {
  uint32_t tiles_x, tiles_y, n_tiles;
};

// One view of a tiled render, and the NV views of a launch (blockIdx.y).
struct TiledView {
  SplatCam cam;
  const SplatCam *cam_dev;  // the camera in device memory instead (graph replays with new cameras), or nullptr
  uint32_t W, H, unit_cap;
  TileGrid tg;
  uint32_t *counters;  // kSegTopWord, kUnitsWord
  uint64_t *recs;
  uint4 *segs;
  unsigned long long *tile_nseg;  // per tile: records << 32 | segments; then u32 tile_fill per tile
  uint32_t *sorted, *tile_off, *tile_units;
  uint2 *units;
  uint64_t *key;
  float *depth;
  uint32_t *rgba;
  uint4 *acc;  // colour sums of the soft z-buffer, or nullptr
};
template <int NV>
struct TiledViews {
  TiledView v[NV];
};
static_assert(sizeof(TiledViews<kViewsPerPass>) + 64 <= 4096, "kernel arguments stay within 4 KB");
template <int NV>
__device__ inline const TiledView &this_view(const TiledViews<NV> &vs) {
  return vs.v[NV == 1 ? 0 : blockIdx.y];
}

// A frame's work items.  Clouds with dense cells (kDenseItem points per item or
// more) take items of up to 8 K points in workgroups of 512 threads: one on-chip
// z-buffer then meets twice the points of a cell, over twice the pixels, so
// fewer entries and segments leave it; others 4 K points and 256 threads.
template <int NT>
struct BinItem {
  static constexpr int kPoints = NT * 16;                 // per item
  static constexpr int kBlocks = NT >= 512 ? 128 : 64;   // 8 x 8 pixel blocks of the on-chip z-buffer
};

// Item: uint2 (start, count); of several views uint4 (start, count, mask of the
// views that see it).  ALL: every drawn point is an entry (the soft z-buffer
// sums them all).  work: the culling counters.
template <int NT, int NV, bool ALL>
__global__ __launch_bounds__(NT, 4) void bin_kernel(const float *__restrict__ xs, const float *__restrict__ ys,
                                                    const float *__restrict__ zs, const void *__restrict__ items,
                                                    uint32_t cap, const uint32_t *__restrict__ work,
                                                    TiledViews<NV> vs) {
  const TiledView &a = this_view(vs);
  const SplatCam cam = a.cam_dev ? *a.cam_dev : a.cam;
  const TileGrid tg = a.tg;
  uint32_t *__restrict__ counters = a.counters;
  uint64_t *__restrict__ recs = a.recs;
  uint4 *__restrict__ segs = a.segs;
  unsigned long long *__restrict__ tile_nseg = a.tile_nseg;
  constexpr int kBlocks = BinItem<NT>::kBlocks, kWaves = NT / 64, kPts = 16;
  constexpr int kZb = ALL ? kHistBins / 2 : kBlocks * 64;
  __shared__ unsigned long long s_zb[kZb];  // z-buffer; or the tile histogram
  __shared__ uint32_t s_off[kBlocks + 1];
  __shared__ uint32_t s_tmp[kWaves];
  __shared__ uint32_t s_bb[4];
  __shared__ uint32_t s_seg_base;
  uint32_t *s_hist = reinterpret_cast<uint32_t *>(s_zb);
  static_assert(kHistBins * 4 <= (int)sizeof(s_zb), "the histogram lies where the z-buffer is");
  uint2 ch;
  if constexpr (NV == 1) {
    if (!work_item(blockIdx.x, work, static_cast<const uint2 *>(items), cap, &ch)) return;
  } else {
    uint4 it;
    if (!work_item(blockIdx.x, work, static_cast<const uint4 *>(items), cap, &it)) return;
    if (!((it.z >> blockIdx.y) & 1u)) return;
    ch = make_uint2(it.x, it.y);
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  ch.x = (uint32_t)__builtin_amdgcn_readfirstlane((int)ch.x);
  ch.y = (uint32_t)__builtin_amdgcn_readfirstlane((int)ch.y);
  const float *xb = xs + ch.x, *yb = ys + ch.x, *zb = zs + ch.x;
  // thread t holds points t, t + NT, ...: depth bits and packed pixel (y << 16 | x; ~0 = not drawn)
  uint32_t wb[kPts], pix[kPts];
  uint32_t x0 = ~0u, y0 = ~0u, x1 = 0, y1 = 0;
  // (groups of four points, so that the loads of all sixteen are not held at once)
#pragma unroll
  for (int g = 0; g < kPts; g += 4) {
    if ((uint32_t)(g * NT) >= ch.y) {  // (the same for the whole block)
#pragma unroll
      for (int q = 0; q < 4; ++q) wb[g + q] = 0u, pix[g + q] = ~0u;
      continue;
    }
    float x[4], y[4], z[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t i = min((uint32_t)(tid + (g + q) * NT), ch.y - 1u);
      x[q] = xb[i];
      y[q] = yb[i];
      z[q] = zb[i];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint32_t px = 0, py = 0;
      const bool drawn = project_pixel(x[q], y[q], z[q], cam, &wb[g + q], &px, &py) &&
                         (uint32_t)(tid + (g + q) * NT) < ch.y;
      pix[g + q] = drawn ? (py << 16) | px : ~0u;
      x0 = min(x0, drawn ? px : ~0u);
      x1 = max(x1, drawn ? px : 0u);
      y0 = min(y0, drawn ? py : ~0u);
      y1 = max(y1, drawn ? py : 0u);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  block_rect(x0, y0, x1, y1, s_bb, &x0, &y0, &x1, &y1);
  if (x0 > x1) return;  // nothing drawn (the same for the whole block)
  const uint32_t tx0 = x0 >> kTileShift, ty0 = y0 >> kTileShift;
  const uint32_t tbw = (x1 >> kTileShift) - tx0 + 1, ty1 = y1 >> kTileShift;
  const uint32_t bx0 = x0 >> 3, by0 = y0 >> 3, nbx = (x1 >> 3) - bx0 + 1, nby = (y1 >> 3) - by0 + 1;
  if (!ALL && nbx <= (uint32_t)kBlocks && nby <= (uint32_t)kBlocks && nbx * nby <= (uint32_t)kBlocks) {
    // ---- the points meet in a z-buffer of 8 x 8 pixel blocks (row order), one
    // wave reads a block at a time, and the blocks' entries are written in
    // tile order
    const uint32_t nblk = nbx * nby;
    for (uint32_t p = tid; p < nblk * 64; p += NT) s_zb[p] = ~0ull;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPts; ++q) {
      uint32_t p = pix[q];
      asm volatile("" : "+v"(p));  // (nothing of it is held in registers beyond its turn)
      if (p != ~0u) {
        const uint32_t px = p & 0xFFFFu, py = p >> 16;
        const uint32_t slot = (((py >> 3) - by0) * nbx + ((px >> 3) - bx0)) * 64 + (py & 7) * 8 + (px & 7);
        atomicMin(&s_zb[slot], ((unsigned long long)wb[q] << 32) | (uint32_t)(tid + q * NT));
      }
    }
    __syncthreads();
    // place of block (bx, by) among the blocks in tile order
    auto place = [&](uint32_t bx, uint32_t by) {
      const uint32_t ty = (by0 + by) >> 2, tx = (bx0 + bx) >> 2;
      const uint32_t ys = max(by0, ty << 2) - by0, ye = min(by0 + nby, (ty + 1) << 2) - by0;
      const uint32_t xs_ = max(bx0, tx << 2) - bx0, xe = min(bx0 + nbx, (tx + 1) << 2) - bx0;
      return ys * nbx + (ye - ys) * xs_ + (by - ys) * (xe - xs_) + (bx - xs_);
    };
    const float inv_nbx = 1.0f / (float)nbx;
    for (uint32_t b = wave; b < nblk; b += kWaves) {
      const uint64_t m = __ballot(s_zb[b * 64 + lane] != ~0ull);
      const uint32_t by = small_div(b, inv_nbx);
      if (lane == 0) s_off[place(b - by * nbx, by)] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    if (wave == 0) {
      // exclusive prefix over the blocks in tile order, two per lane
      const uint32_t i0 = 2 * lane, i1 = 2 * lane + 1;
      const uint32_t c0 = i0 < nblk ? s_off[i0] : 0u, c1 = i1 < nblk ? s_off[i1] : 0u;
      uint32_t incl = c0 + c1;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t o = __shfl_up(incl, off, 64);
        if (lane >= off) incl += o;
      }
      if (i0 < nblk) s_off[i0] = incl - c0 - c1;
      if (i1 < nblk) s_off[i1] = incl - c1;
      if (lane == 63) s_off[nblk] = incl;
    }
    __syncthreads();
    if (wave == 0) {
      // the segments: one lane per tile (at most 34 of them)
      const uint32_t nty = ty1 - ty0 + 1, nt = tbw * nty;
      uint32_t first = 0, cnt = 0, tile = 0;
      if ((uint32_t)lane < nt) {
        const uint32_t tr = lane / tbw, tc = lane - tr * tbw;
        const uint32_t bx = max(bx0, (tx0 + tc) << 2) - bx0, by = max(by0, (ty0 + tr) << 2) - by0;
        const uint32_t ye = min(by0 + nby, (ty0 + tr + 1) << 2) - by0, xe = min(bx0 + nbx, (tx0 + tc + 1) << 2) - bx0;
        const uint32_t r = place(bx, by);
        first = s_off[r];
        cnt = s_off[r + (ye - by) * (xe - bx)] - first;
        tile = (ty0 + tr) * tg.tiles_x + tx0 + tc;
      }
      const uint64_t m = __ballot(cnt != 0);
      uint32_t base = 0;
      if (lane == 0) base = atomicAdd(&counters[kSegTopWord], (uint32_t)__popcll(m));
      base = __shfl(base, 0, 64);
      if (cnt) {
        segs[base + (uint32_t)__popcll(m & ((1ull << lane) - 1ull))] = make_uint4(tile, ch.x + first, cnt, ch.x);
        atomicAdd(&tile_nseg[tile], ((unsigned long long)cnt << 32) | 1ull);
      }
    }
    for (uint32_t b = wave; b < nblk; b += kWaves) {
      const uint64_t k = s_zb[b * 64 + lane];
      const uint64_t m = __ballot(k != ~0ull);
      const uint32_t by = small_div(b, inv_nbx), bx = b - by * nbx;
      if (k != ~0ull) {
        const uint32_t pos = s_off[place(bx, by)] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        const uint32_t local = ((((by0 + by) & 3) * 8 + (lane >> 3)) << kTileShift) | (((bx0 + bx) & 3) * 8 + (lane & 7));
        recs[ch.x + pos] = (k & 0xFFFFFFFF00000000ull) | ((uint64_t)local << kRecOffsetBits) | (uint64_t)(uint32_t)k;
      }
    }
    return;
  }
  // ---- a larger rectangle (a near surface), or ALL: every point is an entry.  Counting
  // sort by tile, in rounds of tile rows so that one round addresses at most
  // kHistBins tiles
  const uint32_t rows_per_round = max(1u, (uint32_t)kHistBins / tbw);
  uint32_t rec_next = 0;  // records written by earlier rounds
  for (uint32_t r0 = ty0; r0 <= ty1; r0 += rows_per_round) {
    const uint32_t r1 = min(ty1 + 1, r0 + rows_per_round);
    const uint32_t tbins = (r1 - r0) * tbw;
    // a row wider than the histogram is split into column ranges
    for (uint32_t c0 = 0; c0 < tbins; c0 += kHistBins) {
      const uint32_t nbins = min((uint32_t)kHistBins, tbins - c0);
      // bin of a drawn point in this round (nbins or more: another round's)
      // (the empty asm keeps the compiler from holding every point's tile across the rounds)
      auto bin_of = [&](uint32_t p) {
        asm volatile("" : "+v"(p));
        const uint32_t ty = (p >> 16) >> kTileShift, tx = (p & 0xFFFFu) >> kTileShift;
        return p == ~0u || ty < r0 || ty >= r1 ? ~0u : (ty - r0) * tbw + (tx - tx0) - c0;
      };
      for (uint32_t b = tid; b < nbins; b += NT) s_hist[b] = 0;
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPts; ++q) {
        const uint32_t bin = bin_of(pix[q]);
        if (bin < nbins) atomicAdd(&s_hist[bin], 1u);
      }
      __syncthreads();
      // exclusive prefix over the bins of record counts and non-empty flags
      // at once (16-bit halves: at most 8192 of each); a thread owns kPer bins
      constexpr int kPer = kHistBins / NT;
      uint32_t cnt[kPer], sum = 0;
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const uint32_t b = tid * kPer + q;
        cnt[q] = b < nbins ? s_hist[b] : 0u;
        sum += (cnt[q] << 16) | (cnt[q] ? 1u : 0u);
      }
      uint32_t total;
      uint32_t run = block_exclusive_scan<NT>(sum, s_tmp, &total);
      const uint32_t n_rec = total >> 16, n_seg = total & 0xFFFFu;
      if (n_rec == 0) continue;  // uniform: nothing in these bins
      if (tid == 0) s_seg_base = atomicAdd(&counters[kSegTopWord], n_seg);
      __syncthreads();
      const uint32_t seg_base = s_seg_base;
#pragma unroll
      for (int q = 0; q < kPer; ++q) {
        const uint32_t b = tid * kPer + q;
        if (b < nbins) {
          const uint32_t first = rec_next + (run >> 16);
          if (cnt[q]) {
            const uint32_t tb = c0 + b;
            const uint32_t tile = (r0 + tb / tbw) * tg.tiles_x + (tx0 + tb % tbw);
            segs[seg_base + (run & 0xFFFFu)] = make_uint4(tile, ch.x + first, cnt[q], ch.x);
            atomicAdd(&tile_nseg[tile], ((unsigned long long)cnt[q] << 32) | 1ull);
          }
          s_hist[b] = first;  // bin -> cursor at its first record
          run += (cnt[q] << 16) | (cnt[q] ? 1u : 0u);
        }
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < kPts; ++q) {
        const uint32_t bin = bin_of(pix[q]);
        if (bin >= nbins) continue;
        const uint32_t pos = atomicAdd(&s_hist[bin], 1u);
        const uint32_t px = pix[q] & 0xFFFFu, py = pix[q] >> 16;
        const uint32_t local = ((py & (kTileSide - 1)) << kTileShift) | (px & (kTileSide - 1));
        recs[ch.x + pos] = ((uint64_t)wb[q] << 32) | ((uint64_t)local << kRecOffsetBits) | (uint64_t)(uint32_t)(tid + q * NT);
      }
      rec_next += n_rec;
      __syncthreads();
    }
  }
}

// Units of a tile (count: records << 32 | segments): enough for kSegsPerUnit
// segments and about recs_per_unit() records each.  Where a near surface puts many
// points of a few work items on a tile, the segments alone would leave one
// workgroup with up to 32 x 8 K records while the others are done.
__device__ inline uint32_t units_of(unsigned long long count, uint32_t n_tiles) {
  const uint32_t ns = (uint32_t)count, nr = (uint32_t)(count >> 32), recs = recs_per_unit(n_tiles);
  const uint32_t nu = max((ns + kSegsPerUnit - 1) / kSegsPerUnit, (nr + recs - 1) / recs);
  return max(1u, min(nu, ns));
}
// segments per unit of a tile of ns segments and nu units (at most kSegsPerUnit)
__device__ inline uint32_t unit_segs(uint32_t ns, uint32_t nu) { return (ns + nu - 1) / nu; }

// One workgroup: per-tile segment offsets (tile_off[n_tiles + 1]) and the
// units of the tile kernel: tile_units[t] of them; units[u] = (tile, first
// segment of the unit within the tile); counters[kUnitsWord] = number of units.
constexpr int kScanThreads = 1024;
template <int NV>
__global__ __launch_bounds__(kScanThreads) void tilescan_kernel(TiledViews<NV> vs) {
  const TiledView &a = this_view(vs);
  const unsigned long long *__restrict__ tile_nseg = a.tile_nseg;
  const TileGrid tg = a.tg;
  uint32_t *__restrict__ tile_off = a.tile_off, *__restrict__ tile_units = a.tile_units;
  uint2 *__restrict__ units = a.units;
  const uint32_t unit_cap = a.unit_cap;
  uint32_t *__restrict__ counters = a.counters;
  __shared__ uint32_t s_tmp[kScanThreads / 64];
  const int tid = threadIdx.x;
  uint32_t seg_base = 0, unit_base = 0;
  for (uint32_t t0 = 0; t0 < tg.n_tiles; t0 += kScanThreads) {
    const uint32_t t = t0 + tid;
    const unsigned long long count = t < tg.n_tiles ? tile_nseg[t] : 0ull;
    const uint32_t ns = (uint32_t)count, nu = t < tg.n_tiles ? units_of(count, tg.n_tiles) : 0u, per = unit_segs(ns, max(1u, nu));
    uint32_t tot_s, tot_u;
    const uint32_t es = block_exclusive_scan<kScanThreads>(ns, s_tmp, &tot_s);
    const uint32_t eu = block_exclusive_scan<kScanThreads>(nu, s_tmp, &tot_u);
    if (t < tg.n_tiles) {
      tile_off[t] = seg_base + es;
      tile_units[t] = nu;
      for (uint32_t k = 0; k < nu; ++k)
        if (unit_base + eu + k < unit_cap) units[unit_base + eu + k] = make_uint2(t, k * per);
    }
    seg_base += tot_s;
    unit_base += tot_u;
  }
  if (tid == 0) {
    tile_off[tg.n_tiles] = seg_base;
    counters[kUnitsWord] = min(unit_base, unit_cap);
  }
}

// Segment ids grouped by tile: segment i of tile t goes to one of the places
// [tile_off[t], tile_off[t + 1]) (their order is irrelevant: the tile kernel
// takes a minimum).  Counts tile_nseg's segments back down to zero.  Also empties the
// key buffer over the tiles of more than one unit, whose units merge into it
// with atomicMin (the tile kernel writes every other tile's keys whole), and
// zeroes their colour sums (acc, the soft z-buffer).
template <int NV>
__global__ __launch_bounds__(kThreads) void segsort_kernel(TiledViews<NV> vs) {
  const TiledView &a = this_view(vs);
  const uint4 *__restrict__ segs = a.segs;
  const uint32_t *__restrict__ counters = a.counters, *__restrict__ tile_off = a.tile_off;
  const uint32_t *__restrict__ tile_units = a.tile_units;
  uint32_t *__restrict__ tile_nseg = reinterpret_cast<uint32_t *>(a.tile_nseg), *__restrict__ sorted = a.sorted;
  const TileGrid tg = a.tg;
  const uint32_t W = a.W, H = a.H;
  uint64_t *__restrict__ key = a.key;
  uint4 *__restrict__ acc = a.acc;
  const uint32_t n = counters[kSegTopWord];
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
    const uint32_t t = segs[i].x;
    sorted[tile_off[t] + atomicSub(&tile_nseg[2 * t], 1u) - 1u] = i;
  }
  for (uint32_t t = blockIdx.x; t < tg.n_tiles; t += gridDim.x) {
    if (tile_units[t] <= 1) continue;  // (the same for the whole block)
    const uint32_t tx = t % tg.tiles_x, ty = t / tg.tiles_x;
    for (int p = threadIdx.x; p < kTilePx; p += kThreads) {
      const uint32_t gx = (tx << kTileShift) + (p & (kTileSide - 1));
      const uint32_t gy = (ty << kTileShift) + (p >> kTileShift);
      if (gx < W && gy < H) {
        key[(size_t)gy * W + gx] = ~0ull;
        if (acc) acc[(size_t)gy * W + gx] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  }
}

// The scan and the segment sort in one launch, for images of at most
// kMaxScanTiles tiles: every workgroup takes the exclusive prefix of the
// per-tile segment counts itself, into LDS (a few thousand words, read from
// L2; each thread sums a run of consecutive tiles, one block scan of the
// sums, then each thread walks its run), so no workgroup waits for another; workgroup 0 also writes tile_off,
// tile_units, units and counters[kUnitsWord] for the tile kernel, as
// tilescan_kernel does.  The places within a tile come from a second counter
// array (tile_fill, zeroed with tile_nseg), since tile_nseg is read by every
// workgroup's scan.  Then, as segsort_kernel: the segment ids grouped by tile,
// and the keys of the tiles of more than one unit emptied.
constexpr uint32_t kMaxScanTiles = 8192;
template <int NV>
__global__ __launch_bounds__(kThreads) void segscan_kernel(TiledViews<NV> vs) {
  const TiledView &a = this_view(vs);
  const uint4 *__restrict__ segs = a.segs;
  uint32_t *__restrict__ counters = a.counters;
  const TileGrid tg = a.tg;
  const unsigned long long *__restrict__ tile_nseg = a.tile_nseg;
  uint32_t *__restrict__ tile_fill = reinterpret_cast<uint32_t *>(a.tile_nseg + tg.n_tiles), *__restrict__ tile_off = a.tile_off;
  uint32_t *__restrict__ tile_units = a.tile_units, *__restrict__ sorted = a.sorted;
  uint2 *__restrict__ units = a.units;
  const uint32_t unit_cap = a.unit_cap, W = a.W, H = a.H;
  uint64_t *__restrict__ key = a.key;
  uint4 *__restrict__ acc = a.acc;
  __shared__ uint32_t s_off[kMaxScanTiles + 1];
  __shared__ uint32_t s_tmp[kThreads / 64];
  const int tid = threadIdx.x;
  const bool first = blockIdx.x == 0;
  // thread tid owns tiles [tid per, (tid + 1) per): its own sums, one block
  // scan of them, then its tiles' offsets in order
  const uint32_t per = (tg.n_tiles + kThreads - 1) / kThreads;
  const uint32_t t_lo = min(tg.n_tiles, tid * per), t_hi = min(tg.n_tiles, t_lo + per);
  uint32_t my_s = 0, my_u = 0;
  for (uint32_t t = t_lo; t < t_hi; ++t) {
    const unsigned long long count = tile_nseg[t];
    my_s += (uint32_t)count;
    my_u += units_of(count, tg.n_tiles);
  }
  uint32_t tot_s, tot_u;
  uint32_t seg = block_exclusive_scan<kThreads>(my_s, s_tmp, &tot_s);
  uint32_t unit = block_exclusive_scan<kThreads>(my_u, s_tmp, &tot_u);
  for (uint32_t t = t_lo; t < t_hi; ++t) {
    const unsigned long long count = tile_nseg[t];
    const uint32_t ns = (uint32_t)count, nu = units_of(count, tg.n_tiles);
    s_off[t] = seg;
    if (first) {
      tile_off[t] = seg;
      tile_units[t] = nu;
      const uint32_t unit_len = unit_segs(ns, nu);
      for (uint32_t k = 0; k < nu; ++k)
        if (unit + k < unit_cap) units[unit + k] = make_uint2(t, k * unit_len);
    }
    seg += ns;
    unit += nu;
  }
  if (tid == 0) {
    s_off[tg.n_tiles] = tot_s;
    if (first) {
      tile_off[tg.n_tiles] = tot_s;
      counters[kUnitsWord] = min(tot_u, unit_cap);
    }
  }
  __syncthreads();
  const uint32_t n = counters[kSegTopWord];
  for (uint32_t i = blockIdx.x * kThreads + tid; i < n; i += gridDim.x * kThreads) {
    const uint32_t t = segs[i].x;
    sorted[s_off[t] + atomicAdd(&tile_fill[t], 1u)] = i;
  }
  for (uint32_t t = blockIdx.x; t < tg.n_tiles; t += gridDim.x) {
    if (units_of(tile_nseg[t], tg.n_tiles) == 1) continue;  // (the same for the whole block)
    const uint32_t tx = t % tg.tiles_x, ty = t / tg.tiles_x;
    for (int p = tid; p < kTilePx; p += kThreads) {
      const uint32_t gx = (tx << kTileShift) + (p & (kTileSide - 1));
      const uint32_t gy = (ty << kTileShift) + (p >> kTileShift);
      if (gx < W && gy < H) {
        key[(size_t)gy * W + gx] = ~0ull;
        if (acc) acc[(size_t)gy * W + gx] = make_uint4(0u, 0u, 0u, 0u);
      }
    }
  }
}

__device__ inline void resolve_px(uint64_t k, const uint32_t *__restrict__ rgbx, size_t i, float *__restrict__ depth,
                                  uint32_t *__restrict__ rgba) {
  if (k == ~0ull) {
    depth[i] = 0.f;
    rgba[i] = 0u;
  } else {
    depth[i] = __uint_as_float((uint32_t)(k >> 32));
    rgba[i] = (rgbx[(uint32_t)k] & 0x00FFFFFFu) | (1u << 24);
  }
}

// The records of a unit: up to kSegsPerUnit segments of one tile, NT threads.
struct UnitSegs {
  uint32_t pref[kSegsPerUnit + 1];  // prefix of the segments' record counts
  uint2 seg[kSegsPerUnit];          // first record, work item start
};
// Segments [beg, end) of the sorted list into u (called by every thread; a
// barrier follows before u is read).
__device__ inline void load_unit(UnitSegs &u, const uint4 *__restrict__ segs, const uint32_t *__restrict__ sorted,
                                 uint32_t beg, uint32_t nb) {
  const int tid = threadIdx.x;
  if (tid >= 64) return;
  uint32_t c = 0;
  if ((uint32_t)tid < nb) {
    const uint4 sg = segs[sorted[beg + tid]];
    u.seg[tid] = make_uint2(sg.y, sg.w);
    c = sg.z;
  }
  uint32_t incl = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t o = __shfl_up(incl, off, 64);
    if (tid >= off) incl += o;
  }
  if (tid <= kSegsPerUnit) u.pref[tid] = incl - c;  // pref[nb] = total
}
// f(depth bits, pixel of the tile, point index) for every record of the unit.
// kInFlight records per thread: their loads are issued before the first is
// used, so their latencies overlap.
template <int NT, typename F>
__device__ inline void for_records(const UnitSegs &u, uint32_t nb, const uint64_t *__restrict__ recs, F f) {
  constexpr int kInFlight = 4;
  const uint32_t total = u.pref[nb];
  for (uint32_t r0 = threadIdx.x; r0 < total; r0 += kInFlight * NT) {
    uint64_t rc[kInFlight];
    uint32_t base[kInFlight];
#pragma unroll
    for (int m = 0; m < kInFlight; ++m) {
      const uint32_t r = r0 + m * NT;
      rc[m] = ~0ull;
      base[m] = 0;
      if (r < total) {
        uint32_t lo = 0, hi = nb;  // the last segment whose prefix is <= r
        while (hi - lo > 1) {
          const uint32_t mid = (lo + hi) >> 1;
          if (u.pref[mid] <= r) lo = mid;
          else hi = mid;
        }
        const uint2 sg = u.seg[lo];
        rc[m] = recs[sg.x + (r - u.pref[lo])];
        base[m] = sg.y;
      }
    }
#pragma unroll
    for (int m = 0; m < kInFlight; ++m) {
      if (rc[m] == ~0ull) continue;
      const uint32_t lo = (uint32_t)rc[m];
      f((uint32_t)(rc[m] >> 32), (lo >> kRecOffsetBits) & (kTilePx - 1), base[m] + (lo & ((1u << kRecOffsetBits) - 1u)));
    }
  }
}

// Colour sums of the soft z-buffer: two words of two 32-bit sums each (red |
// green << 32, blue | points << 32), added to without carries between them.
__device__ inline void add_colour(unsigned long long *sum, uint32_t c) {
  atomicAdd(&sum[0], (unsigned long long)(c & 255u) | ((unsigned long long)((c >> 8) & 255u) << 32));
  atomicAdd(&sum[1], (unsigned long long)((c >> 16) & 255u) | (1ull << 32));
}
// mean of the summed colours, rounded half up, with the fill mask
__device__ inline uint32_t mean_colour(uint64_t rg, uint64_t bn) {
  const uint64_t n = bn >> 32, n2 = 2ull * n;
  const uint32_t r = (uint32_t)((2ull * (uint32_t)rg + n) / n2);
  const uint32_t g = (uint32_t)((2ull * (rg >> 32) + n) / n2);
  const uint32_t b = (uint32_t)((2ull * (uint32_t)bn + n) / n2);
  return r | (g << 8) | (b << 16) | (1u << 24);
}

// Units of work, grid-stride: the LDS z-buffer of one tile over the records
// of up to kSegsPerUnit of its segments.  SOFT: a tile of one unit then goes
// over its records again and sums the colours of the points within one_plus_eps
// of their pixel's nearest depth (in LDS: the sums never go to memory).
template <int NT, int NV, bool SOFT>
__global__ __launch_bounds__(NT) void tile_kernel(TiledViews<NV> vs, const uint32_t *__restrict__ rgbx,
                                                  float one_plus_eps) {
  const TiledView &a = this_view(vs);
  const uint64_t *__restrict__ recs = a.recs;
  const uint4 *__restrict__ segs = a.segs;
  const uint32_t *__restrict__ sorted = a.sorted, *__restrict__ tile_off = a.tile_off;
  const uint32_t *__restrict__ tile_units = a.tile_units, *__restrict__ counters = a.counters;
  const uint2 *__restrict__ units = a.units;
  const TileGrid tg = a.tg;
  const uint32_t W = a.W, H = a.H;
  uint64_t *__restrict__ key = a.key;
  float *__restrict__ depth = a.depth;
  uint32_t *__restrict__ rgba = a.rgba;
  __shared__ unsigned long long zb[kTilePx];
  __shared__ unsigned long long sums[SOFT ? 2 * kTilePx : 1];
  __shared__ UnitSegs us;
  const int tid = threadIdx.x;
  const uint32_t n_units = counters[kUnitsWord];
  for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    const uint2 un = units[u];
    const uint32_t t = un.x;
    const uint32_t off = tile_off[t], next = tile_off[t + 1];
    const uint32_t beg = off + un.y, end = min(next, beg + unit_segs(next - off, tile_units[t]));
    const uint32_t nb = end > beg ? end - beg : 0u;
    const bool alone = tile_units[t] == 1;
    for (int p = tid; p < kTilePx; p += NT) zb[p] = ~0ull;
    if constexpr (SOFT)
      for (int p = tid; p < 2 * kTilePx; p += NT) sums[p] = 0ull;
    load_unit(us, segs, sorted, beg, nb);
    __syncthreads();
    for_records<NT>(us, nb, recs, [&](uint32_t w, uint32_t px, uint32_t j) {
      atomicMin(&zb[px], ((unsigned long long)w << 32) | j);
    });
    __syncthreads();
    if constexpr (SOFT) {
      if (alone) {
        for_records<NT>(us, nb, recs, [&](uint32_t w, uint32_t px, uint32_t j) {
          const float zmin = __uint_as_float((uint32_t)(zb[px] >> 32));
          if (__uint_as_float(w) <= zmin * one_plus_eps) add_colour(&sums[2 * px], rgbx[j]);
        });
        __syncthreads();
      }
    }
    const uint32_t tx = t % tg.tiles_x, ty = t / tg.tiles_x;
    for (int p = tid; p < kTilePx; p += NT) {
      const uint32_t gx = (tx << kTileShift) + (p & (kTileSide - 1));
      const uint32_t gy = (ty << kTileShift) + (p >> kTileShift);
      if (gx >= W || gy >= H) continue;
      const size_t i = (size_t)gy * W + gx;
      const uint64_t k = zb[p];
      if (alone) {
        key[i] = k;
        if constexpr (SOFT) {
          depth[i] = k == ~0ull ? 0.f : __uint_as_float((uint32_t)(k >> 32));
          rgba[i] = k == ~0ull ? 0u : mean_colour(sums[2 * p], sums[2 * p + 1]);
        } else {
          resolve_px(k, rgbx, i, depth, rgba);
        }
      } else if (k != ~0ull) {
        atomicMin(reinterpret_cast<unsigned long long *>(key + i), (unsigned long long)k);
      }
    }
    __syncthreads();
  }
}

// Soft z-buffer of the tiles of more than one unit, once their nearest depths
// have met in the key buffer: each unit sums its colours in LDS and adds them
// to the pixels' sums in memory (two 64-bit atomics per pixel and unit).
template <int NT>
__global__ __launch_bounds__(NT) void soft_units_kernel(TiledViews<1> vs, const uint32_t *__restrict__ rgbx,
                                                        float one_plus_eps) {
  const TiledView &a = vs.v[0];
  const uint64_t *__restrict__ recs = a.recs, *__restrict__ key = a.key;
  const uint4 *__restrict__ segs = a.segs;
  const uint32_t *__restrict__ sorted = a.sorted, *__restrict__ tile_off = a.tile_off;
  const uint32_t *__restrict__ tile_units = a.tile_units, *__restrict__ counters = a.counters;
  const uint2 *__restrict__ units = a.units;
  const TileGrid tg = a.tg;
  const uint32_t W = a.W, H = a.H;
  unsigned long long *__restrict__ acc = reinterpret_cast<unsigned long long *>(a.acc);
  __shared__ unsigned long long sums[2 * kTilePx];
  __shared__ float zmin[kTilePx];
  __shared__ UnitSegs us;
  const int tid = threadIdx.x;
  const uint32_t n_units = counters[kUnitsWord];
  for (uint32_t u = blockIdx.x; u < n_units; u += gridDim.x) {
    const uint2 un = units[u];
    const uint32_t t = un.x;
    if (tile_units[t] == 1) continue;  // (the same for the whole block)
    const uint32_t off = tile_off[t], next = tile_off[t + 1];
    const uint32_t beg = off + un.y, end = min(next, beg + unit_segs(next - off, tile_units[t]));
    const uint32_t nb = end > beg ? end - beg : 0u;
    const uint32_t tx = t % tg.tiles_x, ty = t / tg.tiles_x;
    auto pixel = [&](int p, size_t *i) {
      const uint32_t gx = (tx << kTileShift) + (p & (kTileSide - 1));
      const uint32_t gy = (ty << kTileShift) + (p >> kTileShift);
      *i = (size_t)gy * W + gx;
      return gx < W && gy < H;
    };
    for (int p = tid; p < kTilePx; p += NT) {
      size_t i;
      zmin[p] = pixel(p, &i) ? __uint_as_float((uint32_t)(key[i] >> 32)) : 0.f;
      sums[2 * p] = sums[2 * p + 1] = 0ull;
    }
    load_unit(us, segs, sorted, beg, nb);
    __syncthreads();
    for_records<NT>(us, nb, recs, [&](uint32_t w, uint32_t px, uint32_t j) {
      if (__uint_as_float(w) <= zmin[px] * one_plus_eps) add_colour(&sums[2 * px], rgbx[j]);
    });
    __syncthreads();
    for (int p = tid; p < kTilePx; p += NT) {
      size_t i;
      if (pixel(p, &i) && sums[2 * p + 1]) {
        atomicAdd(&acc[2 * i], sums[2 * p]);
        atomicAdd(&acc[2 * i + 1], sums[2 * p + 1]);
      }
    }
    __syncthreads();
  }
}

// Resolve of the tiles whose units merged through the key buffer (and, with
// acc, through the colour sums).
template <int NV>
__global__ __launch_bounds__(kThreads) void tileres_kernel(TiledViews<NV> vs, const uint32_t *__restrict__ rgbx) {
  const TiledView &a = this_view(vs);
  const uint32_t *__restrict__ tile_units = a.tile_units;
  const TileGrid tg = a.tg;
  const uint32_t W = a.W, H = a.H;
  const uint64_t *__restrict__ key = a.key, *__restrict__ acc = reinterpret_cast<const uint64_t *>(a.acc);
  float *__restrict__ depth = a.depth;
  uint32_t *__restrict__ rgba = a.rgba;
  if (NV > 1 && blockIdx.x >= tg.n_tiles) return;
  const uint32_t t = blockIdx.x;
  if (tile_units[t] == 1) return;
  const uint32_t tx = t % tg.tiles_x, ty = t / tg.tiles_x;
  for (int p = threadIdx.x; p < kTilePx; p += kThreads) {
    const uint32_t gx = (tx << kTileShift) + (p & (kTileSide - 1));
    const uint32_t gy = (ty << kTileShift) + (p >> kTileShift);
    if (gx >= W || gy >= H) continue;
    const size_t i = (size_t)gy * W + gx;
    const uint64_t k = key[i];
    if (acc && k != ~0ull) {
      depth[i] = __uint_as_float((uint32_t)(k >> 32));
      rgba[i] = mean_colour(acc[2 * i], acc[2 * i + 1]);
    } else {
      resolve_px(k, rgbx, i, depth, rgba);
    }
  }
}

// Throughput probe for the z-buffer's operation: each thread issues
// kProbeIters 64-bit atomicMin.  Pattern 0 draws the word of each from a
// per-thread xorshift32 sequence (Marsaglia's 13/17/5 shifts), so the
// operations spread over the buffer as a splat's do over the image; pattern 1
// sends the 64 lanes of a wave to one word.  Values decrease along each
// thread's sequence, so most operations lower the word.
__global__ __launch_bounds__(kThreads) void atomic_probe_kernel(uint64_t *__restrict__ buf, uint32_t n_slots,
                                                                int pattern, uint32_t seed) {
  const uint32_t gid = blockIdx.x * kThreads + threadIdx.x;
  uint32_t x = (gid + 1u) * 0x9E3779B9u ^ seed;
  if (x == 0) x = 1u;
  const uint32_t wave = gid >> 6, nwaves = gridDim.x * (kThreads / 64);
  for (uint32_t i = 0; i < kProbeIters; ++i) {
    uint32_t slot;
    if (pattern == 0) {
      x ^= x << 13;
      x ^= x >> 17;
      x ^= x << 5;
      slot = x % n_slots;
    } else {
      slot = (i * nwaves + wave) % n_slots;
    }
    const uint64_t v = ((uint64_t)(kProbeIters - i) << 32) | gid;
    atomicMin(reinterpret_cast<unsigned long long *>(buf + slot), (unsigned long long)v);
  }
}

// Soft z-buffer (Method, "Point Cloud Projection": colours of points at similar
// depths are averaged) behind the atomic splat.  A second pass over the same
// work items adds the colour of every point whose depth is within (1 + eps) of
// its pixel's nearest depth into integer sums; integer atomics make the result
// order independent.
__global__ __launch_bounds__(kThreads) void soft_accum_kernel(const float *__restrict__ xs, const float *__restrict__ ys,
                                                              const float *__restrict__ zs,
                                                              const uint32_t *__restrict__ rgbx,
                                                              const uint2 *__restrict__ chunks, uint32_t cap,
                                                              const uint32_t *__restrict__ counters, SplatCam cam,
                                                              const uint64_t *__restrict__ key, float one_plus_eps,
                                                              unsigned long long *__restrict__ acc) {
  uint2 ch;
  if (!work_item(blockIdx.x, counters, chunks, cap, &ch)) return;
  for (uint32_t i = threadIdx.x; i < ch.y; i += kThreads) {
    const uint32_t j = ch.x + i;
    uint64_t k;
    uint32_t px, py;
    if (!project_point(xs[j], ys[j], zs[j], j, cam, k, px, py)) continue;
    const size_t p = (size_t)py * cam.W + px;
    const float zmin = __uint_as_float((uint32_t)(key[p] >> 32));
    if (__uint_as_float((uint32_t)(k >> 32)) <= zmin * one_plus_eps) add_colour(acc + 2 * p, rgbx[j]);
  }
}

__global__ __launch_bounds__(kThreads) void resolve_soft_kernel(const uint64_t *__restrict__ key,
                                                                const uint64_t *__restrict__ acc,
                                                                float *__restrict__ depth, uint32_t *__restrict__ rgba,
                                                                uint32_t npix) {
  const uint32_t stride = gridDim.x * kThreads;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < npix; i += stride) {
    const uint64_t k = key[i];
    depth[i] = k == ~0ull ? 0.f : __uint_as_float((uint32_t)(k >> 32));
    rgba[i] = k == ~0ull ? 0u : mean_colour(acc[2ull * i], acc[2ull * i + 1]);
  }
}

__global__ __launch_bounds__(kThreads) void clear_acc_kernel(uint4 *__restrict__ acc, uint32_t npix) {
  const uint32_t stride = gridDim.x * kThreads;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < npix; i += stride) acc[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ __launch_bounds__(kThreads) void resolve_kernel(const uint64_t *__restrict__ key,
                                                           const uint32_t *__restrict__ rgbx, float *__restrict__ depth,
                                                           uint32_t *__restrict__ rgba, uint32_t npix) {
  const uint32_t stride = gridDim.x * kThreads;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < npix; i += stride) {
    const uint64_t k = key[i];
    if (k == ~0ull) {
      depth[i] = 0.f;
      rgba[i] = 0u;
    } else {
      depth[i] = __uint_as_float((uint32_t)(k >> 32));
      rgba[i] = (rgbx[(uint32_t)k] & 0x00FFFFFFu) | (1u << 24);
    }
  }
}

// threads per tile of the soft splat: its records are every drawn point
constexpr int kSoftThreads = 512;

inline uint32_t grid_for(uint32_t n) {
  uint32_t b = (n + kThreads - 1) / kThreads;
  return b < 1 ? 1 : (b > 8192 ? 8192 : b);
}

}  // namespace

hipError_t launch_clear(uint64_t *key, uint32_t npix, uint32_t *counters, uint32_t n_counters, uint32_t *tile_nseg,
                        uint32_t n_tiles, hipStream_t s) {
  clear_kernel<<<grid_for(npix > n_tiles ? npix : n_tiles), kThreads, 0, s>>>(key, npix, counters, n_counters,
                                                                             tile_nseg, n_tiles);
  return hipGetLastError();
}

TiledSplatGrid tiled_splat_grid(uint32_t W, uint32_t H, const CloudDev &c) {
  TiledSplatGrid g;
  g.tiles_x = (W + kTileSide - 1) >> kTileShift;
  g.tiles_y = (H + kTileSide - 1) >> kTileShift;
  g.n_tiles = g.tiles_x * g.tiles_y;
  g.seg_cap = std::max<uint64_t>(1, std::min<uint64_t>(c.n, (uint64_t)c.max_items * g.n_tiles));
  g.unit_cap = tiled_unit_cap(g.n_tiles, g.seg_cap, c.n);
  return g;
}
// units_of() of a tile of s segments and r >= s records is less than
// 1 + max(s / kSegsPerUnit, r / R), at most 1 + s / kSegsPerUnit + (r - s) / R
// for R = recs_per_unit() > kSegsPerUnit; the sum grows with both totals.
uint64_t tiled_unit_cap(uint32_t n_tiles, uint64_t seg_cap, uint32_t n) {
  return (uint64_t)n_tiles + seg_cap / kSegsPerUnit + (n - std::min<uint64_t>(n, seg_cap)) / recs_per_unit(n_tiles) + 1;
}

namespace {
template <int NV>
hipError_t tiled_stage(const CloudDev &c, const void *items, const uint32_t *work, const TiledSplatView *views, int n,
                       float one_plus_eps, int stage, hipStream_t s) {
  TiledViews<NV> vs;
  uint32_t most_tiles = 0, tile_grid = 0;
  const bool merged = tiled_scan_merged(views, n);
  for (int i = 0; i < NV; ++i) {
    const TiledSplatView &w = views[i < n ? i : 0];
    const TiledSplatGrid g = tiled_splat_grid(w.cam.W, w.H, c);
    vs.v[i] = TiledView{w.cam, w.cam_dev, w.cam.W, w.H, (uint32_t)g.unit_cap,
                        TileGrid{g.tiles_x, g.tiles_y, g.n_tiles}, w.counters, w.b.recs, w.b.segs,
                        reinterpret_cast<unsigned long long *>(w.b.tile_nseg), w.b.sorted, w.b.tile_off, w.b.tile_units, w.b.units, w.key, w.depth, w.rgba,
                        static_cast<uint4 *>(w.acc)};
    most_tiles = std::max(most_tiles, g.n_tiles);
    tile_grid = std::max(tile_grid,
                         (uint32_t)std::min<uint64_t>(g.unit_cap, std::max<uint64_t>(2ull * g.n_tiles, 4096)));
  }
  const bool soft = views[0].acc != nullptr;
  const uint32_t ny = (uint32_t)n;
  switch (stage) {
    case 0:
#define LNR_BIN(NT, ALL)                                                                                              \
  bin_kernel<NT, NV, ALL><<<dim3(c.max_items, ny), NT, 0, s>>>(c.x, c.y, c.z, items, c.max_chunks, work, vs)
      if constexpr (NV == 1) {  // (the soft z-buffer renders one view at a time)
        if (soft) {
          if (c.item_points == kBinDense) LNR_BIN(512, true); else LNR_BIN(256, true);
          break;
        }
      }
      if (c.item_points == kBinDense) LNR_BIN(512, false); else LNR_BIN(256, false);
#undef LNR_BIN
      break;
    case 1:
      if (merged) return hipSuccess;  // taken by the segment sort
      tilescan_kernel<NV><<<dim3(1, ny), kScanThreads, 0, s>>>(vs);
      break;
    case 2:
      if (merged)
        segscan_kernel<NV><<<dim3(256, ny), kThreads, 0, s>>>(vs);
      else
        segsort_kernel<NV><<<dim3(1024, ny), kThreads, 0, s>>>(vs);
      break;
    case 3:
      if constexpr (NV == 1) {
        if (soft) {
          tile_kernel<kSoftThreads, 1, true><<<tile_grid, kSoftThreads, 0, s>>>(vs, c.rgbx, one_plus_eps);
          break;
        }
      }
      tile_kernel<kThreads, NV, false><<<dim3(tile_grid, ny), kThreads, 0, s>>>(vs, c.rgbx, 1.f);
      break;
    case 4:
      if constexpr (NV == 1) {
        if (soft) soft_units_kernel<kSoftThreads><<<tile_grid, kSoftThreads, 0, s>>>(vs, c.rgbx, one_plus_eps);
      }
      break;
    case 5:
      tileres_kernel<NV><<<dim3(most_tiles, ny), kThreads, 0, s>>>(vs, c.rgbx);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
}  // namespace

bool tiled_scan_merged(const TiledSplatView *views, int n) {
  for (int i = 0; i < n; ++i) {
    const uint32_t tx = (views[i].cam.W + kTileSide - 1) >> kTileShift, ty = (views[i].H + kTileSide - 1) >> kTileShift;
    if (tx * ty > kMaxScanTiles) return false;
  }
  return true;
}

hipError_t launch_tiled_splat(const CloudDev &c, const uint2 *chunks, const uint32_t *work, const TiledSplatView &view,
                              float one_plus_eps, int stage, hipStream_t s) {
  if (c.max_chunks == 0) return hipErrorInvalidValue;  // a loaded cloud has at least one point
  return tiled_stage<1>(c, chunks, work, &view, 1, one_plus_eps, stage, s);
}

hipError_t launch_tiled_views(const CloudDev &c, const uint4 *items, const uint32_t *work, const TiledSplatView *views,
                              int n, int stage, hipStream_t s) {
  if (c.max_chunks == 0 || n < 1 || n > kViewsPerPass) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (views[i].acc) return hipErrorInvalidValue;  // the soft z-buffer renders one view at a time
  return tiled_stage<kViewsPerPass>(c, items, work, views, n, 1.f, stage, s);
}

hipError_t launch_cull(const CloudDev &c, const CullParams &prm, const CullParams *prm_dev, uint8_t *flags,
                       uint2 *chunks, uint32_t chunk, uint32_t *counters, hipStream_t s) {
  const uint32_t nb = (c.n_cells + kThreads - 1) / kThreads;
  if (prm_dev)
    cull_kernel<true><<<nb, kThreads, 0, s>>>(c.aabb, c.cell_start, c.n_cells, prm, prm_dev, flags, chunks,
                                              c.max_chunks, chunk, counters);
  else
    cull_kernel<false><<<nb, kThreads, 0, s>>>(c.aabb, c.cell_start, c.n_cells, prm, nullptr, flags, chunks,
                                               c.max_chunks, chunk, counters);
  return hipGetLastError();
}

hipError_t launch_splat(const CloudDev &c, const uint2 *chunks, uint32_t *counters, const SplatCam &cam,
                        uint64_t *key, bool count_atomics, hipStream_t s) {
  if (c.max_chunks == 0) return hipSuccess;
  const uint32_t g = c.max_chunks, cap = c.max_chunks;
  if (count_atomics)
    splat_kernel<true><<<g, kThreads, 0, s>>>(c.x, c.y, c.z, chunks, cap, counters, cam, key);
  else
    splat_kernel<false><<<g, kThreads, 0, s>>>(c.x, c.y, c.z, chunks, cap, counters, cam, key);
  return hipGetLastError();
}

hipError_t launch_cull_views(const CloudDev &c, const ViewsCull &prm, const DevCam *dev, uint8_t *flags, uint4 *items,
                             uint32_t chunk, uint32_t *counters, hipStream_t s) {
  if (prm.n < 1 || prm.n > kViewsPerPass) return hipErrorInvalidValue;
  const uint32_t nb = (c.n_cells + kThreads - 1) / kThreads;
  cull_views_kernel<<<nb, kThreads, 0, s>>>(c.aabb, c.cell_start, c.n_cells, prm, dev, flags, items, c.max_chunks,
                                            chunk, counters);
  return hipGetLastError();
}

hipError_t launch_splat_views(const CloudDev &c, const uint4 *items, const uint32_t *counters, const ViewsSplat &vs,
                              hipStream_t s) {
  if (vs.n < 1 || vs.n > kViewsPerPass) return hipErrorInvalidValue;
  if (c.max_chunks == 0) return hipSuccess;
  splat_views_kernel<<<c.max_chunks, kThreads, 0, s>>>(c.x, c.y, c.z, items, c.max_chunks, counters, vs);
  return hipGetLastError();
}

hipError_t launch_atomic_probe(uint64_t *buf, uint32_t n_slots, int pattern, uint32_t grid, uint32_t seed,
                               hipStream_t s) {
  if (n_slots == 0 || grid == 0) return hipErrorInvalidValue;
  atomic_probe_kernel<<<grid, kThreads, 0, s>>>(buf, n_slots, pattern, seed);
  return hipGetLastError();
}

hipError_t launch_resolve(const uint64_t *key, const uint32_t *rgbx, float *depth, uint32_t *rgba, uint32_t npix,
                          hipStream_t s) {
  resolve_kernel<<<grid_for(npix), kThreads, 0, s>>>(key, rgbx, depth, rgba, npix);
  return hipGetLastError();
}

hipError_t launch_soft(const CloudDev &c, const uint2 *chunks, const uint32_t *counters, const SplatCam &cam,
                       const uint64_t *key, float one_plus_eps, void *acc, float *depth, uint32_t *rgba, uint32_t npix,
                       hipStream_t s) {
  clear_acc_kernel<<<grid_for(npix), kThreads, 0, s>>>(static_cast<uint4 *>(acc), npix);
  if (c.max_chunks)
    soft_accum_kernel<<<c.max_chunks, kThreads, 0, s>>>(c.x, c.y, c.z, c.rgbx, chunks, c.max_chunks, counters, cam, key,
                                                       one_plus_eps, static_cast<unsigned long long *>(acc));
  resolve_soft_kernel<<<grid_for(npix), kThreads, 0, s>>>(key, static_cast<const uint64_t *>(acc), depth, rgba, npix);
  return hipGetLastError();
}

}  // namespace lnr
