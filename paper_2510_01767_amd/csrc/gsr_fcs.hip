// Fast camera selection (Sec. 3.2) on gfx950: every pixel's composited
// depth is back-projected through its pixel centre into world space and
// counted into the block boxes that hold it; the ratio V_{c,b} = count / N_p
// (N_p = the view's pixels) selects the cameras with V_{c,b} >= tau.
//
// Grid: x strides over a view's pixels, y is the view.  Each workgroup looks
// its points' boxes up in a table of the boxes' sorted bounds in LDS, counts
// in LDS and adds its counts to the global ones with one atomic per
// (workgroup, block).  A second kernel turns counts into ratios and the
// selection.
#include <hip/hip_runtime.h>

#include "gsr_device.h"
#include "gsr_stages.h"

namespace gsr {

// World point of pixel pix of a view with composited depth D, through the
// pixel's centre: R^T (D ((u + 1/2 - cx) / fx, (v + 1/2 - cy) / fy, 1) - t).
__device__ __forceinline__ void back_project_pixel(const gsr_camera &c, int W, int64_t pix, double D, double w[3]) {
  // (a view has at most 2^28 pixels: a 32-bit division)
  const int py = (int)((uint32_t)pix / (uint32_t)W), px = (int)((uint32_t)pix - (uint32_t)py * (uint32_t)W);
  const double q[3] = {D * (((double)px + 0.5 - (double)c.cx) / (double)c.fx) - (double)c.t[0],
                       D * (((double)py + 0.5 - (double)c.cy) / (double)c.fy) - (double)c.t[1],
                       D - (double)c.t[2]};
#pragma unroll
  for (int a = 0; a < 3; a++) w[a] = (double)c.R[a] * q[0] + (double)c.R[3 + a] * q[1] + (double)c.R[6 + a] * q[2];
}

__global__ __launch_bounds__(kBlock) void k_back_project(ViewTable tbl, const gsr_camera *cams, const float *depth,
                                                         float *points, int64_t total) {
  const int v = blockIdx.y;
  const ViewInfo vi = tbl.v[v];
  const gsr_camera c = cams[v];
  const int64_t P = (int64_t)vi.W * vi.H;
  for (int64_t pix = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; pix < P; pix += (int64_t)gridDim.x * blockDim.x) {
    double w[3];
    back_project_pixel(c, vi.W, pix, (double)depth[vi.pix_base + pix], w);
#pragma unroll
    for (int a = 0; a < 3; a++) points[a * total + vi.pix_base + pix] = (float)w[a];
  }
}

// Up to kGroup boxes at a time.  Per axis, the boxes' bounds in ascending
// order and, for every interval between neighbouring bounds, the set of boxes
// whose half-open range holds it: the boxes of a point are the common members
// of its three intervals' sets, found by three binary searches (21 steps for
// 36 boxes, against six compares a box), with the same comparisons decided.
// A box with an undefined bound holds nothing.
constexpr int kGroup = 63, kBounds = 128;

struct BoxTable {
  float bound[3][kBounds];    // padded with +inf
  uint64_t member[3][kBounds];  // member[a][i]: of points with i bounds at or below them
  float raw[3][2 * kGroup];
  uint32_t cnt[kGroup + 1];
};

// Builds the table of boxes[0, g); all threads, barriers included.
__device__ __forceinline__ void box_table(BoxTable &T, const float *boxes, int g) {
  for (int k = threadIdx.x; k < 3 * kBounds; k += blockDim.x) (&T.bound[0][0])[k] = INFINITY;
  for (int k = threadIdx.x; k < 6 * g; k += blockDim.x) {
    const int b = k / 6, c = k - 6 * b;
    const float v = boxes[k], w = boxes[6 * b + (c + 3) % 6];
    T.raw[c % 3][2 * b + c / 3] = v != v || w != w ? INFINITY : v;  // [inf, inf) holds nothing
  }
  for (int k = threadIdx.x; k <= kGroup; k += blockDim.x) T.cnt[k] = 0u;
  __syncthreads();
  for (int k = threadIdx.x; k < 6 * g; k += blockDim.x) {
    const int a = k / (2 * g), j = k - a * 2 * g;
    const float v = T.raw[a][j];
    int rank = 0;
    for (int i = 0; i < 2 * g; i++) {
      const float u = T.raw[a][i];
      rank += (u < v || (u == v && i < j)) ? 1 : 0;
    }
    T.bound[a][rank] = v;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < 3 * kBounds; k += blockDim.x) {
    const int a = k / kBounds, i = k - a * kBounds;
    uint64_t m = 0;
    if (i > 0 && i <= 2 * g) {
      const float at = T.bound[a][i - 1];
      for (int b = 0; b < g; b++)
        m |= (uint64_t)(T.raw[a][2 * b] <= at && !(T.raw[a][2 * b + 1] <= at) ? 1 : 0) << b;
    }
    T.member[a][i] = m;
  }
  __syncthreads();
}

// The boxes that hold a point; `top` is the largest power of two up to 2 g.
__device__ __forceinline__ uint64_t boxes_of(const BoxTable &T, const float w[3], int top) {
  uint64_t m = ~0ull;
#pragma unroll
  for (int a = 0; a < 3; a++) {
    int pos = 0;
    for (int step = top; step >= 1; step >>= 1)
      if (T.bound[a][pos + step - 1] <= w[a]) pos += step;
    m &= T.member[a][pos];
  }
  return m;
}

// Counts `count` points, given by point(i, w), into the boxes: counts[b] +=
// the points in box b.  The whole workgroup calls it.
template <class F>
__device__ __forceinline__ void count_boxes(BoxTable &T, const float *boxes, int nb, uint32_t *counts, int64_t count,
                                            F point) {
  for (int b0 = 0; b0 < nb; b0 += kGroup) {
    const int g = min(kGroup, nb - b0);
    box_table(T, boxes + 6 * b0, g);
    const int top = 1 << (31 - __clz(2 * g));
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) {
      float w[3];
      point(i, w);
      uint64_t m = boxes_of(T, w, top);
      // one LDS atomic per wavefront and box that its points meet
      for (uint64_t any = __ballot(m != 0ull); any; any = __ballot(m != 0ull)) {
        const int leader = __ffsll((unsigned long long)any) - 1;
        const int b = __builtin_amdgcn_readlane(__ffsll((unsigned long long)m) - 1, leader);
        const uint64_t in = __ballot((m >> b) & 1ull);
        if (lane_id() == leader) atomicAdd(&T.cnt[b], (uint32_t)__popcll(in));
        m &= ~(1ull << b);
      }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < g; b += blockDim.x)
      if (T.cnt[b]) atomicAdd(&counts[b0 + b], T.cnt[b]);
    __syncthreads();
  }
}

__global__ __launch_bounds__(kBlock) void k_coverage(ViewTable tbl, const gsr_camera *cams, const float *depth,
                                                     const float *blocks, int n_blocks, uint32_t *counts) {
  __shared__ BoxTable s_table;
  const int v = blockIdx.y;
  const ViewInfo vi = tbl.v[v];
  const gsr_camera c = cams[v];
  count_boxes(s_table, blocks, n_blocks, counts + (int64_t)v * n_blocks, (int64_t)vi.W * vi.H,
              [&](int64_t pix, float w[3]) {
                double wd[3];
                back_project_pixel(c, vi.W, pix, (double)depth[vi.pix_base + pix], wd);
                // the float32 point gsr_back_project stores, so that both count alike
                for (int a = 0; a < 3; a++) w[a] = (float)wd[a];
              });
}

__global__ __launch_bounds__(kBlock) void k_count_points(const float *points, int64_t total,
                                                         const PartitionView *views, const float *boxes, int nb,
                                                         uint32_t *counts) {
  __shared__ BoxTable s_table;
  const int j = blockIdx.y;
  const int64_t first = views[j].first, count = views[j].count;
  count_boxes(s_table, boxes, nb, counts + (int64_t)j * nb, count, [&](int64_t i, float w[3]) {
    for (int a = 0; a < 3; a++) w[a] = points[a * total + first + i];
  });
}

// Workgroups along a view's points: a few thousand points each or more, so
// that the table's building stays small beside them, and the chip filled.
unsigned count_grid(int64_t pmax, int n_rows) {
  const int64_t fill = std::max((int64_t)1, (int64_t)2048 / n_rows);
  return (unsigned)std::max((int64_t)1, std::min((pmax + 4 * kBlock - 1) / (4 * kBlock), fill));
}

__global__ void k_coverage_ratio(ViewTable tbl, int n_blocks, float tau, const uint32_t *counts, float *ratio,
                                 uint8_t *selected) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (int64_t)tbl.n_views * n_blocks) return;
  const ViewInfo vi = tbl.v[k / n_blocks];
  const double np = (double)vi.W * (double)vi.H;
  if (ratio) ratio[k] = (float)((double)counts[k] / np);
  // count / N_p >= tau exactly: tau N_p is exact in double
  if (selected) selected[k] = (double)counts[k] >= (double)tau * np ? 1 : 0;
}

__global__ void k_zero_u32(uint32_t *p, int64_t count) {
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count; k += (int64_t)gridDim.x * blockDim.x)
    p[k] = 0u;
}

int launch_back_project(const ViewTable &views, const gsr_camera *cams, const float *depth, float *points,
                        void *stream) {
  int64_t pmax = 1, total = 0;
  for (int v = 0; v < views.n_views; v++) {
    pmax = std::max(pmax, (int64_t)views.v[v].W * views.v[v].H);
    total += (int64_t)views.v[v].W * views.v[v].H;
  }
  const unsigned gx = (unsigned)std::min((pmax + kBlock - 1) / kBlock, (int64_t)1024);
  hipLaunchKernelGGL(k_back_project, dim3(gx, (unsigned)views.n_views), dim3(kBlock), 0, (hipStream_t)stream, views,
                     cams, depth, points, total);
  return last_err();
}

int launch_count_points(const float *points, int64_t total, const PartitionView *views, int n_sel, int64_t pmax,
                        const float *boxes, int nb, uint32_t *counts, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const int64_t nc = (int64_t)n_sel * nb;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)std::min((nc + kBlock - 1) / kBlock, (int64_t)4096)), dim3(kBlock),
                     0, s, counts, nc);
  hipLaunchKernelGGL(k_count_points, dim3(count_grid(pmax, n_sel), (unsigned)n_sel), dim3(kBlock), 0, s, points, total, views, boxes, nb,
                     counts);
  return last_err();
}

int launch_coverage(const ViewTable &views, const gsr_camera *cams, const float *depth, const float *blocks,
                    int n_blocks, float tau, uint32_t *counts, float *ratio, uint8_t *selected, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const int64_t nc = (int64_t)views.n_views * n_blocks;
  hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)((nc + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, counts, nc);
  int64_t pmax = 1;
  for (int v = 0; v < views.n_views; v++) pmax = std::max(pmax, (int64_t)views.v[v].W * views.v[v].H);
  hipLaunchKernelGGL(k_coverage, dim3(count_grid(pmax, views.n_views), (unsigned)views.n_views), dim3(kBlock), 0, s, views, cams, depth, blocks,
                     n_blocks, counts);
  if (ratio || selected)
    hipLaunchKernelGGL(k_coverage_ratio, dim3((unsigned)((nc + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, views,
                       n_blocks, tau, counts, ratio, selected);
  return last_err();
}

}  // namespace gsr
