// Load-balanced KD-tree scene partition with cutline refinement (Sec. 3.1,
// App. A.5).  The tree is grown on the host, best-first: the leaf with the
// most cameras is split along the longer of its x / y extents, at a
// percentile of the Gaussian centres it holds; a bisection on the percentile
// within [q_min, q_max] moves the cut toward the heavier child.  Each child's
// cameras are those of the parent whose back-projected pixels fall into it
// with a ratio of at least tau (fast camera selection, Sec. 3.2).
//
// Counting pixels into candidate boxes is the only part that touches the
// pixels.  gsr_partition_blocks counts on the host, one evaluated split at a
// time; gsr_partition_blocks_device counts on the GPU, from points resident
// in device memory, and evaluates every percentile the bisection can reach
// (2^steps - 1 of them) for both children in one pass per split, then walks
// the bisection over that table.  Both count the same float32 points with
// the same comparisons, so their results are identical.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <queue>
#include <vector>

#include "gsr.h"
#include "gsr_internal.h"
#include "gsr_stages.h"

namespace {

struct Node {
  float box[6];           // xmin ymin zmin xmax ymax zmax, half-open
  std::vector<int> cams;  // ascending camera ids
  int64_t first, last;    // the Gaussian centres inside the box: a range of the partition's coordinate arrays
  int64_t id;             // creation order
};

bool inside(const float *b, float x, float y, float z) {
  return x >= b[0] && x < b[3] && y >= b[1] && y < b[4] && z >= b[2] && z < b[5];
}

// count / n_pix >= tau, exactly: tau * n_pix is exact in double (24-bit
// mantissa times an integer below 2^29).
bool selected(int64_t count, int64_t n_pix, float tau) {
  return n_pix > 0 && (double)count >= (double)tau * (double)n_pix;
}

struct Input {
  const float *centers;
  int64_t n;
  const int64_t *offsets;
  int n_views;
  float tau;
};

// The bisection's reachable percentiles as a complete binary tree: node k
// holds q; child 2k + 1 follows "left heavier" (q_high = q, q = (q_low + q)/2),
// child 2k + 2 "right heavier" (q_low = q, q = (q_high + q)/2).
std::vector<double> percentile_tree(int steps, double q_min, double q_max) {
  const int64_t count = ((int64_t)1 << steps) - 1;
  std::vector<double> q(count), lo(count), hi(count);
  q[0] = 0.5;
  lo[0] = q_min;
  hi[0] = q_max;
  for (int64_t k = 0; 2 * k + 2 < count; k++) {
    q[2 * k + 1] = 0.5 * (lo[k] + q[k]);
    lo[2 * k + 1] = lo[k];
    hi[2 * k + 1] = q[k];
    q[2 * k + 2] = 0.5 * (hi[k] + q[k]);
    lo[2 * k + 2] = q[k];
    hi[2 * k + 2] = hi[k];
  }
  return q;
}

// Order statistics of a at the sorted, distinct indices idx[lo, hi), the
// range [first, last) of a holding them, by recursive selection.
void order_stats(std::vector<float> &a, int64_t first, int64_t last, const std::vector<int64_t> &idx, size_t lo,
                 size_t hi, std::vector<float> &out) {
  if (lo >= hi) return;
  const size_t mid = (lo + hi) / 2;
  const int64_t k = idx[mid];
  std::nth_element(a.begin() + first, a.begin() + k, a.begin() + last);
  out[mid] = a[k];
  order_stats(a, first, k, idx, lo, mid, out);
  order_stats(a, k + 1, last, idx, mid + 1, hi, out);
}

// Order statistics of a[0, m) at the sorted, distinct indices idx; every value
// lies in [lo, hi).  A histogram over kBins equal cells (the cell of a value
// is monotone in it, also as rounded) tells which cells hold the wanted
// ranks; only their values are collected and selected from.  Two passes over
// the values where the recursive selection takes about ten (splitting 1 M
// centres at 7 ranks, the reordering included: 33 -> 5 ms on one host core).
// Many ranks, and ranges without finite cells, take the recursive selection
// (on a copy: a is left as it is).
struct Selector {
  static constexpr int kBins = 4096;
  static constexpr size_t kMostRanks = 64;
  std::vector<uint16_t> cell;
  std::vector<int64_t> before;
  std::vector<float> copy;

  void operator()(const float *a, int64_t m, float lo, float hi, const std::vector<int64_t> &idx,
                  std::vector<float> &out) {
    const float scale = (float)kBins / (hi - lo);
    if (idx.size() > kMostRanks || m < 4 * kBins || !(std::isfinite(lo) && std::isfinite(scale) && scale > 0.0f)) {
      copy.assign(a, a + m);
      order_stats(copy, 0, m, idx, 0, idx.size(), out);
      return;
    }
    cell.resize((size_t)m);
    before.assign(kBins + 1, 0);
    uint16_t *const cells = cell.data();
    for (int64_t k = 0; k < m; k++) {
      const float c = (a[k] - lo) * scale;
      cells[k] = (uint16_t)(int)(c < (float)(kBins - 1) ? c : (float)(kBins - 1));
    }
    // (four histograms: neighbouring values often share a cell)
    std::vector<uint32_t> hist(4 * kBins, 0u);
    for (int64_t k = 0; k < m; k++) hist[(size_t)(k & 3) * kBins + cells[k]]++;
    for (int c = 0; c < kBins; c++)
      for (int h = 0; h < 4; h++) before[(size_t)c + 1] += hist[(size_t)h * kBins + (size_t)c];
    for (int c = 0; c < kBins; c++) before[(size_t)c + 1] += before[(size_t)c];
    // the wanted cells, numbered in ascending order, and their values
    std::vector<uint8_t> number(kBins, 0);
    std::vector<std::vector<float>> values;
    std::vector<size_t> of_rank(idx.size());
    int prev = -1;
    for (size_t r = 0; r < idx.size(); r++) {
      const int c = (int)(std::upper_bound(before.begin(), before.end(), idx[r]) - before.begin()) - 1;
      if (c != prev) {
        values.emplace_back();
        values.back().reserve((size_t)(before[(size_t)c + 1] - before[(size_t)c]));
        number[(size_t)c] = (uint8_t)values.size();
        prev = c;
      }
      of_rank[r] = values.size() - 1;
    }
    for (int64_t k = 0; k < m; k++)
      if (const int w = number[cells[k]]) values[(size_t)w - 1].push_back(a[k]);
    // (a cell's ranks together: values that crowd into one cell, as in a box
    // stretched by outliers, take one recursive selection, not one per rank)
    std::vector<int64_t> local(idx.size());
    for (size_t r0 = 0, r1; r0 < idx.size(); r0 = r1) {
      std::vector<float> &v = values[of_rank[r0]];
      const int64_t below = *(std::upper_bound(before.begin(), before.end(), idx[r0]) - 1);
      for (r1 = r0; r1 < idx.size() && of_rank[r1] == of_rank[r0]; r1++) local[r1] = idx[r1] - below;
      order_stats(v, 0, (int64_t)v.size(), local, r0, r1, out);
    }
  }
};

// Counts, per camera of `cams` and per box, of that camera's pixels inside
// the box: counts[j * nb + b].
struct HostCounter {
  const float *xyz;  // [3][total]
  int64_t total;
  const int64_t *offsets;
  gsr_status operator()(const std::vector<int> &cams, const float *boxes, int nb, std::vector<int64_t> &counts) {
    counts.assign(cams.size() * (size_t)nb, 0);
    for (size_t j = 0; j < cams.size(); j++)
      for (int64_t k = offsets[cams[j]]; k < offsets[cams[j] + 1]; k++) {
        const float x = xyz[k], y = xyz[total + k], z = xyz[2 * total + k];
        for (int b = 0; b < nb; b++) counts[j * nb + b] += inside(boxes + 6 * b, x, y, z) ? 1 : 0;
      }
    return GSR_OK;
  }
};

struct DeviceCounter {
  const float *xyz;  // device [3][total]
  int64_t total;
  const int64_t *offsets;  // host
  int n_views;
  char *ws;  // device
  hipStream_t stream;
  std::vector<uint32_t> h_counts;
  std::vector<gsr::PartitionView> h_list;

  gsr_status operator()(const std::vector<int> &cams, const float *boxes, int nb, std::vector<int64_t> &counts) {
    counts.assign(cams.size() * (size_t)nb, 0);
    if (cams.empty()) return GSR_OK;
    const gsr::PartitionWs w = gsr::partition_ws(ws, n_views);
    h_list.resize(cams.size());
    int64_t pmax = 1;
    for (size_t j = 0; j < cams.size(); j++) {
      h_list[j].first = offsets[cams[j]];
      h_list[j].count = offsets[cams[j] + 1] - offsets[cams[j]];
      pmax = std::max(pmax, h_list[j].count);
    }
    h_counts.resize(cams.size() * (size_t)nb);
    if (hipMemcpyAsync(w.views, h_list.data(), cams.size() * sizeof(gsr::PartitionView), hipMemcpyHostToDevice,
                       stream) != hipSuccess ||
        hipMemcpyAsync(w.boxes, boxes, (size_t)nb * 6 * sizeof(float), hipMemcpyHostToDevice, stream) != hipSuccess)
      return GSR_ERR_HIP;
    if (gsr::launch_count_points(xyz, total, w.views, (int)cams.size(), pmax, w.boxes, nb, w.counts, stream))
      return GSR_ERR_HIP;
    if (hipMemcpyAsync(h_counts.data(), w.counts, h_counts.size() * sizeof(uint32_t), hipMemcpyDeviceToHost,
                       stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
      return GSR_ERR_HIP;
    for (size_t k = 0; k < h_counts.size(); k++) counts[k] = h_counts[k];
    return GSR_OK;
  }
};

gsr_status check_args(const float *scene_aabb, const float *centers, int64_t n, const float *points,
                      const int64_t *view_offsets, int32_t n_views, int32_t n_blocks, float tau, int32_t refine_steps,
                      float q_min, float q_max, const float *blocks_out) {
  if (!scene_aabb || (!centers && n > 0) || !points || !view_offsets || !blocks_out || n < 0 || n_views < 1 ||
      n_blocks < 1 || refine_steps < 1 || refine_steps > GSR_MAX_REFINE_STEPS ||
      !(q_min > 0.0f && q_min < q_max && q_max < 1.0f) || !std::isfinite(tau))
    return GSR_ERR_INVALID_ARG;
  if (view_offsets[0] != 0) return GSR_ERR_INVALID_ARG;
  for (int v = 0; v < n_views; v++)
    if (view_offsets[v + 1] < view_offsets[v]) return GSR_ERR_INVALID_ARG;
  return GSR_OK;
}

// Alg. 1 with the camera selection of each candidate child by `count`.
// Eager: all reachable percentiles of a split in one call; else one call
// per evaluated split.
template <class Counter>
gsr_status partition(const Input &in, const float *scene_aabb, int n_blocks, int steps, float q_min, float q_max,
                     bool eager, Counter &count, float *blocks_out, uint8_t *assign_out, int32_t *workload_out) {
  const std::vector<double> qtree = percentile_tree(steps, q_min, q_max);
  auto lighter = [](const Node *a, const Node *b) {  // max-heap; equal workloads: earliest node first
    if (a->cams.size() != b->cams.size()) return a->cams.size() < b->cams.size();
    return a->id > b->id;
  };
  std::vector<std::unique_ptr<Node>> all;
  std::priority_queue<Node *, std::vector<Node *>, decltype(lighter)> pq(lighter);
  all.emplace_back(new Node());
  Node *root = all.back().get();
  std::memcpy(root->box, scene_aabb, sizeof root->box);
  for (int c = 0; c < in.n_views; c++) root->cams.push_back(c);
  // The x and y coordinates of the centres inside the scene box, the only ones
  // that cuts compare.  Every node owns a range of them; a split reorders its
  // range, left child first (the order inside a range means nothing).
  const float *C = in.centers;
  std::vector<float> xy[2] = {std::vector<float>((size_t)in.n), std::vector<float>((size_t)in.n)}, right[2];
  int64_t held = 0;
  for (int64_t i = 0; i < in.n; i++) {
    xy[0][(size_t)held] = C[i];
    xy[1][(size_t)held] = C[in.n + i];
    held += inside(root->box, C[i], C[in.n + i], C[2 * in.n + i]) ? 1 : 0;
  }
  right[0].resize((size_t)held);
  right[1].resize((size_t)held);
  root->first = 0;
  root->last = held;
  root->id = 0;
  pq.push(root);
  int64_t next_id = 1;
  std::vector<float> boxes, cuts;
  Selector select_ranks;
  std::vector<int64_t> counts, idx;
  std::vector<int> cams_l, cams_r;

  while ((int32_t)pq.size() < n_blocks) {
    Node *p = pq.top();
    pq.pop();
    const int a = (p->box[3] - p->box[0]) >= (p->box[4] - p->box[1]) ? 0 : 1;
    const int64_t m = p->last - p->first;
    // the cut at percentile q: the order statistic of index floor(q (m - 1))
    // of the node's centres along a, or the extent's middle for m = 0
    const size_t nq = eager ? qtree.size() : 0;
    std::vector<float> cut_of(qtree.size());
    if (m == 0) {
      std::fill(cut_of.begin(), cut_of.end(), 0.5f * (p->box[a] + p->box[3 + a]));
    } else {
      idx.clear();
      for (double q : qtree) idx.push_back((int64_t)std::floor(q * (double)(m - 1)));
      std::vector<int64_t> uniq(idx);
      std::sort(uniq.begin(), uniq.end());
      uniq.erase(std::unique(uniq.begin(), uniq.end()), uniq.end());
      cuts.assign(uniq.size(), 0.0f);
      select_ranks(xy[a].data() + p->first, m, p->box[a], p->box[3 + a], uniq, cuts);
      for (size_t k = 0; k < qtree.size(); k++)
        cut_of[k] = cuts[std::lower_bound(uniq.begin(), uniq.end(), idx[k]) - uniq.begin()];
    }
    auto child_boxes = [&](float cut, float *l, float *r) {
      std::memcpy(l, p->box, 6 * sizeof(float));
      std::memcpy(r, p->box, 6 * sizeof(float));
      l[3 + a] = cut;
      r[a] = cut;
    };
    auto select = [&](const int64_t *cnt_l, const int64_t *cnt_r, int stride) {
      cams_l.clear();
      cams_r.clear();
      for (size_t j = 0; j < p->cams.size(); j++) {
        const int c = p->cams[j];
        const int64_t np = in.offsets[c + 1] - in.offsets[c];
        if (selected(cnt_l[j * stride], np, in.tau)) cams_l.push_back(c);
        if (selected(cnt_r[j * stride], np, in.tau)) cams_r.push_back(c);
      }
    };
    if (eager) {
      boxes.resize(12 * nq);
      for (size_t k = 0; k < nq; k++) child_boxes(cut_of[k], &boxes[12 * k], &boxes[12 * k + 6]);
      const gsr_status st = count(p->cams, boxes.data(), (int)(2 * nq), counts);
      if (st != GSR_OK) return st;
    }
    float box_l[6], box_r[6];
    int64_t k = 0;  // node of the percentile tree being evaluated
    for (int it = 0; it < steps; it++) {
      child_boxes(cut_of[k], box_l, box_r);
      if (eager) {
        select(&counts[2 * k], &counts[2 * k + 1], (int)(2 * nq));
      } else {
        float pair[12];
        std::memcpy(pair, box_l, sizeof box_l);
        std::memcpy(pair + 6, box_r, sizeof box_r);
        const gsr_status st = count(p->cams, pair, 2, counts);
        if (st != GSR_OK) return st;
        select(&counts[0], &counts[1], 2);
      }
      if (cams_l.size() > cams_r.size())
        k = 2 * k + 1;
      else if (cams_r.size() > cams_l.size())
        k = 2 * k + 2;
      else
        break;
    }
    // the children of the last evaluated split
    all.emplace_back(new Node());
    Node *L = all.back().get();
    all.emplace_back(new Node());
    Node *R = all.back().get();
    std::memcpy(L->box, box_l, sizeof box_l);
    std::memcpy(R->box, box_r, sizeof box_r);
    L->cams = cams_l;
    R->cams = cams_r;
    // left of the cut to the front of the range, the others behind them
    int64_t to = p->first, others = 0;
    for (int64_t j = p->first; j < p->last; j++) {
      const float u = xy[a][(size_t)j], w = xy[1 - a][(size_t)j];
      const bool left = u < box_l[3 + a];
      xy[a][(size_t)to] = u;
      xy[1 - a][(size_t)to] = w;
      right[0][(size_t)others] = u;
      right[1][(size_t)others] = w;
      to += left ? 1 : 0;
      others += left ? 0 : 1;
    }
    std::copy(right[0].begin(), right[0].begin() + others, xy[a].begin() + to);
    std::copy(right[1].begin(), right[1].begin() + others, xy[1 - a].begin() + to);
    L->first = p->first;
    L->last = R->first = to;
    R->last = p->last;
    L->id = next_id++;
    R->id = next_id++;
    pq.push(L);
    pq.push(R);
  }
  std::vector<Node *> leaves;
  while (!pq.empty()) {
    leaves.push_back(pq.top());
    pq.pop();
  }
  std::sort(leaves.begin(), leaves.end(), [](const Node *x, const Node *y) { return x->id < y->id; });
  for (int b = 0; b < n_blocks; b++) {
    std::memcpy(blocks_out + 6 * b, leaves[b]->box, 6 * sizeof(float));
    if (workload_out) workload_out[b] = (int32_t)leaves[b]->cams.size();
    if (assign_out) {
      std::memset(assign_out + (int64_t)b * in.n_views, 0, (size_t)in.n_views);
      for (int c : leaves[b]->cams) assign_out[(int64_t)b * in.n_views + c] = 1;
    }
  }
  return GSR_OK;
}

}  // namespace

extern "C" gsr_status gsr_partition_blocks(const float *scene_aabb, const float *centers, int64_t n,
                                           const float *points, const int64_t *view_offsets, int32_t n_views,
                                           int32_t n_blocks, float tau, int32_t refine_steps, float q_min,
                                           float q_max, float *blocks_out, uint8_t *assign_out,
                                           int32_t *workload_out) {
  const gsr_status st = check_args(scene_aabb, centers, n, points, view_offsets, n_views, n_blocks, tau,
                                   refine_steps, q_min, q_max, blocks_out);
  if (st != GSR_OK) return st;
  const Input in{centers, n, view_offsets, n_views, tau};
  HostCounter count{points, view_offsets[n_views], view_offsets};
  return partition(in, scene_aabb, n_blocks, refine_steps, q_min, q_max, false, count, blocks_out, assign_out,
                   workload_out);
}

extern "C" gsr_status gsr_partition_workspace_size(int32_t n_views, size_t *bytes) {
  if (n_views < 1 || !bytes) return GSR_ERR_INVALID_ARG;
  *bytes = gsr::partition_ws_bytes(n_views);
  return GSR_OK;
}

extern "C" gsr_status gsr_partition_blocks_device(const float *scene_aabb, const float *centers, int64_t n,
                                                  const float *points, const int64_t *view_offsets, int32_t n_views,
                                                  int32_t n_blocks, float tau, int32_t refine_steps, float q_min,
                                                  float q_max, void *ws, size_t ws_bytes, void *stream,
                                                  float *blocks_out, uint8_t *assign_out, int32_t *workload_out) {
  const gsr_status st = check_args(scene_aabb, centers, n, points, view_offsets, n_views, n_blocks, tau,
                                   refine_steps, q_min, q_max, blocks_out);
  if (st != GSR_OK) return st;
  if (!ws || ws_bytes < gsr::partition_ws_bytes(n_views)) return GSR_ERR_WORKSPACE_TOO_SMALL;
  const Input in{centers, n, view_offsets, n_views, tau};
  DeviceCounter count{points, view_offsets[n_views], view_offsets, n_views, (char *)ws, (hipStream_t)stream, {}, {}};
  // every reachable percentile's two children in one pass when the boxes fit
  const bool eager = 2 * (((int64_t)1 << refine_steps) - 1) <= GSR_MAX_COVERAGE_BLOCKS;
  return partition(in, scene_aabb, n_blocks, refine_steps, q_min, q_max, eager, count, blocks_out, assign_out,
                   workload_out);
}
