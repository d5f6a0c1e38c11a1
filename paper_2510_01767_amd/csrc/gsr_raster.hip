// Tile rasterization kernels (gfx950): front-to-back compositing (the
// blending sum of Sec. 3.2), the L1 image gradient and the back-to-front
// reverse pass, as plain per-tile kernels and as one persistent fused kernel.
//
// Work decomposition.  One workgroup (4 wavefronts, 256 lanes) owns one tile
// of 256 pixels, one lane per pixel.  The tile's ordered entry list is
// streamed through LDS in batches of B records.  Each wavefront owns a
// 64-pixel strip of the tile and each 16-lane row of it a 16-pixel
// sub-block; the batch is culled against the strip, then against each
// sub-block: an entry is kept for a sub-block only if the ellipse on which
// its alpha reaches alpha_min (its "reach", precomputed per record) can
// touch a pixel centre of the sub-block.  Each row then walks its own kept
// list in depth order.  Culled entries have alpha < alpha_min at every pixel
// they skip, so the result is identical to evaluating them; on city-scale
// scenes most entries of a tile list miss most sub-blocks, which is where
// the time would otherwise go.
//
// Reverse pass.  Each row reduces the nine per-pixel terms of its entry
// (the moments of dL/dp over the pixel offset, which the reverse projection
// maps through the record's conic, then dL/dopacity and dL/dcolour) by a
// reduce-scatter over its 16 lanes; nine lanes then either add the sums to
// the record's gradient slot with device atomics, or (the other variants the
// autotuner weighs) into a per-batch LDS accumulator flushed with one device
// atomic per (entry, component).
#include <hip/hip_runtime.h>

#include "gsr_cull.h"
#include "gsr_device.h"

namespace gsr {

struct TileCtx {
  int64_t t;  // global tile id
  int v;      // view
  ViewInfo vi;
  int px, py;  // this lane's pixel
  bool inside;
  int64_t start, end;  // entry range [start, end) in keys
  int64_t pix;         // pixel index within the view
  float wx0, wx1, wy0, wy1;  // pixel-centre box of this lane's wavefront
  int sw, sh, snx;           // sub-block width and height, sub-blocks per strip row
};

template <int TW, int TH>
__device__ __forceinline__ void tile_ctx(const KWs &ws, const ViewInfo *views, int n_views, int64_t t,
                                         TileCtx &c) {
  static_assert(TW * TH == kBlock && 64 % TW == 0, "tile must be 256 pixels, whole rows per wavefront");
  constexpr int kRows = 64 / TW;
  c.t = t;
  c.v = view_of_tile(views, n_views, t);
  c.vi = views[c.v];
  const int64_t local = t - c.vi.tile_base;
  const int tx0 = (int)(local % c.vi.tiles_x) * TW, ty0 = (int)(local / c.vi.tiles_x) * TH;
  // Each wavefront owns a strip of 64 pixels (TW x kRows) and each 16-lane
  // row of it a sub-block of 16 pixels: 4 x 4 for 8- and 16-wide tiles, 8 x 2
  // for 32-wide ones (SNX sub-blocks side by side).
  constexpr int SW = TW == 32 ? 8 : 4, SH = 16 / SW, SNX = TW / SW;
  static_assert((kRows / SH) * SNX == 4, "four sub-blocks per strip");
  const int wave = threadIdx.x >> 6, lane = (int)threadIdx.x & 63, row = lane >> 4, sl = lane & 15;
  c.px = tx0 + (row % SNX) * SW + sl % SW;
  c.py = ty0 + wave * kRows + (row / SNX) * SH + sl / SW;
  c.sw = SW;
  c.sh = SH;
  c.snx = SNX;
  c.inside = c.px < c.vi.W && c.py < c.vi.H;
  c.pix = (int64_t)c.py * c.vi.W + c.px;
  c.start = ws.tile_start[t];
  c.end = min((int64_t)ws.tile_start[t + 1], ws.capacity);
  if (c.end < c.start) c.end = c.start;
  c.wx0 = (float)tx0 + 0.5f;
  c.wx1 = (float)(tx0 + TW) - 0.5f;
  c.wy0 = (float)(ty0 + wave * kRows) + 0.5f;
  c.wy1 = c.wy0 + (float)(kRows - 1);
}

// A batch of records in LDS as separate arrays: the four 16-lane rows of a
// wavefront read four different entries at once, which in a 64-byte record
// array would start on the same banks.  r2 holds the colour and, in place of
// the record's exponent bound (that is kept with the reach, for the culling),
// the record's index.  A batch has at most B - 1 entries; the last place is
// kNone, an entry whose alpha is 0 at every pixel, which fills up the shorter
// lists of a wavefront's four sub-blocks: no step of a walk then asks whether
// its row still has an entry.  Its record index is the spare slot behind the
// records': the reverse walk's products with its alpha of 0 are NaN where the
// image gradient is infinite or NaN, and a NaN is added somewhere.  (With that, the stop kept as lane masks and the
// banked reduction below, a walk takes 25 vector operations an entry forward
// and 66 in reverse.  The fused kernel before -> with them, a city of 8 M
// Gaussians in 32 full-HD views 7.65 -> 7.20 ms, a cloud of 20 M in 8 views of
// 3840 x 2160 45.9 -> 44.4; a block of 3 M in 16 views, which waits for its
// atomics, 4.84 -> 4.81.)
template <int B>
struct LdsBatch {
  static constexpr int kCap = B - 1, kNone = B - 1;
  float4 r0[B], r1[B], r2[B];
  float2 cull[B];  // reach, base-2 pmin
};

template <int B>
__device__ __forceinline__ void init_none(LdsBatch<B> &s, const KWs &ws, float *s_depth = nullptr) {
  if (threadIdx.x == 0) {
    if (s_depth) s_depth[LdsBatch<B>::kNone] = 0.0f;
    constexpr int e = LdsBatch<B>::kNone;
    s.r0[e] = s.r1[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    s.r2[e] = make_float4(0.0f, 0.0f, 0.0f, __uint_as_float((uint32_t)ws.vn));
    s.cull[e] = make_float2(-1.0f, 0.0f);
  }
}

template <int B>
__device__ __forceinline__ LdsRec rec_at(const LdsBatch<B> &s, int j) {
  LdsRec R;
  R.r0 = s.r0[j];
  R.r1 = s.r1[j];
  R.r2 = s.r2[j];
  const float2 q = s.cull[j];
  R.reach = q.x;
  R.r2.w = q.y;
  return R;
}

template <int B>
__device__ __forceinline__ void put_rec(LdsBatch<B> &s, int j, uint32_t idx, const float4 &r0, const float4 &r1,
                                        const float4 &r2, const uint4 &r3) {
  s.r0[j] = r0;
  s.r1[j] = r1;
  s.r2[j] = make_float4(r2.x, r2.y, r2.z, __uint_as_float(idx));
  s.cull[j] = make_float2(__uint_as_float(r3.w), r2.w);
}

template <int B>
__device__ __forceinline__ void load_batch(const KWs &ws, int64_t lo, int nb, LdsBatch<B> &s_rec,
                                           float *s_depth = nullptr) {
  if ((int)threadIdx.x < nb) {
    const uint32_t r = (uint32_t)ws.keys[lo + threadIdx.x];
    const float4 *rec = rec_ptr(ws, r);
    const uint4 r3 = reinterpret_cast<const uint4 *>(rec)[3];
    put_rec(s_rec, threadIdx.x, r, rec[0], rec[1], rec[2], r3);
    if (s_depth) s_depth[threadIdx.x] = __uint_as_float(r3.z);
  }
}

// The same in two halves, for launches with few tiles: the loads of a batch
// into registers, its key's while the batch before it is culled and its
// record's while that one is walked, then the registers into LDS.
struct NextRec {
  uint32_t idx;
  float4 r0, r1, r2;
  uint4 r3;
};

__device__ __forceinline__ void next_key(const KWs &ws, int64_t lo, int nb, NextRec &q) {
  if ((int)threadIdx.x < nb) q.idx = (uint32_t)ws.keys[lo + threadIdx.x];
}

__device__ __forceinline__ void next_rec(const KWs &ws, int nb, NextRec &q) {
  if ((int)threadIdx.x < nb) {
    const float4 *rec = rec_ptr(ws, q.idx);
    q.r0 = rec[0];
    q.r1 = rec[1];
    q.r2 = rec[2];
    q.r3 = reinterpret_cast<const uint4 *>(rec)[3];
  }
}

template <int B>
__device__ __forceinline__ void store_next(const NextRec &q, int nb, LdsBatch<B> &s_rec, float *s_depth) {
  if ((int)threadIdx.x < nb) {
    put_rec(s_rec, threadIdx.x, q.idx, q.r0, q.r1, q.r2, q.r3);
    if (s_depth) s_depth[threadIdx.x] = __uint_as_float(q.r3.z);
  }
}

// The kept entries of the batch for each of the wavefront's four
// sub-blocks, in list order: an entry is tested against the strip's circle,
// then each band of sub-blocks gets its interval and each sub-block two
// compares.  The lists are filled up with kNone to the length of the longest
// and on to a multiple of four.  Returns the count of this lane's own
// sub-block; kmax: the longest count, the same in every lane.
template <int B>
__device__ __forceinline__ int sub_lists(const LdsBatch<B> &s_rec, int nb, const TileCtx &c, uint8_t (*lists)[B],
                                         int &kmax) {
  static_assert(B <= 256 && B % 4 == 0, "byte indices, lists padded to a multiple of four");
  const int lane = lane_id();
  const uint64_t below = (1ull << lane) - 1ull;
  int cnt[4] = {0, 0, 0, 0};
  for (int jb = 0; jb < nb; jb += 64) {
    const int j = jb + lane;
    const LdsRec R = rec_at(s_rec, j < nb ? j : 0);
    const bool strip = j < nb && reaches_strip(R, c.wx0, c.wx1, c.wy0, c.wy1);
    const ReachShape S = reach_shape(R);
    float xl = 3.0e38f, xr = -3.0e38f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const float bx0 = c.wx0 + (float)((q % c.snx) * c.sw), by0 = c.wy0 + (float)((q / c.snx) * c.sh);
      if (q % c.snx == 0) band_interval(R, S, by0, by0 + (float)(c.sh - 1), xl, xr);
      const float x0 = (bx0 - R.r0.x) - R.r0.z, x1 = ((bx0 + (float)(c.sw - 1)) - R.r0.x) - R.r0.z;
      const bool keep = strip && (S.thin || (x1 >= xl && x0 <= xr));
      const uint64_t m = __ballot(keep);
      if (keep) lists[q][cnt[q] + __popcll(m & below)] = (uint8_t)j;
      cnt[q] += __popcll(m);
    }
  }
  kmax = max(max(cnt[0], cnt[1]), max(cnt[2], cnt[3]));
  const int row = lane >> 4, own = row < 2 ? (row == 0 ? cnt[0] : cnt[1]) : (row == 2 ? cnt[2] : cnt[3]);
  for (int k = own + (lane & 15); k < ((kmax + 3) & ~3); k += 16) lists[row][k] = (uint8_t)LdsBatch<B>::kNone;
  return own;
}

// The batch that a tile pass left in LDS: entries [lo, lo + nb) of the list
// in s_rec, and this wavefront's culled list of it (cnt entries in s_list).  nb == 0: nothing usable.
struct Resident {
  int64_t lo;
  int nb, cnt;  // cnt: this lane's sub-block list length
};

// Front-to-back compositing of one tile.  Returns the colour, the final
// transmittance and `last` (list entries processed before the stop, or the
// list length).  With HIST it stores, for every evaluated entry, the
// transmittance in front of it (0 when the entry was skipped).  Batches
// start at c.start + k (B - 1); the last one loaded stays resident (`res`).
// The pair update is branch-free: a skipped pair adds 0 * colour and keeps T.
// With DEPTH it also composites the records' depths, D = sum d alpha T
// (the depth form of the blending sum, Sec. 3.2), from s_depth.  With COUNT
// (profiling) it counts the pairs this lane evaluates after the culling and
// the pairs it blends.
//
// FEW (launches with few tiles): four entries at a time, and the next batch's
// loads in flight while this one is culled and walked.  With a wavefront or
// two per SIMD nothing hides the latency of a step (list byte, record,
// exponential) or of a batch (key, then record), so the four entries' list
// bytes, records and alphas, which do not depend on one another, are in flight
// together, and only the transmittance update goes entry by entry, in the same
// order and with the same operations.
constexpr int kAhead = 4;

template <int B, bool HIST, bool FEW, bool DEPTH = false, bool COUNT = false>
__device__ __forceinline__ void tile_forward(const KWs &ws, const KOpts &o, const TileCtx &c, LdsBatch<B> &s_rec,
                                             uint8_t (*s_list)[4][B], float C[3], float &T, int &last,
                                             float *hist, Resident &res, float *s_depth = nullptr,
                                             float *D = nullptr, uint32_t *n_eval = nullptr,
                                             uint32_t *n_blend = nullptr) {
  constexpr int kCap = LdsBatch<B>::kCap;
  const float pxc = (float)c.px + 0.5f, pyc = (float)c.py + 0.5f;
  const float amax = o.alpha_max;
  const int wave = threadIdx.x >> 6, row = ((int)threadIdx.x & 63) >> 4;
  T = 1.0f;
  C[0] = C[1] = C[2] = 0.0f;
  bool done = !c.inside;
  bool stopped = false;
  last = 0;
  res.nb = 0;
  [[maybe_unused]] NextRec next = {};
  if (FEW && c.start < c.end) {
    const int nb = (int)min((int64_t)kCap, c.end - c.start);
    next_key(ws, c.start, nb, next);
    next_rec(ws, nb, next);
  }
  for (int64_t b = c.start; b < c.end; b += kCap) {
    if (__syncthreads_and(done)) break;
    const int nb = (int)min((int64_t)kCap, c.end - b);
    const int nb_next = FEW ? (int)max((int64_t)0, min((int64_t)kCap, c.end - b - kCap)) : 0;
    if constexpr (FEW) {
      store_next(next, nb, s_rec, DEPTH ? s_depth : nullptr);
      next_key(ws, b + kCap, nb_next, next);
    } else {
      load_batch(ws, b, nb, s_rec, DEPTH ? s_depth : nullptr);
    }
    __syncthreads();
    int kmax;
    const int cnt = sub_lists<B>(s_rec, nb, c, s_list[wave], kmax);
    if constexpr (FEW) next_rec(ws, nb_next, next);
    __syncthreads();
    res.lo = b;
    res.nb = nb;
    res.cnt = cnt;
    const uint8_t *mine = s_list[wave][row];
    // each 16-lane row walks its own sub-block's list (kNone past its end)
    if constexpr (FEW) {
      const bool stopped_before = stopped;
      for (int k0 = 0; k0 < kmax; k0 += kAhead) {
        if (__ballot(!done) == 0ull) break;
        const uint32_t bytes = *reinterpret_cast<const uint32_t *>(mine + k0);
        int j[kAhead];
        float4 r2[kAhead];
        PairAlpha a[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
          j[u] = (int)(bytes >> (8 * u) & 255u);
          r2[u] = s_rec.r2[j[u]];
          a[u] = pair_alpha<false>(pxc, pyc, s_rec.r0[j[u]], s_rec.r1[j[u]], amax);
        }
#pragma unroll
        for (int u = 0; u < kAhead; u++) {
          const bool hit = !done && a[u].in && a[u].alpha >= o.alpha_min;
          const float Tn = T * (1.0f - a[u].alpha);
          const bool stop = hit && Tn < o.T_min;
          const bool take = hit && !stop;
          const float w = take ? a[u].alpha * T : 0.0f;
          // (a stopped lane does not take 0 times an infinite colour either)
          C[0] = done ? C[0] : __fmaf_rn(w, r2[u].x, C[0]);
          C[1] = done ? C[1] : __fmaf_rn(w, r2[u].y, C[1]);
          C[2] = done ? C[2] : __fmaf_rn(w, r2[u].z, C[2]);
          if (DEPTH) *D = __fmaf_rn(w, s_depth[j[u]], *D);
          T = take ? Tn : T;
          last = stop ? j[u] : last;
          stopped = stopped || stop;
          done = done || stop;
        }
      }
      if (stopped && !stopped_before) last += (int)(b - c.start);
    } else if (!done) {
      int j = 0;
      bool stop = false;
      for (int k = 0; k < kmax && !stop; k++) {
        j = mine[k];
        const PairAlpha a = pair_alpha<false>(pxc, pyc, s_rec.r0[j], s_rec.r1[j], amax);
        const float4 col = s_rec.r2[j];
        const float Tn = T * (1.0f - a.alpha);
        // as lane masks: a compare for each condition, the rest scalar
        const uint64_t hits = __ballot(a.in) & __ballot(a.alpha >= o.alpha_min), low = __ballot(Tn < o.T_min);
        stop = __builtin_amdgcn_inverse_ballot_w64(hits & low);
        const bool take = __builtin_amdgcn_inverse_ballot_w64(hits & ~low);
        const float w = take ? a.alpha * T : 0.0f;
        C[0] = __fmaf_rn(w, col.x, C[0]);
        C[1] = __fmaf_rn(w, col.y, C[1]);
        C[2] = __fmaf_rn(w, col.z, C[2]);
        if (DEPTH) *D = __fmaf_rn(w, s_depth[j], *D);
        if (COUNT) {
          *n_eval += j != LdsBatch<B>::kNone ? 1u : 0u;
          *n_blend += take ? 1u : 0u;
        }
        if (HIST && j != LdsBatch<B>::kNone && !stop) hist[(b + j) * 256 + threadIdx.x] = take ? T : 0.0f;
        T = take ? Tn : T;
      }
      if (stop) {
        last = (int)(b - c.start) + j;  // the lane left the walk at the entry that stopped it
        stopped = done = true;
      }
    }
  }
  if (!stopped) last = c.inside ? (int)(c.end - c.start) : 0;
}

// Reduce-scatter of the nine terms over each 16-lane row, in four steps
// between lanes i and i ^ 7, i ^ 1, i ^ 2, i ^ 8 (row_half_mirror, two quad
// permutations, row_ror:8), each leaving a lane about half of the components
// it carried, summed with its partner's.  The first and the last step choose
// by groups of four lanes, which the bank mask of a DPP addition does by
// itself: two additions into one register, where choosing inside the quads
// takes two selects and an addition.  22 operations (27 with selects
// throughout, 44 with four full row sums and a select); lane q < 9 of a row
// ends with component q, so that an entry's nine words leave in three quads
// of lanes: with four quads, which an operation fewer would give, the fused
// kernel took 5.58 ms instead of 4.81 on the 16-view block.  All 64 lanes must
// be active.
// The waits are the two that a DPP read needs after the write of its operand.
__device__ __forceinline__ float row_reduce_scatter(const float v[9], uint64_t odd, uint64_t high) {
  float a0 = v[0], a1 = v[2], a2 = v[1], a3 = v[3], a4 = v[8], s0, s1;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %2, %2, %2 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %3, %3, %3 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %4, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %7, %7 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %1, %8, %8 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %2, %9, %9 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %3, %10, %10 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_e64 %5, %2, %0, %11\n\t"
      "v_cndmask_b32_e64 %0, %0, %2, %11\n\t"
      "v_cndmask_b32_e64 %6, %3, %1, %11\n\t"
      "v_cndmask_b32_e64 %1, %1, %3, %11\n\t"
      "v_add_f32_dpp %0, %5, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %6, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_e64 %5, %1, %0, %12\n\t"
      "v_cndmask_b32_e64 %0, %0, %1, %12\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %0, %5, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc"
      : "+v"(a0), "+v"(a1), "+v"(a2), "+v"(a3), "+v"(a4), "=&v"(s0), "=&v"(s1)
      : "v"(v[4]), "v"(v[6]), "v"(v[5]), "v"(v[7]), "s"(odd), "s"(high));
  return a0;
}

// Back-to-front reverse pass of one tile.  g = dL/dC_out of this lane's
// pixel, T its final transmittance (recovered entry by entry unless the
// forward stored it).  Each contributing pair gives nine terms, summed per
// entry into its slot: the five moments of dL/dp over the pixel offset, then
// dL/dopacity and dL/dcolour.
//   RED = 0: per row entry, the reduce-scatter of the nine terms over the
//            row and one device atomic per component from nine lanes.
//   RED = 1: contributing lanes add their terms into an LDS accumulator
//            of the batch (ds_add_f32, combining the four wavefronts); one
//            device atomic per non-zero (entry, component) after the batch.
//   RED = 2, 3, 4: as 1 after DPP sums over lane quads (2), over 16-lane
//            rows (3), or a reduce-scatter over 16-lane rows (4).
// Batches are aligned like the forward's (c.start + k (B - 1)), so when the
// forward's last batch `res` is the first one needed here it is used as it
// sits in LDS, culled lists included.
//   FEW (RED = 0): four entries at a time, as in the forward pass: their
//            alphas and reciprocals together, the transmittance and suffix
//            updates in order, then the four reductions together.
template <int B, int RED, bool HIST, bool FEW>
__device__ __forceinline__ void tile_backward(const KWs &ws, const KOpts &o, const TileCtx &c, LdsBatch<B> &s_rec,
                                              uint8_t (*s_list)[4][B], float (*s_acc)[9], int *s_max, float T,
                                              int last, const float g[3], const float *hist, Resident res) {
  constexpr int kCap = LdsBatch<B>::kCap;
  const float pxc = (float)c.px + 0.5f, pyc = (float)c.py + 0.5f;
  const float amax = o.alpha_max;  // as in the forward pass
  const int wave = threadIdx.x >> 6, lane = lane_id();
  // the reduce-scatter's lane roles: the lanes with bit 0 and bit 1 set
  constexpr uint64_t kOdd = 0xAAAAAAAAAAAAAAAAull, kHigh = 0xCCCCCCCCCCCCCCCCull;
  const int comp_of_lane = (lane & 15) < 9 ? lane & 15 : -1;
  // gS = sum_ch g_ch S_ch with S the colour composited behind the current
  // entry (T_final bg to start); dL/dalpha_i = T_i (g . c_i) - gS / (1 - alpha_i)
  float gS = T * (g[0] * o.bg[0] + g[1] * o.bg[1] + g[2] * o.bg[2]);
  const bool active = c.inside && (g[0] != 0.0f || g[1] != 0.0f || g[2] != 0.0f);
  // A wavefront with an infinite or undefined g walks entry by entry: an entry
  // that none of its pixels blends is then left out by itself (its terms, g
  // times 0, would not be 0).  Asked here, once a tile: asked for each of the
  // four entries it took 2 % of a step on three small views.
  const bool by_four = FEW && __ballot(!(fabsf(g[0]) + fabsf(g[1]) + fabsf(g[2]) < INFINITY)) == 0ull;
  __syncthreads();
  if (threadIdx.x == 0) *s_max = 0;
  __syncthreads();
  if (active && last > 0) atomicMax(s_max, last);
  __syncthreads();
  const int top = *s_max;  // entries [0, top) of the list can contribute
  [[maybe_unused]] NextRec next = {};
  [[maybe_unused]] bool loaded = false;
  for (int64_t lo = c.start + (int64_t)((top - 1) / kCap) * kCap; top > 0 && lo >= c.start; lo -= kCap) {
    const int nb_top = (int)min((int64_t)kCap, c.start + top - lo);
    int nb, cnt;
    // the batch in front, loaded while this one is walked (all of its entries
    // lie below `top`)
    const int nb_next = FEW && lo > c.start ? kCap : 0;
    __syncthreads();
    if (res.nb > 0 && res.lo == lo) {
      // the forward's last batch, still in LDS with this wavefront's list
      nb = res.nb;
      cnt = res.cnt;
      res.nb = 0;
      if (RED >= 1)
        for (int e = threadIdx.x; e < nb * 9; e += blockDim.x) (&s_acc[0][0])[e] = 0.0f;
      __syncthreads();
    } else {
      nb = nb_top;
      if (FEW && loaded) store_next(next, nb, s_rec, nullptr);
      else load_batch(ws, lo, nb, s_rec);
      if (RED >= 1)
        for (int e = threadIdx.x; e < nb * 9; e += blockDim.x) (&s_acc[0][0])[e] = 0.0f;
      __syncthreads();
      int longest;
      cnt = sub_lists<B>(s_rec, nb, c, s_list[wave], longest);
      __syncthreads();
    }
    if constexpr (FEW) {
      next_key(ws, lo - kCap, nb_next, next);
      next_rec(ws, nb_next, next);
      loaded = nb_next > 0;
    }
    // entries at or past `top` contribute to no pixel: the walk starts below
    // them in the longest list (a shorter one may still hold some: jj_last
    // leaves them out)
    const uint8_t *mine = s_list[wave][(lane & 63) >> 4];
    while (cnt > 0 && (int)mine[cnt - 1] >= nb_top) cnt--;
    int kmax = max(cnt, __shfl_xor(cnt, 16));  // the longest of the wavefront's four row lists
    kmax = __builtin_amdgcn_readfirstlane(max(kmax, __shfl_xor(kmax, 32)));  // uniform: a scalar loop counter
    int jj_last = active ? last - (int)(lo - c.start) : 0;  // this pixel's entries: jj < jj_last
    asm("" : "+v"(jj_last));  // one register, not recomputed at every entry
    if constexpr (FEW) {
      static_assert(RED == 0 && !HIST, "the device-atomic form only");
      for (int k0 = by_four ? (kmax - 1) & ~(kAhead - 1) : -1; k0 >= 0; k0 -= kAhead) {
        const uint32_t bytes = *reinterpret_cast<const uint32_t *>(mine + k0);
        int jj[kAhead];
        float4 r2[kAhead];
        PairAlpha a[kAhead];
        bool contrib[kAhead], any = false;
#pragma unroll
        for (int u = kAhead - 1; u >= 0; u--) {
          jj[u] = (int)(bytes >> (8 * u) & 255u);
          r2[u] = s_rec.r2[jj[u]];
          a[u] = pair_alpha<true>(pxc, pyc, s_rec.r0[jj[u]], s_rec.r1[jj[u]], amax);
          contrib[u] = a[u].in && jj[u] < jj_last && a[u].alpha >= o.alpha_min;
          any = any || contrib[u];
        }
        if (__ballot(any) == 0ull) continue;
        float v[kAhead][9];
#pragma unroll
        for (int u = kAhead - 1; u >= 0; u--) {
          const float al = contrib[u] ? a[u].alpha : 0.0f;
          const float inv_om = __builtin_amdgcn_rcpf(1.0f - al);
          const float Ti = T * inv_om, wgt = al * Ti;
          // (0 for a pixel that the entry does not blend into: its suffix stays
          // as it is also where the colour or g is not finite)
          const float gc = contrib[u] ? __fmaf_rn(g[2], r2[u].z, __fmaf_rn(g[1], r2[u].y, g[0] * r2[u].x)) : 0.0f;
          const float dLda = __fmaf_rn(Ti, gc, -gS * inv_om);
          gS = __fmaf_rn(wgt, gc, gS);
          T = Ti;
          const float dLdam = (contrib[u] && a[u].raw < o.alpha_max) ? dLda : 0.0f;
          const float gp = dLdam * a[u].alpha;
          const float gpx = gp * a[u].dx, gpy = gp * a[u].dy;
          v[u][0] = gpx;
          v[u][1] = gpy;
          v[u][2] = gpx * a[u].dx;
          v[u][3] = gpx * a[u].dy;
          v[u][4] = gpy * a[u].dy;
          v[u][5] = dLdam * a[u].G;
          for (int ch = 0; ch < 3; ch++) v[u][6 + ch] = g[ch] * wgt;
        }
        float x[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; u++) x[u] = row_reduce_scatter(v[u], kOdd, kHigh);
#pragma unroll
        for (int u = kAhead - 1; u >= 0; u--)
          if (comp_of_lane >= 0 && x[u] != 0.0f)
            unsafeAtomicAdd(&ws.grad2d[(int64_t)__float_as_uint(r2[u].w) * kGrad2dStride + comp_of_lane], x[u]);
      }
    }
    for (int k = by_four ? -1 : kmax - 1; k >= 0; k--) {
      const int jj = mine[k];
      const int64_t j = lo + jj;
      const PairAlpha a = pair_alpha<true>(pxc, pyc, s_rec.r0[jj], s_rec.r1[jj], amax);
      const bool contrib = a.in && jj < jj_last && a.alpha >= o.alpha_min;
      if (__ballot(contrib) == 0ull) continue;
      const float4 r2 = s_rec.r2[jj];
      // Every lane evaluates the terms (all finite: alpha <= 0.99).  The
      // non-contributing lanes take alpha = 0 here: 1 / (1 - 0) is exactly 1,
      // so their T and suffix stay as they are and they add exact zeros.
      // 1 / (1 - alpha) by the hardware reciprocal (1 ulp): T and the
      // suffix only feed gradients, never a discrete decision.
      const float al = contrib ? a.alpha : 0.0f;
      const float inv_om = __builtin_amdgcn_rcpf(1.0f - al);
      const float Ti = HIST ? (contrib ? hist[j * 256 + threadIdx.x] : T) : T * inv_om;
      const float wgt = al * Ti;
      const float col[3] = {r2.x, r2.y, r2.z};
      float v[9];
      const float gc = __fmaf_rn(g[2], col[2], __fmaf_rn(g[1], col[1], g[0] * col[0]));
      const float dLda = __fmaf_rn(Ti, gc, -gS * inv_om);
      gS = __fmaf_rn(wgt, gc, gS);
#pragma unroll
      for (int ch = 0; ch < 3; ch++) v[6 + ch] = g[ch] * wgt;
      // the geometric terms vanish where alpha is clamped at alpha_max
      const float dLdam = (contrib && a.raw < o.alpha_max) ? dLda : 0.0f;
      const float gp = dLdam * a.alpha;  // dL/dp
      v[5] = dLdam * a.G;
      // the moments of dL/dp over the pixel offsets d = pixel - mean:
      // sum gp dx, gp dy, gp dx^2, gp dx dy, gp dy^2.  The geometric 2D
      // gradient is linear in them with the record's conic Q as coefficients
      // (dL/dmean = Q (m0, m1), dL/dQ = -(m2 / 2, m3, m4 / 2)), so the
      // reverse projection applies Q once per record instead of every pixel
      // applying it here.
      const float gpx = gp * a.dx, gpy = gp * a.dy;
      v[0] = gpx;
      v[1] = gpy;
      v[2] = gpx * a.dx;
      v[3] = gpx * a.dy;
      v[4] = gpy * a.dy;
      T = Ti;
      if (RED == 0) {
        // the row's reduce-scatter, then one device atomic per component from
        // nine lanes of the row into its entry's gradient slot
        const float u = row_reduce_scatter(v, kOdd, kHigh);
        if (comp_of_lane >= 0 && u != 0.0f)
          unsafeAtomicAdd(&ws.grad2d[(int64_t)__float_as_uint(r2.w) * kGrad2dStride + comp_of_lane], u);
      } else if (RED == 1) {
        if (contrib) {
#pragma unroll
          for (int q = 0; q < 9; q++)
            if (v[q] != 0.0f) atomicAdd(&s_acc[jj][q], v[q]);
        }
      } else if (RED == 3) {
        // row sums (four DPP steps leave every lane of a 16-lane row with the
        // row's total), then lane 16 row + q adds component q: one LDS atomic
        // instruction per entry, four rows per address
        // (the nine chains interleaved step by step, so no DPP result is
        // read back-to-back)
#pragma unroll
        for (int q = 0; q < 9; q++) v[q] += dpp_or_zero<0xB1>(v[q]);   // quad_perm [1,0,3,2]
#pragma unroll
        for (int q = 0; q < 9; q++) v[q] += dpp_or_zero<0x4E>(v[q]);   // quad_perm [2,3,0,1]
#pragma unroll
        for (int q = 0; q < 9; q++) v[q] += dpp_or_zero<0x141>(v[q]);  // row_half_mirror
#pragma unroll
        for (int q = 0; q < 9; q++) v[q] += dpp_or_zero<0x140>(v[q]);  // row_mirror
        const int q = lane & 15;
        float mine = v[0];
#pragma unroll
        for (int k = 1; k < 9; k++) mine = q == k ? v[k] : mine;
        if (q < 9 && mine != 0.0f) atomicAdd(&s_acc[jj][q], mine);
      } else if (RED == 4) {
        const float u = row_reduce_scatter(v, kOdd, kHigh);
        if (comp_of_lane >= 0 && u != 0.0f) atomicAdd(&s_acc[jj][comp_of_lane], u);
      } else {
        // quad sums (two DPP steps), then one LDS atomic per quad and component
#pragma unroll
        for (int q = 0; q < 9; q++) v[q] += dpp_or_zero<0xB1>(v[q]);  // quad_perm [1,0,3,2]
#pragma unroll
        for (int q = 0; q < 9; q++) v[q] += dpp_or_zero<0x4E>(v[q]);  // quad_perm [2,3,0,1]
#pragma unroll
        for (int q = 0; q < 9; q++)
          if ((lane & 3) == 0 && v[q] != 0.0f) atomicAdd(&s_acc[jj][q], v[q]);
      }
    }
    if (RED >= 1) {
      __syncthreads();
      for (int e = threadIdx.x; e < nb * 9; e += blockDim.x) {
        const int jj = e / 9, q = e - jj * 9;
        const float val = s_acc[jj][q];
        if (val != 0.0f) unsafeAtomicAdd(&ws.grad2d[(int64_t)__float_as_uint(s_rec.r2[jj].w) * kGrad2dStride + q], val);
      }
    }
  }
}

__device__ __forceinline__ float block_sum_fixed(float x, float *s_w) {
  x = wave_sum_lane63(x);
  if (lane_id() == 63) s_w[threadIdx.x >> 6] = x;
  __syncthreads();
  const float r = (s_w[0] + s_w[1]) + (s_w[2] + s_w[3]);
  __syncthreads();
  return r;
}

// COUNT (profiling): pair_counts[p] = pairs blended into pixel p,
// pair_counts[pixels_total + p] = pairs its lane evaluated.
template <int TW, int TH, int B, bool HIST, bool DEPTH, bool COUNT, bool FEW>
__global__ __launch_bounds__(kBlock) void k_raster_fwd(KWs ws, KOpts o, int64_t tile_lo, int64_t tile_count,
                                                       float *images, int n_views, float *depth,
                                                       uint32_t *pair_counts) {
  __shared__ LdsBatch<B> s_rec;
  __shared__ float s_depth[DEPTH ? B : 1];
  alignas(16) __shared__ uint8_t s_list[4][4][B];  // [wavefront][sub-block][entry index in the batch]
  __shared__ ViewInfo s_views[GSR_MAX_VIEWS];
  for (int v = threadIdx.x; v < n_views; v += blockDim.x) s_views[v] = ws.views[v];
  init_none(s_rec, ws, DEPTH ? s_depth : nullptr);
  __syncthreads();
  const int64_t b = xcd_remap(blockIdx.x, tile_count);
  if (b >= tile_count) return;
  TileCtx c;
  tile_ctx<TW, TH>(ws, s_views, n_views, tile_lo + b, c);
  float C[3], T;
  int last;
  Resident res;
  float D = 0.0f;
  uint32_t n_eval = 0u, n_blend = 0u;
  tile_forward<B, HIST, FEW, DEPTH, COUNT>(ws, o, c, s_rec, s_list, C, T, last, ws.history, res, s_depth, &D,
                                      &n_eval, &n_blend);
  if (c.inside) {
    const int64_t P = (int64_t)c.vi.W * c.vi.H;
    float *img = images + c.vi.pix_base * 3;
#pragma unroll
    for (int ch = 0; ch < 3; ch++) img[ch * P + c.pix] = __fmaf_rn(T, o.bg[ch], C[ch]);
    ws.pix_T[c.vi.pix_base + c.pix] = T;
    ws.pix_last[c.vi.pix_base + c.pix] = (uint32_t)last;
    if (DEPTH) depth[c.vi.pix_base + c.pix] = D;
    if (COUNT) {
      pair_counts[c.vi.pix_base + c.pix] = n_blend;
      pair_counts[ws.pixels_total + c.vi.pix_base + c.pix] = n_eval;
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_l1(KWs ws, KOpts o, int64_t tile_lo, int64_t tile_count,
                                               const float *images, const float *targets, int n_views, int tw,
                                               int th) {
  __shared__ float s_w[4];
  __shared__ ViewInfo s_views[GSR_MAX_VIEWS];
  for (int v = threadIdx.x; v < n_views; v += blockDim.x) s_views[v] = ws.views[v];
  __syncthreads();
  const int64_t t = tile_lo + blockIdx.x;
  const int v = view_of_tile(s_views, n_views, t);
  const ViewInfo vi = s_views[v];
  const int64_t local = t - vi.tile_base;
  const int px = (int)(local % vi.tiles_x) * tw + (int)(threadIdx.x % tw);
  const int py = (int)(local / vi.tiles_x) * th + (int)(threadIdx.x / tw);
  float acc = 0.0f;
  if (px < vi.W && py < vi.H) {
    const int64_t P = (int64_t)vi.W * vi.H;
    const int64_t base = vi.pix_base * 3 + (int64_t)py * vi.W + px;
#pragma unroll
    for (int ch = 0; ch < 3; ch++) {
      const float d = images[base + ch * P] - targets[base + ch * P];
      acc += fabsf(d);
      ws.pix_dLdC[base + ch * P] = d > 0.0f ? vi.loss_scale : (d < 0.0f ? -vi.loss_scale : 0.0f);
    }
  }
  const float s = block_sum_fixed(acc, s_w);
  if (threadIdx.x == 0) ws.tile_loss[t] = s;
}

template <int TW, int TH, int B, int RED, bool HIST, bool FEW>
__global__ __launch_bounds__(kBlock) void k_raster_bwd(KWs ws, KOpts o, int64_t tile_lo, int64_t tile_count,
                                                       const float *dLdC, int n_views) {
  __shared__ LdsBatch<B> s_rec;
  alignas(16) __shared__ uint8_t s_list[4][4][B];  // [wavefront][sub-block][entry index in the batch]
  __shared__ float s_acc[RED >= 1 ? B : 1][9];
  __shared__ int s_max;
  __shared__ ViewInfo s_views[GSR_MAX_VIEWS];
  for (int v = threadIdx.x; v < n_views; v += blockDim.x) s_views[v] = ws.views[v];
  init_none(s_rec, ws);
  __syncthreads();
  const int64_t b = xcd_remap(blockIdx.x, tile_count);
  if (b >= tile_count) return;
  TileCtx c;
  tile_ctx<TW, TH>(ws, s_views, n_views, tile_lo + b, c);
  float g[3] = {0.f, 0.f, 0.f};
  float T = 1.0f;
  int last = 0;
  if (c.inside) {
    const int64_t P = (int64_t)c.vi.W * c.vi.H;
    const float *d = dLdC + c.vi.pix_base * 3 + c.pix;
    g[0] = d[0];
    g[1] = d[P];
    g[2] = d[2 * P];
    T = ws.pix_T[c.vi.pix_base + c.pix];
    last = (int)ws.pix_last[c.vi.pix_base + c.pix];
  }
  tile_backward<B, RED, HIST, FEW>(ws, o, c, s_rec, s_list, s_acc, &s_max, T, last, g, ws.history,
                              Resident{0, 0, 0});
}

// Persistent fused forward + L1 + reverse pass.  Workgroups take tiles
// (in `order` when given) until their counter passes the last tile; no
// workgroup ever waits for another.  Workgroup class x = blockIdx mod 8 takes
// items x, x + 8, x + 16, ... from a counter of its own: the hardware hands
// consecutive workgroups to the 8 XCDs in turn, so each counter is shared by
// one XCD's workgroups instead of one counter by the whole chip.  The grid
// is a multiple of 8, so every class has workgroups and every tile is taken.
// The reduce-scatter form (RED 0) is held to 64 VGPRs, eight wavefronts per
// SIMD, which its LDS also allows (a few registers spill); the LDS
// accumulator forms are limited by their LDS anyway.
template <int TW, int TH, int B, int RED, bool HIST, bool FEW>
__global__ __launch_bounds__(kBlock, RED == 0 && !HIST && !FEW ? 8 : 1) void k_fused(KWs ws, KOpts o, const float *targets, float *images,
                                                  int n_views, const uint32_t *order) {
  __shared__ LdsBatch<B> s_rec;
  alignas(16) __shared__ uint8_t s_list[4][4][B];  // [wavefront][sub-block][entry index in the batch]
  __shared__ float s_acc[RED >= 1 ? B : 1][9];
  __shared__ int s_max;
  __shared__ float s_w[4];
  __shared__ int64_t s_item;
  __shared__ ViewInfo s_views[GSR_MAX_VIEWS];
  for (int v = threadIdx.x; v < n_views; v += blockDim.x) s_views[v] = ws.views[v];
  init_none(s_rec, ws);
  float *hist = ws.history;
  const int cls = (int)(blockIdx.x & 7u);
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_item = cls + 8 * (int64_t)atomicAdd(&ws.hdr->queue[cls][0], 1u);
    __syncthreads();
    const int64_t item = s_item;
    if (item >= ws.tiles_total) break;
    const int64_t t = order ? (int64_t)order[item] : item;
    TileCtx c;
    tile_ctx<TW, TH>(ws, s_views, n_views, t, c);
    float C[3], T;
    int last;
    Resident res;
    tile_forward<B, HIST, FEW>(ws, o, c, s_rec, s_list, C, T, last, hist, res);
    float g[3] = {0.f, 0.f, 0.f};
    float acc = 0.0f;
    if (c.inside) {
      const int64_t P = (int64_t)c.vi.W * c.vi.H;
      const int64_t base = c.vi.pix_base * 3 + c.pix;
#pragma unroll
      for (int ch = 0; ch < 3; ch++) {
        const float out = __fmaf_rn(T, o.bg[ch], C[ch]);
        images[base + ch * P] = out;
        const float d = out - targets[base + ch * P];
        acc += fabsf(d);
        g[ch] = d > 0.0f ? c.vi.loss_scale : (d < 0.0f ? -c.vi.loss_scale : 0.0f);
      }
      ws.pix_T[c.vi.pix_base + c.pix] = T;
      ws.pix_last[c.vi.pix_base + c.pix] = (uint32_t)last;
    }
    const float s = block_sum_fixed(acc, s_w);
    if (threadIdx.x == 0) ws.tile_loss[t] = s;
    tile_backward<B, RED, HIST, FEW>(ws, o, c, s_rec, s_list, s_acc, &s_max, T, last, g, hist, res);
  }
}

// ------------------------------------------------------- longest list first
// The persistent kernel takes tiles in descending list length (bins of 4
// entries), so the longest tiles start first and the tail of the launch is
// made of short ones.  The order only schedules work: every tile's result is
// the same whichever workgroup computes it, whenever.

// (the histogram of the list lengths comes out of the scan)
//
// Every workgroup scans the 1024 bins for itself, then places its tiles with
// one device atomic per bin it holds (the ranks inside the workgroup from LDS
// atomics): the bins of the many short or empty tiles would otherwise take
// one atomic per tile on a single address.
__global__ __launch_bounds__(kBlock) void k_order_scatter(KWs ws) {
  constexpr int kPer = kOrderBins / kBlock;
  __shared__ uint32_t s_cnt[kOrderBins], s_base[kOrderBins], s_first[kOrderBins], s_wave[kBlock / 64];
  uint32_t x[kPer], sum = 0u;
#pragma unroll
  for (int k = 0; k < kPer; k++) {
    x[k] = ws.hdr->order_bins[kPer * threadIdx.x + k];
    sum += x[k];
  }
  uint32_t incl = sum;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t y = __shfl_up(incl, (unsigned)off);
    if (lane_id() >= off) incl += y;
  }
  if (lane_id() == 63) s_wave[threadIdx.x >> 6] = incl;
  __syncthreads();
  uint32_t first = incl - sum;
  for (int w = 0; w < (int)(threadIdx.x >> 6); w++) first += s_wave[w];
#pragma unroll
  for (int k = 0; k < kPer; k++) {
    s_first[kPer * threadIdx.x + k] = first;
    first += x[k];
  }
  for (int64_t t0 = (int64_t)blockIdx.x * blockDim.x; t0 < ws.tiles_total; t0 += (int64_t)gridDim.x * blockDim.x) {
    for (int k = threadIdx.x; k < kOrderBins; k += blockDim.x) s_cnt[k] = 0u;
    __syncthreads();
    const int64_t t = t0 + threadIdx.x;
    int bin = -1;
    uint32_t off = 0u;
    if (t < ws.tiles_total) {
      bin = order_bin(ws.tile_start[t + 1] - ws.tile_start[t]);
      off = atomicAdd(&s_cnt[bin], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kOrderBins; k += blockDim.x)
      if (s_cnt[k]) s_base[k] = s_first[k] + atomicAdd(&ws.hdr->order_cursor[k], s_cnt[k]);
    __syncthreads();
    if (bin >= 0) ws.tile_order[s_base[bin] + off] = (uint32_t)t;
    __syncthreads();
  }
}

int launch_tile_order(const KWs &ws, void *stream) {
  const int g = (int)min((int64_t)512, (ws.tiles_total + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_order_scatter, dim3(g), dim3(kBlock), 0, (hipStream_t)stream, ws);
  return last_err();
}

// ---------------------------------------------------------------- launchers

#define GSR_TILE_DISPATCH(TW_, TH_, CALL)                                   \
  if (o.tile_w == TW_ && o.tile_h == TH_) {                                 \
    if (lds_batch == 64) {                                                  \
      constexpr int B = 64;                                                 \
      CALL(TW_, TH_, B);                                                    \
    } else if (lds_batch == 128) {                                          \
      constexpr int B = 128;                                                \
      CALL(TW_, TH_, B);                                                    \
    } else {                                                                \
      constexpr int B = 256;                                                \
      CALL(TW_, TH_, B);                                                    \
    }                                                                       \
    return last_err();                                                      \
  }

// reverse-pass kernels also select the reduction mode; the stored-history
// variant always takes the row reduce-scatter (4)
#define GSR_RED_CALL(KER, TILES, TW_, TH_, B_, ...)                                                              \
  do {                                                                                                           \
    if (hist) hipLaunchKernelGGL((KER<TW_, TH_, B_, 4, true, false>), grid, block, 0, s, __VA_ARGS__);           \
    else if (red == 4) hipLaunchKernelGGL((KER<TW_, TH_, B_, 4, false, false>), grid, block, 0, s, __VA_ARGS__); \
    else if (red == 3) hipLaunchKernelGGL((KER<TW_, TH_, B_, 3, false, false>), grid, block, 0, s, __VA_ARGS__); \
    else if (red == 2) hipLaunchKernelGGL((KER<TW_, TH_, B_, 2, false, false>), grid, block, 0, s, __VA_ARGS__); \
    else if (red == 1) hipLaunchKernelGGL((KER<TW_, TH_, B_, 1, false, false>), grid, block, 0, s, __VA_ARGS__); \
    else if ((TILES) <= kFewTiles)                                                                               \
      hipLaunchKernelGGL((KER<TW_, TH_, kFewTilesBatch, 0, false, true>), grid, block, 0, s, __VA_ARGS__);                  \
    else hipLaunchKernelGGL((KER<TW_, TH_, B_, 0, false, false>), grid, block, 0, s, __VA_ARGS__);               \
  } while (0)

int launch_raster_fwd(const KWs &ws, const KOpts &o, int64_t tile_lo, int64_t tile_count, float *images,
                      int n_views, int store_history, int lds_batch, float *depth, uint32_t *pair_counts,
                      void *stream) {
  if (tile_count <= 0) return 0;
  const dim3 grid((unsigned)xcd_grid(tile_count)), block(kBlock);
  hipStream_t s = (hipStream_t)stream;
  const bool few = tile_count <= kFewTiles;
#define CALL_FWD(a, b_, B)                                                                                        \
  do {                                                                                                              \
    if (pair_counts)                                                                                                \
      hipLaunchKernelGGL((k_raster_fwd<a, b_, B, false, false, true, false>), grid, block, 0, s, ws, o, tile_lo,           \
                         tile_count, images, n_views, depth, pair_counts);                                          \
    else if (depth && few)                                                                                          \
      hipLaunchKernelGGL((k_raster_fwd<a, b_, kFewTilesBatch, false, true, false, true>), grid, block, 0, s, ws, o, tile_lo,     \
                         tile_count, images, n_views, depth, pair_counts);                                          \
    else if (depth)                                                                                                 \
      hipLaunchKernelGGL((k_raster_fwd<a, b_, B, false, true, false, false>), grid, block, 0, s, ws, o, tile_lo,    \
                         tile_count, images, n_views, depth, pair_counts);                                          \
    else if (store_history)                                                                                         \
      hipLaunchKernelGGL((k_raster_fwd<a, b_, B, true, false, false, false>), grid, block, 0, s, ws, o, tile_lo,           \
                         tile_count, images, n_views, depth, pair_counts);                                          \
    else if (few)                                                                                                   \
      hipLaunchKernelGGL((k_raster_fwd<a, b_, kFewTilesBatch, false, false, false, true>), grid, block, 0, s, ws, o, tile_lo,    \
                         tile_count, images, n_views, depth, pair_counts);                                          \
    else                                                                                                            \
      hipLaunchKernelGGL((k_raster_fwd<a, b_, B, false, false, false, false>), grid, block, 0, s, ws, o, tile_lo,          \
                         tile_count, images, n_views, depth, pair_counts);                                          \
  } while (0)
  GSR_TILE_DISPATCH(16, 16, CALL_FWD)
  GSR_TILE_DISPATCH(32, 8, CALL_FWD)
  GSR_TILE_DISPATCH(8, 32, CALL_FWD)
#undef CALL_FWD
  return (int)hipErrorInvalidValue;
}

int launch_l1(const KWs &ws, const KOpts &o, int64_t tile_lo, int64_t tile_count, const float *images,
              const float *targets, int n_views, void *stream) {
  if (tile_count <= 0) return 0;
  hipLaunchKernelGGL(k_l1, dim3((unsigned)tile_count), dim3(kBlock), 0, (hipStream_t)stream, ws, o, tile_lo,
                     tile_count, images, targets, n_views, o.tile_w, o.tile_h);
  return last_err();
}

int launch_raster_bwd(const KWs &ws, const KOpts &o, int64_t tile_lo, int64_t tile_count, const float *dLdC,
                      int n_views, int use_history, int lds_batch, int red, void *stream) {
  if (tile_count <= 0) return 0;
  const dim3 grid((unsigned)xcd_grid(tile_count)), block(kBlock);
  hipStream_t s = (hipStream_t)stream;
  const bool hist = use_history != 0;
#define CALL_BWD(a, b_, B) GSR_RED_CALL(k_raster_bwd, tile_count, a, b_, B, ws, o, tile_lo, tile_count, dLdC, n_views)
  GSR_TILE_DISPATCH(16, 16, CALL_BWD)
  GSR_TILE_DISPATCH(32, 8, CALL_BWD)
  GSR_TILE_DISPATCH(8, 32, CALL_BWD)
#undef CALL_BWD
  return (int)hipErrorInvalidValue;
}

int launch_fused(const KWs &ws, const KOpts &o, const float *targets, float *images, int n_views, int use_history,
                 int lds_batch, int red, int grid_blocks, void *stream) {
  // a multiple of 8: every workgroup class of the per-XCD counters is present
  const dim3 grid((unsigned)xcd_grid(grid_blocks > 8 ? grid_blocks : 8)), block(kBlock);
  hipStream_t s = (hipStream_t)stream;
  const uint32_t *order = ws.tile_order;
  const bool hist = use_history != 0;
#define CALL_FUSED(a, b_, B) GSR_RED_CALL(k_fused, ws.tiles_total, a, b_, B, ws, o, targets, images, n_views, order)
  GSR_TILE_DISPATCH(16, 16, CALL_FUSED)
  GSR_TILE_DISPATCH(32, 8, CALL_FUSED)
  GSR_TILE_DISPATCH(8, 32, CALL_FUSED)
#undef CALL_FUSED
  return (int)hipErrorInvalidValue;
}

}  // namespace gsr
