// Foveal neural-point splat, forward (Sec. 3.3 sub-frustum + depth cull;
// Sec. 4 "Inference": one count, one scan and one fill over all pyramid
// layers and all crops).
//
// Fragments go straight to per-pixel segments: emission counts each layer
// pixel's fragments, a scan turns the counts into segment offsets, and each
// fragment's place in its segment is its rank by (float32 bits of t.z,
// point index) among the segment's fragments -- so the lists come out in
// blend order with no global sort, and deterministically (atomics only
// place survivors and fragments in scratch lists whose order the ranking
// removes).
//   k_pt_prep      per-pixel counters, the survivor and fragment counts and
//                  the pixel scan's temporary zeroed, crop grid
//   k_pt_select    one thread per point, points read once for all crops:
//                  projection, layer, crop footprints, then the depth cull;
//                  survivors (depth key, entry, fragment offset) compacted in
//                  the same pass, one 64-bit atomic per workgroup for the
//                  survivor and fragment bases, and the survivor that opens
//                  each emission chunk
//   k_pt_ord_*     where the counted fragments make dense lists: the survivors
//                  into the order of screen buckets (count, scan, move)
//   k_pt_emit      one workgroup per chunk of 1024 consecutive fragments,
//                  one thread per survivor of the chunk: writes its
//                  fragments (layer pixel, weight | point index, depth key),
//                  counts them per pixel and takes each one a free place in
//                  its pixel's segment (the counting atomics' old values)
//   scan           per-pixel counts -> segment offsets
//   k_pt_scatter   each fragment's record (point index, depth key, weight,
//                  pixel) to its segment place: no atomics
//   k_pt_resolve   dense lists: a wave or a workgroup per pixel ranks its
//                  segment and composites it
//   k_pt_rank      otherwise, one thread per segment place: the record's rank
//                  in its segment -> its final place (the lanes of one segment
//                  read the same records)
//   k_pt_blend     one thread per layer pixel walks its list front to back
#include <hip/hip_fp16.h>

#include "pt_device.h"

namespace vrs {

struct SplatWs {
  size_t surv, ctr, live, frag_count,   // survivors: (entry, depth key, fragment offset,
                                        // fragments | bucket << 16)
      left,
      chunk_first,                 // per emission chunk: the survivor holding its first fragment
      fkey0, fval0, fdep, fslot,   // fragments in emission order, place in segment
      seg,                         // (point index, depth key, weight, pixel) per segment place
      fkey1, fval1,                // fragments in blend order
      pcnt, poff,                  // per layer pixel: fragment count, segment offsets [P + 1]
      surv2, ord_hist,             // dense lists: survivors by bucket (0: none), the buckets' counts
      hide,                        // per view pixel: depth that hides points (0: none kept),
                               // over the fragments
      grid, scan_tmp, total;
  int ord_parts;
  int gx, gy;   // crop-lookup grid cells per view row / column
  int64_t vn, pix_total;
};

// Fragments per emission workgroup (one chunk of the fragment range).
constexpr int kEmitFrags = 1024;

// Fragments per layer pixel above which lists are dense: survivors are put
// in screen order before the emission and k_pt_resolve ranks and blends.
constexpr int64_t kRsDense = 12;
// Per-pixel mark (in place of its fragment count) of a list that k_pt_resolve
// leaves to k_pt_rank and k_pt_blend.
constexpr uint32_t kRsLeft = 0xffffffffu;
// Screen buckets of dense survivors, and those counted per workgroup.
constexpr int kOrdBuckets = 2048, kOrdBlock = 512;

static int64_t pyramid_pixels(const vrs_crop* crops, int n_crops, int levels) {
  int64_t s = 0;
  for (int k = 0; k < n_crops; ++k)
    for (int l = 0; l < levels; ++l) {
      int64_t e = crops[k].size >> l;
      s += e * e;
    }
  return s;
}

// Crop-lookup grid: cells of kGridCell x kGridCell view pixels, per view.
constexpr int kGridCell = 32;

static bool splat_layout(int64_t np, int nv, int W, int H, const vrs_crop* crops, int n_crops,
                         int levels, int64_t max_frags, SplatWs* L) {
  if (np < 0 || nv < 1 || nv > VRS_MAX_VIEWS || n_crops < 0 || n_crops > VRS_MAX_CROPS ||
      levels < 1 || levels > VRS_MAX_LEVELS || max_frags < 0 || (n_crops > 0 && !crops) ||
      W < 1 || H < 1)
    return false;
  L->gx = (W + kGridCell - 1) / kGridCell;
  L->gy = (H + kGridCell - 1) / kGridCell;
  L->vn = np * nv;
  L->pix_total = pyramid_pixels(crops, n_crops, levels);
  const int64_t vn = std::max<int64_t>(L->vn, 1), mf = std::max<int64_t>(max_frags, 1);
  const int64_t pt = std::max<int64_t>(L->pix_total, 1);
  Carver c;
  L->surv = c.take(vn * 16);
  L->ctr = c.take(12);   // survivors in the low word, fragments in the high word,
  L->live = L->ctr;
  L->frag_count = L->ctr + 4;
  L->left = L->ctr + 8;   // then the pixels that k_pt_resolve leaves to rank and blend
  L->chunk_first = c.take((mf / kEmitFrags + 2) * 4);
  L->pcnt = c.take(pt * 4);
  L->poff = c.take((pt + 1) * 4);
  L->surv2 = L->ord_hist = 0;
  L->ord_parts = 0;
  if (max_frags > kRsDense * L->pix_total && n_crops > 0) {
    const int64_t most = std::min(vn, mf);   // a survivor has a fragment
    L->ord_parts = (int)std::min<int64_t>(512, div_up(most, 4 * kOrdBlock));
    L->surv2 = c.take(most * 16);
    L->ord_hist = c.take(((size_t)L->ord_parts + 1) * kOrdBuckets * 8);
  }
  L->grid = c.take((size_t)nv * L->gx * L->gy * 4);
  L->scan_tmp = c.take(scan_tmp_bytes(pt));
  L->fkey0 = c.take(mf * 4);
  L->fval0 = c.take(mf * 8);
  L->fdep = c.take(mf * 4);
  L->fslot = c.take(mf * 4);
  L->seg = c.take(mf * 16);
  L->fkey1 = c.take(mf * 4);
  L->fval1 = c.take(mf * 8);
  {
    // pairs that look a pixel up, about, against four pixels of the image; the
    // selection is done with it when the first fragment is written, so it lies
    // over the fragments
    double area = 0.0;
    for (int k = 0; k < n_crops; ++k) area += (double)crops[k].size * crops[k].size;
    const double pixels = (double)nv * W * H;
    L->hide = 0;
    if ((double)L->vn * area * 4.0 >= pixels * pixels) {
      L->hide = L->fkey0;
      c.off = std::max(c.off, L->hide + (size_t)pixels * 4);
    }
  }
  L->total = c.off;
  return true;
}

static bool splat_layout_for(int64_t np, int n_views, const vrs_view* views, const vrs_crop* crops,
                             int n_crops, int levels, int64_t max_frags, SplatWs* L) {
  if (!views || n_views < 1) return false;
  return splat_layout(np, n_views, views[0].width, views[0].height, crops, n_crops, levels,
                      max_frags, L);
}

// host: crop table with packed-pyramid and packed-output bases; with a
// device placement table the host origins are not used (nor checked)
bool make_crops(const vrs_crop* crops, int n_crops, int levels, const KViews& kv, KCrops* out,
                const vrs_crop_place* place, bool check_origins = true) {
  if (n_crops < 0 || n_crops > VRS_MAX_CROPS || levels < 1 || levels > VRS_MAX_LEVELS)
    return false;
  if (n_crops > 0 && !crops) return false;
  out->n = n_crops;
  out->place = reinterpret_cast<const int4*>(place);
  int64_t pb = 0, ob = 0;
  const int unit = 1 << (levels - 1);
  for (int k = 0; k < n_crops; ++k) {
    const vrs_crop& c = crops[k];
    if (c.view < 0 || c.view >= kv.n) return false;
    if (c.size < unit || c.size % unit != 0) return false;
    const KView& v = kv.v[c.view];
    if (c.size > v.W || c.size > v.H) return false;
    if (!place && check_origins &&
        (c.x0 < 0 || c.y0 < 0 || c.x0 + c.size > v.W || c.y0 + c.size > v.H))
      return false;
    KCrop& d = out->c[k];
    d.view = c.view; d.x0 = c.x0; d.y0 = c.y0; d.size = c.size;
    d.gx = c.gaze_x; d.gy = c.gaze_y;
    d.mx0 = v.W - c.size;
    d.my0 = v.H - c.size;
    d.pix_base = (int)pb;
    d.out_base = (int)ob;
    for (int l = 0; l < levels; ++l) pb += (int64_t)(c.size >> l) * (c.size >> l);
    ob += (int64_t)3 * c.size * c.size;
    if (pb > (int64_t(1) << 30) || ob > (int64_t(1) << 30)) return false;
  }
  return true;
}

struct PtArgs {
  float cov_min, slack;
  int levels;
  uint32_t view_mask;  // views that own at least one crop
  int ord_side;        // screen buckets' side in pixels (0: survivors are never reordered)
};

// Smallest side whose buckets over all crops fit.
static int ord_side(const vrs_crop* crops, int n_crops) {
  for (int side = 8;; ++side) {
    int64_t n = 0;
    for (int k = 0; k < n_crops; ++k) {
      const int64_t t = (crops[k].size + side - 1) / side;
      n += t * t;
    }
    if (n <= kOrdBuckets) return side;
  }
}

// ---------------------------------------------------------------- select
// Crop-lookup grid: per view and cell, the bit set of crops that a point
// whose pixel lies in the cell may reach.  A footprint at layer l < levels
// reaches at most 2^(l-1) + 1 view pixels beyond its crop, so crop k is
// listed in every cell that meets [x0 - 2^levels - 2, x0 + size + 2^levels + 2)
// (likewise y); border cells extend to infinity so that lookups of pixels
// outside the view clamp to them.
// ox, oy: the crops' origins (a workgroup's copy in LDS).
__device__ inline void pt_cropgrid_cell(const KCrops& crops, int levels, int gx, int gy,
                                        int64_t idx, const int* ox, const int* oy,
                                        uint32_t* __restrict__ grid) {
  const int v = (int)(idx / ((int64_t)gx * gy));
  const int cell = (int)(idx - (int64_t)v * gx * gy);
  const int cy = cell / gx, cx = cell - cy * gx;
  const int M = (1 << levels) + 2;
  const int64_t lo_x = cx == 0 ? INT32_MIN : (int64_t)cx * kGridCell;
  const int64_t hi_x = cx == gx - 1 ? INT32_MAX : (int64_t)(cx + 1) * kGridCell;
  const int64_t lo_y = cy == 0 ? INT32_MIN : (int64_t)cy * kGridCell;
  const int64_t hi_y = cy == gy - 1 ? INT32_MAX : (int64_t)(cy + 1) * kGridCell;
  uint32_t mask = 0;
  for (int k = 0; k < crops.n; ++k) {
    const KCrop& c = crops.c[k];
    if (c.view != v) continue;
    const int cx0 = ox[k], cy0 = oy[k];
    const int64_t x0 = (int64_t)cx0 - M, x1 = (int64_t)cx0 + c.size + M;
    const int64_t y0 = (int64_t)cy0 - M, y1 = (int64_t)cy0 + c.size + M;
    if (x0 < hi_x && x1 > lo_x && y0 < hi_y && y1 > lo_y) mask |= 1u << k;
  }
  grid[idx] = mask;
}

// Crop k placed on its gaze point g: the crop of size S centred on the gaze,
// x0 = clamp(rint(g.x - S/2), 0, W - S) (ties to even), y0 likewise; the
// gaze itself in the last two words.
__device__ inline int4 place_crop(const KCrops& kc, int k, float2 g) {
  const float h = 0.5f * (float)kc.c[k].size;
  const float fx = rintf(g.x - h), fy = rintf(g.y - h);
  // clamp in float first: a non-finite or huge gaze gives a valid origin
  const float cx = fminf(fmaxf(fx, 0.0f), (float)kc.c[k].mx0);
  const float cy = fminf(fmaxf(fy, 0.0f), (float)kc.c[k].my0);
  return make_int4(cx == cx ? (int)cx : 0, cy == cy ? (int)cy : 0, __float_as_int(g.x),
                   __float_as_int(g.y));
}

// Crop origins from gaze points on the device (Sec. 4 "Inference": the eye
// tracker is read after the periphery is rendered), one thread per crop.
__global__ void k_place_crops(const float2* __restrict__ gaze, KCrops kc, int4* __restrict__ out) {
  const int k = threadIdx.x;
  if (k >= kc.n) return;
  out[k] = place_crop(kc, k, gaze[k]);
}

// Per-call set-up in one launch: the per-pixel fragment counters, the
// survivor and fragment counts and the pixel scan's temporary zeroed, and
// the crop-lookup grid.
// With gaze, the crops are placed here as well (what the placement entry
// point computes): every workgroup places them for its own cells, the first
// one writes the placement table that the later kernels read.
__global__ void k_pt_prep(uint32_t* __restrict__ pcnt, int64_t pix_total,
                          uint64_t* __restrict__ ctr, uint32_t* __restrict__ scan_tmp,
                          int64_t scan_words, KCrops crops, int nv, int levels, int gx, int gy,
                          uint32_t* __restrict__ grid, const float2* __restrict__ gaze,
                          int4* __restrict__ place_out, const float* __restrict__ depth,
                          const float* __restrict__ tfinal, PtArgs a, float* __restrict__ hide,
                          int64_t pixels) {
  const int64_t cells = (int64_t)nv * gx * gy;
  const int64_t gt = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  // crop origins read once per workgroup (from the device placement table
  // when there is one): a cell's crop loop would otherwise wait on each
  __shared__ int s_ox[VRS_MAX_CROPS], s_oy[VRS_MAX_CROPS];
  if (threadIdx.x < crops.n) {
    if (gaze) {
      const int4 pl = place_crop(crops, threadIdx.x, gaze[threadIdx.x]);
      s_ox[threadIdx.x] = pl.x;
      s_oy[threadIdx.x] = pl.y;
      if (blockIdx.x == 0) place_out[threadIdx.x] = pl;
    } else {
      s_ox[threadIdx.x] = crop_x0(crops, threadIdx.x);
      s_oy[threadIdx.x] = crop_y0(crops, threadIdx.x);
    }
  }
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  // the counters in 16-byte stores (the workspace's sub-buffers are 256-byte
  // aligned), the tail word by word
  uint4* p4 = reinterpret_cast<uint4*>(pcnt);
  for (int64_t q = gt; q < pix_total / 4; q += stride) p4[q] = make_uint4(0u, 0u, 0u, 0u);
  for (int64_t i = (pix_total & ~int64_t(3)) + gt; i < pix_total; i += stride) pcnt[i] = 0u;
  for (int64_t i = gt; i < scan_words; i += stride) scan_tmp[i] = 0u;
  if (gt == 0) {
    ctr[0] = 0ull;
    *reinterpret_cast<uint32_t*>(ctr + 1) = 0u;
  }
  for (int64_t i = gt; i < cells; i += stride)
    pt_cropgrid_cell(crops, levels, gx, gy, i, s_ox, s_oy, grid);
  if (hide)
    for (int64_t i = gt; i < pixels; i += stride)
      hide[i] = pt_hide_limit(tfinal[i], depth[i], a.cov_min, a.slack);
}

// Candidate crops of one point in view v: the crop-lookup grid cell of a
// reciprocal-based pixel estimate (within 1e-2 px of the exact one, well
// inside the grid's slack).  A non-positive or non-finite estimate gives
// every crop.
__device__ inline uint32_t pt_candidates(const KView& cv, int v, int n_crops,
                                         const uint32_t* __restrict__ grid, int gx, int gy,
                                         float x, float y, float z) {
  uint32_t cand = n_crops >= 32 ? 0xffffffffu : ((1u << n_crops) - 1u);
  const float tx = cv.R[0] * x + cv.R[1] * y + cv.R[2] * z + cv.t[0];
  const float ty = cv.R[3] * x + cv.R[4] * y + cv.R[5] * z + cv.t[1];
  const float tz = cv.R[6] * x + cv.R[7] * y + cv.R[8] * z + cv.t[2];
  if (tz > 0.0f) {
    const float rz = __builtin_amdgcn_rcpf(tz);
    const float ex = (cv.fx * (tx * rz) + cv.cx) * (1.0f / kGridCell);
    const float ey = (cv.fy * (ty * rz) + cv.cy) * (1.0f / kGridCell);
    if (isfinite(ex) && isfinite(ey)) {
      const float fx = fminf(fmaxf(floorf(ex), 0.0f), (float)(gx - 1));
      const float fy = fminf(fmaxf(floorf(ey), 0.0f), (float)(gy - 1));
      cand = grid[((int64_t)v * gy + (int)fy) * gx + (int)fx];
    }
  }
  return cand;
}

// Footprint targets of a projected point over the candidate crops of view v
// and the point's one or two pyramid layers; cview, csize, ox, oy: the
// crops' views, sizes and origins (a workgroup's copy in LDS: a lane's crop
// index is its own, so a read from the kernel arguments would be a vector
// load and a wait per crop).
__device__ inline uint32_t pt_targets_over(const PtGeom& g, int v, uint32_t cand, int levels,
                                           const int* cview, const int* csize, const int* ox,
                                           const int* oy) {
  uint32_t cnt = 0;
  const float M = (float)(1 << levels);
  while (cand) {
    const int k = __builtin_ctz(cand);
    cand &= cand - 1;
    if (cview[k] != v) continue;
    const int cx0 = ox[k], cy0 = oy[k], size = csize[k];
    const float ax = g.px - (float)cx0, ay = g.py - (float)cy0, lim = (float)size + M;
    if (!(ax >= -M && ax < lim && ay >= -M && ay < lim)) continue;
    for (int li = 0; li < (g.two ? 2 : 1); ++li) {
      const int l = g.l0 + li, Sl = size >> l;
      float xl, yl;
      int ix, iy;
      if (pt_layer32(g, cx0, cy0, l, Sl, xl, yl, ix, iy)) cnt += pt_targets(ix, iy, Sl);
    }
  }
  return cnt;
}

// Workgroup b holds four rounds of kSelBlock points.  Per round and view each
// lane's fragment count (and screen bucket) goes to LDS and each wave ballots
// its survivors; a scan over the (view, round, wave) slots places them and
// their fragments within the workgroup, and one 64-bit atomic on the (survivor,
// fragment) counts gives the workgroup's output bases, so no separate scan of
// fragment counts is needed.  The compacted order is therefore arbitrary
// across workgroups, which nothing downstream sees: each fragment's final place
// is its rank by (depth key, point index) in its pixel.  One atomic per workgroup: a single counter address serialises
// its atomics, so workgroups are kept large.
constexpr int kSelRounds = 4;

// ORD: a survivor also carries its screen bucket.
template <int kSelBlock, bool ORD>
__global__ __launch_bounds__(kSelBlock) void k_pt_select(
    const float* __restrict__ pos, const float* __restrict__ radius, int64_t np, KViews views,
    KCrops crops, PtArgs a, const float* __restrict__ depth, const float* __restrict__ tfinal,
    const float* __restrict__ hide,
    const uint32_t* __restrict__ grid, int gx, int gy, uint4* __restrict__ surv,
    uint64_t* __restrict__ ctr, uint32_t* __restrict__ chunk_first, int64_t max_frags,
    int32_t* status) {
  constexpr int NW = kSelBlock / 64, kSelPart = kSelBlock * kSelRounds;
  constexpr int NSLOT = kSelRounds * VRS_MAX_VIEWS * NW;   // (view, round, wave), view-major
  static_assert(NSLOT <= kSelBlock, "one slot per thread in the slot scan");
  __shared__ uint32_t s_base, s_fbase;
  __shared__ uint64_t s_mask[NSLOT];
  __shared__ uint32_t s_pre[NSLOT], s_fsum[NSLOT], s_fpre[NSLOT];
  __shared__ uint32_t s_wsum[NW], s_wfsum[NW];
  // crop origins (from the device placement table when there is one),
  // views and sizes read once: a survivor's crop loop would otherwise wait
  // on loads per crop
  __shared__ int s_ox[VRS_MAX_CROPS], s_oy[VRS_MAX_CROPS], s_cv[VRS_MAX_CROPS], s_cs[VRS_MAX_CROPS];
  __shared__ int s_ob[VRS_MAX_CROPS];   // first screen bucket of the crop
  extern __shared__ __align__(16) char s_dyn[];
  const int nv = views.n;
  uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_dyn);   // [round][view][tid]
  // and the depths, where there is room for them
  constexpr bool DEPTHS = kSelBlock <= 256;
  float* s_zd = reinterpret_cast<float*>(s_dyn) + kSelRounds * nv * kSelBlock;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int e = tid; e < NSLOT; e += kSelBlock) {
    s_mask[e] = 0;
    s_fsum[e] = 0;
  }
  if (tid < crops.n) {
    s_ox[tid] = crop_x0(crops, tid);
    s_oy[tid] = crop_y0(crops, tid);
    s_cv[tid] = crops.c[tid].view;
    s_cs[tid] = crops.c[tid].size;
    if (ORD) {
      int ob = 0;
      for (int k = 0; k < tid; ++k) {
        const int t = (crops.c[k].size + a.ord_side - 1) / a.ord_side;
        ob += t * t;
      }
      s_ob[tid] = ob;
    }
  }
  __syncthreads();
  const int64_t part = blockIdx.x;
  // ---- counts of every (round, view, point), in stages so that each
  // stage's loads (positions; grid cells; T' and depth under the points) are
  // in flight together: a point's fragment count is its footprint targets
  // over the candidate crops, zero if the depth cull hides it.  The cull
  // runs before the targets (the result is the same: a hidden point counts
  // zero either way) because it removes most points that reach a crop.
  float px[kSelRounds], py[kSelRounds], pz[kSelRounds], pr[kSelRounds];
  bool pin[kSelRounds];
#pragma unroll
  for (int j = 0; j < kSelRounds; ++j) {
    const int64_t i = part * kSelPart + (int64_t)j * kSelBlock + tid;
    pin[j] = i < np;
    px[j] = py[j] = pz[j] = pr[j] = 0.0f;
    if (pin[j]) { px[j] = pos[i]; py[j] = pos[np + i]; pz[j] = pos[2 * np + i]; pr[j] = radius[i]; }
  }
  // one source or the other without a branch between the loads
  const float* __restrict__ under_t = hide ? hide : tfinal;
  const float* __restrict__ under_d = hide ? hide : depth;
  for (int v = 0; v < nv; ++v) {
    const KView& cv = views.v[v];
    const bool vm = (a.view_mask >> v) & 1u;
    const int64_t plane = (int64_t)cv.W * cv.H;
    uint32_t cand[kSelRounds];
#pragma unroll
    for (int j = 0; j < kSelRounds; ++j)
      cand[j] = pin[j] && vm ? pt_candidates(cv, v, crops.n, grid, gx, gy, px[j], py[j], pz[j]) : 0u;
    bool ok[kSelRounds], cull[kSelRounds];
    float tz[kSelRounds], tf[kSelRounds], dp[kSelRounds];
#pragma unroll
    for (int j = 0; j < kSelRounds; ++j) {
      ok[j] = cull[j] = false;
      tz[j] = tf[j] = dp[j] = 0.0f;
      if (cand[j]) {
        PtGeom g;
        ok[j] = pt_geom32(cv, px[j], py[j], pz[j], pr[j], a.levels, g);
        tz[j] = g.t[2];
        int64_t pi;
        cull[j] = ok[j] && tfinal && pt_cull_pixel(cv, g, pi);
        if (cull[j]) {   // T' and depth, or the pixel's hiding depth
          tf[j] = under_t[v * plane + pi];
          dp[j] = under_d[v * plane + pi];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < kSelRounds; ++j) {
      uint32_t cnt = 0, bucket = 0;
      if (ok[j] && !(cull[j] && (hide ? tz[j] > tf[j]
                                   : pt_hidden(tz[j], tf[j], dp[j], a.cov_min, a.slack)))) {
        PtGeom g;   // recomputed for the few points the cull keeps
        pt_geom32(cv, px[j], py[j], pz[j], pr[j], a.levels, g);
        cnt = pt_targets_over(g, v, cand[j], a.levels, s_cv, s_cs, s_ox, s_oy);
        if (ORD && cnt) {   // its place on the first of its view's candidate crops
          uint32_t cm = cand[j];
          while (s_cv[__builtin_ctz(cm)] != v) cm &= cm - 1;
          const int k = __builtin_ctz(cm);
          const int t = (s_cs[k] + a.ord_side - 1) / a.ord_side;
          const float inv = 1.0f / (float)a.ord_side, top = (float)(t - 1);
          const int bx = (int)fminf(fmaxf((g.px - (float)s_ox[k]) * inv, 0.0f), top);
          const int by = (int)fminf(fmaxf((g.py - (float)s_oy[k]) * inv, 0.0f), top);
          bucket = (uint32_t)(s_ob[k] + by * t + bx);
        }
      }
      s_cnt[(j * nv + v) * kSelBlock + tid] = ORD ? cnt | bucket << 16 : cnt;
      if (DEPTHS) s_zd[(j * nv + v) * kSelBlock + tid] = tz[j];
      const uint64_t m = __ballot(cnt != 0);
      if (m) {   // the slot's fragment total
        uint32_t fs = cnt;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) fs += __shfl_xor(fs, o, 64);
        if (lane == 0) {
          s_mask[(v * kSelRounds + j) * NW + wave] = m;
          s_fsum[(v * kSelRounds + j) * NW + wave] = fs;
        }
      }
    }
  }
  __syncthreads();
  // ---- exclusive scans of the slot survivor and fragment counts in output
  // order, then the workgroup's bases
  {
    const uint32_t c = tid < NSLOT ? (uint32_t)__popcll(s_mask[tid]) : 0u;
    const uint32_t f = tid < NSLOT ? s_fsum[tid] : 0u;
    uint32_t ic = c, jf = f;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(ic, o, 64), z = __shfl_up(jf, o, 64);
      if (lane >= o) {
        ic += y;
        jf += z;
      }
    }
    if (lane == 63) {
      s_wsum[wave] = ic;
      s_wfsum[wave] = jf;
    }
    __syncthreads();
    uint32_t woff = 0, wfoff = 0, total = 0, ftotal = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      if (w < wave) {
        woff += s_wsum[w];
        wfoff += s_wfsum[w];
      }
      total += s_wsum[w];
      ftotal += s_wfsum[w];
    }
    if (tid < NSLOT) {
      s_pre[tid] = woff + ic - c;
      s_fpre[tid] = wfoff + jf - f;
    }
    if (tid == 0) {
      const uint64_t old = total ? atomicAdd(ctr, ((uint64_t)ftotal << 32) | total) : 0ull;
      s_base = (uint32_t)old;
      s_fbase = (uint32_t)(old >> 32);
      // the fragment count wraps only far beyond any capacity
      if ((old >> 32) + ftotal > 0xffffffffull) set_status(status, VRS_ECAPACITY);
    }
  }
  __syncthreads();
  // ---- survivors to their positions, with their fragment offsets
  const uint32_t base = s_base, fbase = s_fbase;
  for (int j = 0; j < kSelRounds; ++j) {
    const int64_t i = part * kSelPart + (int64_t)j * kSelBlock + tid;
    for (int v = 0; v < nv; ++v) {
      const int slot = (v * kSelRounds + j) * NW + wave;
      const uint64_t m = s_mask[slot];
      if (!m) continue;   // uniform
      const uint32_t cw = s_cnt[(j * nv + v) * kSelBlock + tid], cnt = ORD ? cw & 0xffffu : cw;
      uint32_t fi = cnt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(fi, o, 64);
        if (lane >= o) fi += y;
      }
      if (!cnt) continue;
      const uint32_t below = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
      const uint32_t p = base + s_pre[slot] + below;
      const uint32_t fo = fbase + s_fpre[slot] + fi - cnt;
      float z;
      if constexpr (DEPTHS) {
        z = s_zd[(j * nv + v) * kSelBlock + tid];
      } else {
        PtGeom g;
        pt_geom32(views.v[v], pos[i], pos[np + i], pos[2 * np + i], radius[i], a.levels, g);
        z = g.t[2];
      }
      surv[p] = make_uint4((uint32_t)(v * np + i), __float_as_uint(z), fo, cw);
      // the emission chunks whose first fragment is one of this survivor's
      for (uint64_t c = ((uint64_t)fo + kEmitFrags - 1) / kEmitFrags;
           c * kEmitFrags < (uint64_t)fo + cnt && c * kEmitFrags < (uint64_t)max_frags; ++c)
        chunk_first[c] = p;
    }
  }
}

// -------------------------------------------------- dense lists: screen order
// Points come in any order, and the emission then finds a chunk's fragments on
// as many pixels: 28M fragments cost 28M device-scope atomics on the pixel
// counters (about 20 per ns), and their records scatter over the segments.
// Where the counted fragments make dense lists the survivors are first put in
// the order of screen buckets (a few hundred pixels each): counts per
// workgroup and bucket, their prefix, then every survivor with its position to
// its place, its fragments numbered anew by the same packed cursor (survivors
// low, fragments high; the order within a bucket is free, as the emission
// order is).  A chunk's fragments then share some 200 pixels, its atomics and
// its records' lines.  5M points, one 512 crop: 0.17 ms for the order, emission
// 1.8 ms -> 0.48, scatter 0.86 -> 0.53, whole splat 3.38 -> 2.32; 0.9M points
// (15 fragments per layer pixel) 0.68 -> 0.52, four views of 2M points with
// their adjoint 13.2 -> 11.3.
__device__ inline bool pt_dense(int64_t total, int64_t max_frags, int64_t pix_total) {
  return total > kRsDense * pix_total && total <= max_frags;
}

__global__ __launch_bounds__(kOrdBlock) void k_pt_ord_count(
    const uint4* __restrict__ surv, const uint32_t* __restrict__ live_p,
    const uint32_t* __restrict__ total_p, int64_t max_frags, int64_t pix_total,
    uint64_t* __restrict__ hist) {
  __shared__ unsigned long long s_h[kOrdBuckets];
  if (!pt_dense(*total_p, max_frags, pix_total)) return;
  const int64_t live = *live_p;
  const int64_t lo = live * blockIdx.x / gridDim.x, hi = live * (blockIdx.x + 1) / gridDim.x;
  for (int d = threadIdx.x; d < kOrdBuckets; d += kOrdBlock) s_h[d] = 0;
  __syncthreads();
  for (int64_t j = lo + threadIdx.x; j < hi; j += kOrdBlock) {
    const uint32_t w = surv[j].w;
    atomicAdd(&s_h[w >> 16], (unsigned long long)(w & 0xffffu) << 32 | 1ull);
  }
  __syncthreads();
  uint64_t* out = hist + (int64_t)blockIdx.x * kOrdBuckets;
  for (int d = threadIdx.x; d < kOrdBuckets; d += kOrdBlock) out[d] = s_h[d];
}

// hist [parts + 1][buckets]: each bucket's counts to their prefix over the
// parts, its total to the last row.  A wave reads 64 buckets of a part.
__global__ __launch_bounds__(1024) void k_pt_ord_scan(const uint32_t* __restrict__ total_p,
                                                      int64_t max_frags, int64_t pix_total,
                                                      uint64_t* __restrict__ hist, int parts) {
  __shared__ uint64_t s_sum[16][64];
  if (!pt_dense(*total_p, max_frags, pix_total)) return;
  const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
  uint64_t* h = hist + blockIdx.x * 64 + lane;
  const int lo = parts * g / 16, hi = parts * (g + 1) / 16;
  uint64_t sum = 0;
#pragma unroll 8
  for (int p = lo; p < hi; ++p) sum += h[(int64_t)p * kOrdBuckets];
  s_sum[g][lane] = sum;
  __syncthreads();
  uint64_t run = 0, tot = 0;
  for (int q = 0; q < 16; ++q) {
    run += q < g ? s_sum[q][lane] : 0;
    tot += s_sum[q][lane];
  }
#pragma unroll 8
  for (int p = lo; p < hi; ++p) {
    const uint64_t c = h[(int64_t)p * kOrdBuckets];
    h[(int64_t)p * kOrdBuckets] = run;
    run += c;
  }
  if (g == 0) h[(int64_t)parts * kOrdBuckets] = tot;
}

__global__ __launch_bounds__(kOrdBlock) void k_pt_ord_move(
    const float* __restrict__ pos, const float* __restrict__ radius, int64_t np,
    const uint4* __restrict__ surv, const uint32_t* __restrict__ live_p,
    const uint32_t* __restrict__ total_p, int64_t max_frags, int64_t pix_total,
    const uint64_t* __restrict__ hist, uint4* __restrict__ surv2, float4* __restrict__ at2,
    uint32_t* __restrict__ chunk_first) {
  constexpr int PER = kOrdBuckets / kOrdBlock, NW = kOrdBlock / 64;
  __shared__ unsigned long long s_cur[kOrdBuckets], s_w[NW];
  if (!pt_dense(*total_p, max_frags, pix_total)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  {
    const uint64_t* tot = hist + (int64_t)gridDim.x * kOrdBuckets;
    const uint64_t* mine = hist + (int64_t)blockIdx.x * kOrdBuckets;
    unsigned long long c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      c[q] = sum;
      sum += tot[tid * PER + q];
    }
    unsigned long long incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    unsigned long long base = incl - sum;
    for (int w = 0; w < wave; ++w) base += s_w[w];
#pragma unroll
    for (int q = 0; q < PER; ++q) s_cur[tid * PER + q] = base + c[q] + mine[tid * PER + q];
  }
  __syncthreads();
  const int64_t live = *live_p;
  const int64_t lo = live * blockIdx.x / gridDim.x, hi = live * (blockIdx.x + 1) / gridDim.x;
  for (int64_t j = lo + tid; j < hi; j += kOrdBlock) {
    const uint4 sv = surv[j];
    const int64_t i = sv.x % (uint32_t)np;
    const float4 at = make_float4(pos[i], pos[np + i], pos[2 * np + i], radius[i]);
    const uint32_t cnt = sv.w & 0xffffu;
    const uint64_t old = atomicAdd(&s_cur[sv.w >> 16], (unsigned long long)cnt << 32 | 1ull);
    const uint32_t p = (uint32_t)old;
    const uint64_t fo = old >> 32;
    surv2[p] = make_uint4(sv.x, sv.y, (uint32_t)fo, sv.w);
    at2[p] = at;
    for (uint64_t c = (fo + kEmitFrags - 1) / kEmitFrags; c * kEmitFrags < fo + cnt; ++c)
      chunk_first[c] = p;
  }
}

// ------------------------------------------------------------------ emit
// Per-workgroup pixel table in LDS: open addressing with a short linear
// probe.  Device-scope atomics on one address serialise, so fragment counts
// (and segment places) are gathered per workgroup first and the table's
// entries go out as one atomic each; a fragment whose probe finds no place
// falls back to its own atomic.
constexpr int kPixProbe = 8;
constexpr uint32_t kPixEmpty = 0xffffffffu;
template <int N>   // places, a power of two
struct PixHash {
  static constexpr int kBits = N == 4096 ? 12 : (N == 2048 ? 11 : (N == 1024 ? 10 : 9));
  static_assert((1 << kBits) == N, "PixHash size");
  uint32_t key[N], cnt[N];
  __device__ void clear() {
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
      key[i] = kPixEmpty;
      cnt[i] = 0u;
    }
  }
  // one more fragment of pixel px: its table place (or -1) and its rank
  // among the table's fragments of px
  __device__ int add(uint32_t px, uint32_t& rank) {
    uint32_t s = (px * 2654435761u) >> (32 - kBits);
    for (int q = 0; q < kPixProbe; ++q) {
      const uint32_t k = atomicCAS(&key[s], kPixEmpty, px);
      if (k == kPixEmpty || k == px) {
        rank = atomicAdd(&cnt[s], 1u);
        return (int)s;
      }
      s = (s + 1) & (N - 1);
    }
    return -1;
  }
};

// One workgroup per chunk of kEmitFrags consecutive fragments (the chunks'
// first survivors are recorded by k_pt_select), one thread per survivor of
// the chunk: its fragments that fall in the chunk, each with its layer
// pixel, weight | point index, depth key and place in the pixel's segment.
// Places come from the pixel counters' old values: the workgroup gathers
// its fragments per pixel in the LDS table (at most half full: a chunk
// holds kEmitFrags fragments), each table entry adds its count with one
// atomic whose old value is the entry's first place, and a fragment's
// place is that plus its rank in the entry.  The chunk is staged in LDS
// and goes out as coalesced stores once the places are known.  Balanced by
// construction: every workgroup emits one chunk, however the fragments
// spread over survivors.
constexpr int kEmitPlaces = 2 * kEmitFrags, kEmitBlock = 256;
constexpr uint32_t kSlotRef = 0x80000000u;   // tag | table place << kRankBits | rank
constexpr int kRankBits = 19;
static_assert(kEmitPlaces <= (1 << (31 - kRankBits)) && kEmitFrags < (1 << kRankBits),
              "table place and rank fit the tag");
static_assert(kEmitPlaces % kEmitBlock == 0 && kEmitFrags % kEmitBlock == 0,
              "table entries and staged fragments per thread");
__global__ __launch_bounds__(kEmitBlock) void k_pt_emit(
    const float* __restrict__ pos, const float* __restrict__ radius, int64_t np, KViews views,
    KCrops crops, PtArgs a, const uint4* __restrict__ surv1, const uint4* __restrict__ surv2,
    const float4* __restrict__ at2, int64_t pix_total, const uint32_t* __restrict__ live_p,
    const uint32_t* __restrict__ chunk_first, const uint32_t* __restrict__ total_p,
    int64_t max_frags, uint32_t* __restrict__ fkey, uint64_t* __restrict__ fval,
    uint32_t* __restrict__ fdep, uint32_t* __restrict__ fslot, uint32_t* __restrict__ pcnt,
    const uint32_t* __restrict__ grid, int gx, int gy, int32_t* status) {
  __shared__ PixHash<kEmitPlaces> h;
  // staged fragments: layer pixel, weight bits, place (or tag), owning
  // survivor slot; per survivor slot its point index and depth key
  __shared__ uint32_t s_spx[kEmitFrags], s_sw[kEmitFrags], s_stag[kEmitFrags];
  __shared__ uint16_t s_sown[kEmitFrags];
  __shared__ uint32_t s_pi[kEmitFrags + 1], s_dz[kEmitFrags + 1];
  __shared__ int s_cx0[VRS_MAX_CROPS], s_cy0[VRS_MAX_CROPS], s_cs[VRS_MAX_CROPS],
      s_pb[VRS_MAX_CROPS];
  // crop origins (from the device placement table when there is one), sizes
  // and pyramid bases read once: the crop loop below would otherwise wait on
  // loads per crop
  if (threadIdx.x < crops.n) {
    s_cx0[threadIdx.x] = crop_x0(crops, threadIdx.x);
    s_cy0[threadIdx.x] = crop_y0(crops, threadIdx.x);
    s_cs[threadIdx.x] = crops.c[threadIdx.x].size;
    s_pb[threadIdx.x] = crops.c[threadIdx.x].pix_base;
  }
  __syncthreads();
  const int64_t live = *live_p;
  const int64_t total = *total_p;
  if (blockIdx.x == 0 && threadIdx.x == 0 && total > max_frags) set_status(status, VRS_ECAPACITY);
  if (total > max_frags) return;   // uniform
  const bool ord = surv2 && pt_dense(total, max_frags, pix_total);
  const uint4* __restrict__ surv = ord ? surv2 : surv1;
  const int64_t nchunks = (total + kEmitFrags - 1) / kEmitFrags;
  for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
    const int64_t f0 = ch * kEmitFrags, f1 = std::min<int64_t>(f0 + kEmitFrags, total);
    const int64_t s0 = chunk_first[ch];
    h.clear();
    __syncthreads();
    // survivors s0, s0 + 1, ... while their fragments start before f1 (at
    // most kEmitFrags + 1 of them: each has at least one fragment)
    for (int64_t j = s0 + threadIdx.x; j < live; j += kEmitBlock) {
      const uint4 sv = surv[j];
      const int64_t lo = sv.z;
      if (lo >= f1) break;   // offsets ascend with j
      const int slot = (int)(j - s0);
      const uint32_t e = sv.x;
      const int v = (int)(e / np);
      const int64_t i = e - (int64_t)v * np;
      s_pi[slot] = (uint32_t)i;
      s_dz[slot] = sv.y;
      const KView& cv = views.v[v];
      PtGeom g;
      // the depth cull already passed in k_pt_select; the same single-precision
      // sequence gives identical geometry here
      const float4 p4 = ord ? at2[j]
                            : make_float4(pos[i], pos[np + i], pos[2 * np + i], radius[i]);
      const float x = p4.x, y = p4.y, z = p4.z;
      if (!pt_geom32(cv, x, y, z, p4.w, a.levels, g)) continue;
      float f = 0.0f;
      if (g.two) f = log2f(g.s) - (float)g.l0;
      FF ux, uy;   // the weights' position, compensated
      pt_plane_ff(cv, x, y, z, ux, uy);
      int64_t o = lo;
      // the crops the selection counted this point's fragments over (its
      // crop-grid candidates: the other crops give it none), in crop order
      for (uint32_t cand = pt_candidates(cv, v, crops.n, grid, gx, gy, x, y, z); cand && o < f1;
           cand &= cand - 1) {
        const int k = __builtin_ctz(cand);
        const int cx0 = s_cx0[k], cy0 = s_cy0[k], size = s_cs[k];
        int lb = s_pb[k];
        int l = 0;
        for (; l < g.l0; ++l) lb += (size >> l) * (size >> l);
        for (int li = 0; li < (g.two ? 2 : 1); ++li, ++l) {
          const int Sl = size >> l;
          const float wl = g.two ? (li == 0 ? 1.0f - f : f) : 1.0f;
          float xl, yl;
          int ix, iy;
          if (pt_layer32(g, cx0, cy0, l, Sl, xl, yl, ix, iy)) {
            const float bx = pt_frac_ff(cv.fx, ux, cv.cx, cx0, l, ix);
            const float by = pt_frac_ff(cv.fy, uy, cv.cy, cy0, l, iy);
            for (int dy = 0; dy < 2; ++dy)
              for (int dx = 0; dx < 2; ++dx) {
                const int xx = ix + dx, yy = iy + dy;
                if (xx < 0 || xx >= Sl || yy < 0 || yy >= Sl) continue;
                if (o >= f0 && o < f1) {
                  const int local = (int)(o - f0);
                  const uint32_t px = (uint32_t)(lb + yy * Sl + xx);
                  // a point reaches a pixel once, so a pixel's rank in the
                  // table is below the chunk's fragment count
                  uint32_t r;
                  const int hs = h.add(px, r);
                  s_spx[local] = px;
                  s_sw[local] = __float_as_uint(wl * (dx ? bx : 1.0f - bx) * (dy ? by : 1.0f - by));
                  s_stag[local] = hs >= 0 ? (kSlotRef | (uint32_t)hs << kRankBits | r)
                                          : atomicAdd(&pcnt[px], 1u);
                  s_sown[local] = (uint16_t)slot;
                }
                ++o;
              }
          }
          lb += Sl * Sl;
        }
      }
    }
    __syncthreads();
    {
      // every entry's atomic issued before any result is awaited (device-
      // scope atomics take about a microsecond each); the old values
      // replace the counts
      constexpr int kPer = kEmitPlaces / kEmitBlock;
      uint32_t first[kPer];
#pragma unroll
      for (int r = 0; r < kPer; ++r) {
        const int q = threadIdx.x + r * kEmitBlock;
        const uint32_t key = h.key[q];
        first[r] = key != kPixEmpty ? atomicAdd(&pcnt[key], h.cnt[q]) : 0u;
      }
#pragma unroll
      for (int r = 0; r < kPer; ++r) h.cnt[threadIdx.x + r * kEmitBlock] = first[r];
    }
    __syncthreads();
    // the chunk out, coalesced, with its places
    for (int q = threadIdx.x; q < (int)(f1 - f0); q += kEmitBlock) {
      const uint32_t t = s_stag[q];
      const int own = s_sown[q];
      fkey[f0 + q] = s_spx[q];
      fval[f0 + q] = ((uint64_t)s_sw[q] << 32) | (uint64_t)s_pi[own];
      fdep[f0 + q] = s_dz[own];
      fslot[f0 + q] = (t & kSlotRef)
                          ? h.cnt[(t & ~kSlotRef) >> kRankBits] + (t & ((1u << kRankBits) - 1u))
                          : t;
    }
    __syncthreads();   // the stage is reused by the next chunk
  }
}

// Each fragment's record (point index, depth key, weight, pixel) to its
// segment place (checked against the segment, so an unresolved place can
// never write outside it).  The place replaces the fragment's slot and, once
// the fragment is ranked, its final place goes to the depth keys' array (free
// by then), by place: the adjoint's way from a point's fragments to the sorted
// lists.
__global__ __launch_bounds__(256) void k_pt_scatter(const uint32_t* __restrict__ fkey,
                                                    const uint64_t* __restrict__ fval,
                                                    const uint32_t* __restrict__ fdep,
                                                    uint32_t* __restrict__ fslot,
                                                    const uint32_t* __restrict__ poff,
                                                    const uint32_t* __restrict__ total_p,
                                                    int64_t max_frags, uint4* __restrict__ seg) {
  const int64_t total = *total_p;
  if (total > max_frags) return;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t px = fkey[i];
    const uint64_t v = fval[i];
    const uint32_t at = poff[px] + fslot[i];
    if (at < poff[px + 1]) seg[at] = make_uint4((uint32_t)v, fdep[i], (uint32_t)(v >> 32), px);
    fslot[i] = at;
  }
}

// One thread per segment place: the record's final place is its segment's
// offset plus the number of the segment's records before it in (depth key,
// point id) order, the id being the point's index in the caller's numbering
// (ids[i] for stored point i when a numbering is given, else i; a point
// reaches a layer pixel at most once, so the pairs are distinct).  Equal
// depth keys are rare, so the numbering is looked up only for them.
// Consecutive places share segments, so the lanes of a segment read the
// same records; places go in reverse, so that the long segments of each
// crop's coarse layers start early.
// DENSE: the capacity allows dense lists; then only what k_pt_resolve left.
template <bool DENSE>
__global__ __launch_bounds__(256) void k_pt_rank(const uint4* __restrict__ seg,
                                                 uint32_t* __restrict__ fin,
                                                 const uint32_t* __restrict__ poff,
                                                 const uint32_t* __restrict__ total_p,
                                                 int64_t max_frags, int64_t pix_total,
                                                 const uint32_t* __restrict__ left_p,
                                                 const uint32_t* __restrict__ pcnt,
                                                 const uint32_t* __restrict__ ids,
                                                 uint32_t* __restrict__ okey,
                                                 uint64_t* __restrict__ oval) {
  const uint32_t left = DENSE ? *left_p : 0u;   // (read with the count: most workgroups only leave)
  const int64_t total = *total_p;
  const bool dense = DENSE && total > kRsDense * pix_total;
  if (total > max_frags || (dense && left == 0)) return;
  const uint64_t* key = reinterpret_cast<const uint64_t*>(seg);   // depth key << 32 | index
  for (int64_t sr = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; sr < total;
       sr += (int64_t)gridDim.x * blockDim.x) {
    const uint4 rec = seg[total - 1 - sr];
    if (rec.w >= pix_total) continue;   // every place is filled; never taken
    if (dense && pcnt[rec.w] != kRsLeft) continue;
    const uint64_t own = ((uint64_t)rec.y << 32) | rec.x;
    const uint32_t start = poff[rec.w], n = poff[rec.w + 1] - start;
    uint32_t rank = 0;
    if (ids) {
      // keys in groups of kRankBatch, every group's loads in flight before
      // the comparisons; equal depth keys (rare) are settled after the
      // group by the original indices, so no index load sits between the
      // key loads and their use
      const uint32_t own_id = ids[rec.x];
      constexpr int kRankBatch = 8;
      for (uint32_t j0 = 0; j0 < n; j0 += kRankBatch) {
        uint64_t kk[kRankBatch];
#pragma unroll
        for (int q = 0; q < kRankBatch; ++q)
          kk[q] = j0 + q < n ? key[2 * (int64_t)(start + j0 + q)] : 0ull;
        uint32_t ties = 0;
#pragma unroll
        for (int q = 0; q < kRankBatch; ++q) {
          if (j0 + q >= n) continue;
          const uint32_t kd = (uint32_t)(kk[q] >> 32);
          rank += kd < rec.y ? 1u : 0u;
          if (kd == rec.y && kk[q] != own) ties |= 1u << q;
        }
        while (ties) {
          const int q = __builtin_ctz(ties);
          ties &= ties - 1;
          rank += ids[(uint32_t)kk[q]] < own_id ? 1u : 0u;
        }
      }
    } else {
#pragma unroll 8
      for (uint32_t j = 0; j < n; ++j) rank += key[2 * (int64_t)(start + j)] < own ? 1u : 0u;
    }
    okey[start + rank] = rec.w;
    oval[start + rank] = ((uint64_t)rec.z << 32) | rec.x;
    fin[total - 1 - sr] = start + rank;
  }
}

// ----------------------------------------------------------------- blend
// One thread per layer pixel: its list front to back (zero where empty).
// Pixels go in reverse pyramid order: each crop's coarse layers (the long
// lists) come after its finest layer in the pyramid, so in reverse the
// long lists start early and the finest layers' short lists fill the end.
template <bool DENSE>   // as k_pt_rank
__global__ __launch_bounds__(256) void k_pt_blend(const uint64_t* __restrict__ fval,
                                                  const uint32_t* __restrict__ poff,
                                                  const uint32_t* __restrict__ total_p,
                                                  int64_t max_frags,
                                                  const uint32_t* __restrict__ left_p,
                                                  const uint32_t* __restrict__ pcnt,
                                                  const uint16_t* __restrict__ feat,
                                                  const float* __restrict__ opacity, int64_t np,
                                                  int64_t pix_total, float4* __restrict__ pyr) {
  // dense lists are k_pt_resolve's (launched wherever the capacity allows
  // them) but for those it left
  const uint32_t left = DENSE ? *left_p : 0u;
  const bool dense = DENSE && min((int64_t)*total_p, max_frags) > kRsDense * pix_total;
  if (dense && left == 0) return;
  const bool over = (int64_t)*total_p > max_frags;
  for (int64_t kr = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; kr < pix_total;
       kr += (int64_t)gridDim.x * blockDim.x) {
    const int64_t k = pix_total - 1 - kr;
    if (dense && pcnt[k] != kRsLeft) continue;
    float T = 1.0f;
    float4 F = make_float4(0, 0, 0, 0);
    const uint32_t start = over ? 0u : poff[k], n = over ? 0u : poff[k + 1] - start;
    // fragments in groups of kPtBatch, every group's loads in flight before
    // its (sequential) compositing: long lists are otherwise one load
    // latency per fragment
    constexpr int kPtBatch = 8;
    for (uint32_t j0 = 0; j0 < n; j0 += kPtBatch) {
      uint64_t vv[kPtBatch];
      float op[kPtBatch];
      uint2 hb[kPtBatch];
#pragma unroll
      for (int q = 0; q < kPtBatch; ++q)
        vv[q] = j0 + q < n ? fval[start + j0 + q] : ~0ull;
#pragma unroll
      for (int q = 0; q < kPtBatch; ++q) {
        const uint32_t id = (uint32_t)vv[q];
        const bool ok = id < (uint64_t)np;
        op[q] = ok && opacity ? opacity[id] : 1.0f;
        hb[q] = ok ? *reinterpret_cast<const uint2*>(feat + (int64_t)id * 4) : make_uint2(0, 0);
      }
#pragma unroll
      for (int q = 0; q < kPtBatch; ++q) {
        if (j0 + q >= n || (uint32_t)vv[q] >= (uint64_t)np) continue;
        const float w = __uint_as_float((uint32_t)(vv[q] >> 32));
        const float al = opacity ? w * op[q] : w;
        const float aT = al * T;
        F.x += h2f((uint16_t)(hb[q].x & 0xffffu)) * aT;
        F.y += h2f((uint16_t)(hb[q].x >> 16)) * aT;
        F.z += h2f((uint16_t)(hb[q].y & 0xffffu)) * aT;
        F.w += h2f((uint16_t)(hb[q].y >> 16)) * aT;
        T = T * (1.0f - al);
      }
    }
    pyr[k] = F;
  }
}

// ------------------------------------------------- dense fragment lists
// Ranking and blend in one kernel for splats whose pixels hold many
// fragments (culling off).  k_pt_rank compares every fragment with its whole
// segment and k_pt_blend walks a segment in one thread, so both grow with
// the list length: 5M points under one 512 crop (27M fragments, lists to
// 2000) took 7.4 + 0.95 ms.  Here a wave takes each pixel, and the workgroup
// together those with more than 256 fragments: they are ranked through 1024
// depth buckets (count, scan, place, then a comparison within the bucket
// alone; up to 64 a lane's one fragment against all, up to 256 four; a bucket
// beyond the LDS leaves its pixel to k_pt_rank and k_pt_blend), then each wave
// composites its pixel: the lanes gather 64 fragments' weights and features at a
// time, and the sums run over them one by one in list order, a channel per lane
// (the same operations in the same order as k_pt_blend, so the results are the
// same to the bit): 0.97 ms for those 27M, of which the records, the lists and
// 8-byte features from scattered lines are most.
//
// It takes the splats that counted over kRsDense fragments per layer pixel;
// the count is on the device, so where the capacity allows that many all three
// kernels are launched and those not meant leave at once (9 us for the screen
// order's and this one).  Whole splat, this way with the screen order against the
// two kernels: one 512 crop 256 us and 169 at 3.2 fragments per pixel, 328 and 322
// at 6.3, 399 and 497 at 9.5, 1.94 ms and 10.9 at 76; crops of 64, 128 and 256 59
// and 55, 74 and 65, 129 and 118 at 8, 61 and 69, 77 and 79, 138 and 144 at 10 (a
// wave per pixel idles on short lists).  The sides meet at 6.5 for a large crop and
// at 10 for small ones; the line is above both, as the launches that only leave
// are an eighth of a small splat's time.
constexpr uint32_t kRsWave = 256;   // fragments that one wave ranks
constexpr int kRsCap = 4096, kRsBuckets = 1024, kRsPix = 4;   // pixels per workgroup, one wave each

// A list of at most 64 R fragments ranked by one wave, R per lane in registers,
// each compared with all of them by broadcast.  Beyond one fragment per lane
// the ranks' sum tells whether any depths are equal (each equal pair is
// missing from it); those take the points' own order.
template <int R>
__device__ inline void rs_rank_wave(const uint4* __restrict__ seg, uint32_t start, int n,
                                    uint32_t pixel, uint32_t* __restrict__ fin,
                                    const uint32_t* __restrict__ ids, uint32_t* okey,
                                    uint64_t* oval, int lane) {
  uint4 rec[R];
  uint32_t rank[R], sum = 0, same = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    rec[r] = lane + 64 * r < n ? seg[start + lane + 64 * r] : make_uint4(0, 0, 0, 0);
    rank[r] = 0;
  }
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int m = min(64, n - 64 * q);
    for (int j = 0; j < m; ++j) {
      const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)rec[q].y, j);
#pragma unroll
      for (int r = 0; r < R; ++r) rank[r] += d < rec[r].y ? 1u : 0u;
      if (R == 1) same += d == rec[0].y ? 1u : 0u;
    }
  }
  bool ties;
  if (R == 1) {
    ties = __ballot(lane < n && same > 1) != 0;
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) sum += lane + 64 * r < n ? rank[r] : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += (uint32_t)__shfl_xor((int)sum, o, 64);
    ties = __builtin_amdgcn_readfirstlane((int)sum) != n * (n - 1) / 2;
  }
  if (ties) {
    uint32_t own[R];
#pragma unroll
    for (int r = 0; r < R; ++r) own[r] = ids && lane + 64 * r < n ? ids[rec[r].x] : rec[r].x;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const int m = min(64, n - 64 * q);
      for (int j = 0; j < m; ++j) {
        const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)rec[q].y, j);
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)own[q], j);
#pragma unroll
        for (int r = 0; r < R; ++r) rank[r] += d == rec[r].y && o < own[r] ? 1u : 0u;
      }
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (lane + 64 * r >= n) continue;
    okey[start + rank[r]] = pixel;
    oval[start + rank[r]] = ((uint64_t)rec[r].z << 32) | rec[r].x;
    fin[start + lane + 64 * r] = start + rank[r];
  }
}

__global__ __launch_bounds__(256) void k_pt_resolve(
    const uint4* __restrict__ seg, uint32_t* __restrict__ fin,
    const uint32_t* __restrict__ poff,
    const uint32_t* __restrict__ total_p, int64_t max_frags, int64_t pix_total,
    uint32_t* __restrict__ left, uint32_t* __restrict__ pcnt,
    const uint32_t* __restrict__ ids, const uint16_t* __restrict__ feat,
    const float* __restrict__ opacity, int64_t np, uint32_t* __restrict__ okey,
    uint64_t* oval, float4* __restrict__ pyr) {
  __shared__ __align__(16) uint64_t s_key[kRsCap];      // (depth key << 32 | segment place), by bucket
  __shared__ uint32_t s_cur[kRsBuckets];   // bucket starts, advanced to their ends by the placing
  __shared__ uint32_t s_n[kRsPix], s_left[kRsPix], s_w[4], s_v[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t total = *total_p;
  if (total <= kRsDense * pix_total) return;
  const bool over = total > max_frags;
  // most fragments that a workgroup compares with one another: what the LDS
  // holds (a bucket of 4096 takes it about 0.5 ms), less where there are fewer
  // pixels than workgroups and that would be the launch's time
  const uint32_t bucket_cap = pix_total < 1024 ? 512 : kRsCap;
  // pixels in reverse: the coarse layers' long lists start early
  for (int64_t k0 = pix_total - kRsPix * ((int64_t)blockIdx.x + 1); k0 > -kRsPix;
       k0 -= kRsPix * (int64_t)gridDim.x) {
    const int64_t kw = k0 + wave;   // the wave's pixel
    uint32_t start_w = 0, nw = 0;
    if (kw >= 0 && !over) {
      start_w = poff[kw];
      nw = poff[kw + 1] - start_w;
    }
    if (lane == 0) {
      s_n[wave] = nw;
      s_left[wave] = 0u;
    }
    // (uniform over the wave)
    if (nw <= 64) rs_rank_wave<1>(seg, start_w, (int)nw, (uint32_t)kw, fin, ids, okey, oval, lane);
    else if (nw <= 128) rs_rank_wave<2>(seg, start_w, (int)nw, (uint32_t)kw, fin, ids, okey, oval, lane);
    else if (nw <= kRsWave) rs_rank_wave<4>(seg, start_w, (int)nw, (uint32_t)kw, fin, ids, okey, oval, lane);
    __syncthreads();
    for (int w = 0; w < kRsPix; ++w) {
      const uint32_t n = s_n[w];
      if (n <= kRsWave) continue;   // uniform over the workgroup
      const int64_t k = k0 + w;
      const uint32_t start = poff[k];
      const uint4* sg = seg + start;
      // range of the depth keys
      uint32_t lo = ~0u, hi = 0u;
      for (uint32_t i = tid; i < n; i += 256) {
        const uint32_t d = sg[i].y;
        lo = min(lo, d);
        hi = max(hi, d);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
      }
      if (lane == 0) {
        s_w[wave] = lo;
        s_v[wave] = hi;
      }
      for (int b = tid; b < kRsBuckets; b += 256) s_cur[b] = 0;
      __syncthreads();
      lo = min(min(s_w[0], s_w[1]), min(s_w[2], s_w[3]));
      hi = max(max(s_v[0], s_v[1]), max(s_v[2], s_v[3]));
      // bucket of a key: every step is monotone, so buckets are in key order
      const float scale = (float)kRsBuckets / ((float)(hi - lo) + 1.0f);
      auto bucket = [&](uint32_t d) {
        return min((int)((float)(d - lo) * scale), kRsBuckets - 1);
      };
      for (uint32_t i = tid; i < n; i += 256) atomicAdd(&s_cur[bucket(sg[i].y)], 1u);
      __syncthreads();
      bool wide;
      // exclusive scan of the counts, four buckets per thread
      {
        uint32_t c[4], sum = 0, most = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          c[q] = s_cur[tid * 4 + q];
          sum += c[q];
          most = max(most, c[q]);
        }
        if (n > bucket_cap && __syncthreads_or(most > bucket_cap)) {
          // thousands of nearly equal depths: one workgroup would compare each
          // with all, so the pixel is left to the kernels that share it out
          if (tid == 0) {
            pcnt[k] = kRsLeft;
            s_left[w] = 1u;
            atomicAdd(left, 1u);
          }
          continue;
        }
        // large buckets: equal depths may be many (see below)
        wide = __syncthreads_or(most >= (n <= kRsCap ? 64u : 1024u)) != 0;   // s_w is read above
        uint32_t inc = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t t = (uint32_t)__shfl_up((int)inc, o, 64);
          if (lane >= o) inc += t;
        }
        if (lane == 63) s_w[wave] = inc;
        __syncthreads();
        uint32_t base = inc - sum;
        for (int q = 0; q < wave; ++q) base += s_w[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          s_cur[tid * 4 + q] = base;
          base += c[q];
        }
      }
      __syncthreads();
      // buckets [b0, b1) whose fragments fit the LDS at a time: all of them
      // for segments up to kRsCap.  A fragment is compared with its bucket's;
      // where buckets are small its equals (rare) are looked up one by one, where
      // they are large every word holds the tie's order and every group walks
      // the segment again (4M points of one depth, one 512 crop: 7.7 ms, 7.8 with
      // a numbering; 24.5 and 142 by lookups)
      uint32_t done = 0;   // fragments of the buckets before b0
      for (int b0 = 0; b0 < kRsBuckets && done < n;) {
        int b1 = kRsBuckets;
        if (n - done > kRsCap) {
          int most = b0 + 1;
          for (int b = tid * 4; b < tid * 4 + 4; ++b)
            if (b > b0 && s_cur[b] - done <= kRsCap) most = max(most, b);
#pragma unroll
          for (int o = 32; o > 0; o >>= 1) most = max(most, __shfl_xor(most, o, 64));
          __syncthreads();
          if (lane == 0) s_w[wave] = (uint32_t)most;
          __syncthreads();
          b1 = (int)max(max(s_w[0], s_w[1]), max(s_w[2], s_w[3]));
        }
        const uint32_t cnt = (b1 < kRsBuckets ? s_cur[b1] : n) - done;
        __syncthreads();   // b1's start is read before any placing moves a cursor
        auto put = [&](const uint4& rec, uint32_t i, uint32_t rank) {
          okey[start + rank] = (uint32_t)k;
          oval[start + rank] = ((uint64_t)rec.z << 32) | rec.x;
          fin[start + i] = start + rank;
        };
        auto own_id = [&](uint32_t x) { return ids ? ids[x] : x; };
        // the words of a key's bucket
        auto span = [&](int b, uint32_t& first, uint32_t& last) {
          first = b == b0 ? 0u : s_cur[b - 1] - done;
          last = s_cur[b] - done;
        };
        if (wide) {
          // words of the points' own order, and the fragments by place
          for (uint32_t i = tid; i < n; i += 256) {
            const uint4 rec = sg[i];
            const int b = bucket(rec.y);
            if (b >= b0 && b < b1)
              s_key[atomicAdd(&s_cur[b], 1u) - done] = ((uint64_t)rec.y << 32) | own_id(rec.x);
          }
          __syncthreads();
          for (uint32_t i = tid; i < n; i += 256) {
            const uint4 rec = sg[i];
            const int b = bucket(rec.y);
            if (b < b0 || b >= b1) continue;
            const uint64_t own = ((uint64_t)rec.y << 32) | own_id(rec.x);
            uint32_t first, last;
            span(b, first, last);
            uint32_t rank = first;
            for (uint32_t q = first; q < last; ++q) rank += s_key[q] < own ? 1u : 0u;
            put(rec, i, done + rank);
          }
        } else {
          for (uint32_t i = tid; i < n; i += 256) {
            const uint32_t d = sg[i].y;
            const int b = bucket(d);
            if (b >= b0 && b < b1)
              s_key[atomicAdd(&s_cur[b], 1u) - done] = ((uint64_t)d << 32) | i;
          }
          __syncthreads();
          for (uint32_t p = tid; p < cnt; p += 256) {
            const uint64_t e = s_key[p];
            const uint32_t d = (uint32_t)(e >> 32);
            const uint4 rec = sg[(uint32_t)e];
            uint32_t first, last;
            span(bucket(d), first, last);
            uint32_t rank = first;
            for (uint32_t q = first; q < last; ++q) {
              const uint64_t f = s_key[q];
              const uint32_t df = (uint32_t)(f >> 32);
              rank += df < d ? 1u : 0u;
              if (df == d && q != p)   // equal depths: the points' own order
                rank += own_id(sg[(uint32_t)f].x) < own_id(rec.x) ? 1u : 0u;
            }
            put(rec, (uint32_t)e, done + rank);
          }
        }
        __syncthreads();
        done += cnt;
        b0 = b1;
      }
    }
    __syncthreads();   // the sorted lists are written, s_key is free
    const bool skip = s_left[wave] != 0u;
    if (skip) nw = 0;
    // weights, 1 - weights and four features of 64 fragments, per wave
    float* st = reinterpret_cast<float*>(s_key) + wave * (6 * 64);
    const uint64_t* list = oval + start_w;
    const int ch = lane & 3;
    float F = 0.0f, T = 1.0f;
    uint64_t v = lane < (int)nw ? list[lane] : ~0ull;
    for (uint32_t j0 = 0; j0 < nw; j0 += 64) {
      const uint32_t id = (uint32_t)v;
      const bool ok = id < (uint64_t)np;
      const float w = __uint_as_float((uint32_t)(v >> 32));
      float al = 0.0f;
      uint2 hb = make_uint2(0, 0);
      if (ok) {
        al = opacity ? w * opacity[id] : w;
        hb = *reinterpret_cast<const uint2*>(feat + (int64_t)id * 4);
      }
      v = j0 + 64 + lane < nw ? list[j0 + 64 + lane] : ~0ull;
      st[lane] = al;
      st[64 + lane] = 1.0f - al;
      st[128 + lane] = h2f((uint16_t)(hb.x & 0xffffu));
      st[192 + lane] = h2f((uint16_t)(hb.x >> 16));
      st[256 + lane] = h2f((uint16_t)(hb.y & 0xffffu));
      st[320 + lane] = h2f((uint16_t)(hb.y >> 16));
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // (lanes past the list hold weight 0 and leave both sums as they are)
      const int cnt = (int)min(nw - j0, 64u);
#pragma unroll 4
      for (int i = 0; i < cnt; i += 4) {
        const float4 a4 = *reinterpret_cast<const float4*>(st + i);
        const float4 o4 = *reinterpret_cast<const float4*>(st + 64 + i);
        const float4 h4 = *reinterpret_cast<const float4*>(st + 128 + ch * 64 + i);
        const float a[4] = {a4.x, a4.y, a4.z, a4.w}, o[4] = {o4.x, o4.y, o4.z, o4.w};
        const float h[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float aT = a[q] * T;
          F += h[q] * aT;
          T = T * o[q];
        }
      }
      __builtin_amdgcn_wave_barrier();   // read before the next batch's stores
    }
    if (lane < 4 && kw >= 0 && !skip) reinterpret_cast<float*>(pyr + kw)[lane] = F;
    __syncthreads();   // the shared words are reused by the next pixels
  }
}

__global__ void k_zero4(float4* p, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

}  // namespace vrs

using namespace vrs;

static bool check_views(const vrs_view* views, int nv, KViews* kv) {
  if (!make_views(views, nv, kv)) return false;
  for (int i = 1; i < nv; ++i)
    if (views[i].width != views[0].width || views[i].height != views[0].height) return false;
  return true;
}

extern "C" size_t vrs_splat_workspace_size(int64_t np, int n_views, const vrs_view* views,
                                           const vrs_crop* crops, int n_crops, int levels,
                                           int64_t max_frags) {
  SplatWs L;
  KViews kv;
  KCrops kc;
  if (!check_views(views, n_views, &kv) ||
      !make_crops(crops, n_crops, levels, kv, &kc, nullptr, false))
    return 0;
  if (!splat_layout_for(np, n_views, views, crops, n_crops, levels, max_frags, &L)) return 0;
  return L.total;
}

extern "C" vrs_status vrs_splat_workspace_layout(int64_t np, int n_views, const vrs_view* views,
                                                 const vrs_crop* crops, int n_crops, int levels,
                                                 int64_t max_frags, vrs_splat_layout* out) {
  SplatWs L;
  if (!out || !splat_layout_for(np, n_views, views, crops, n_crops, levels, max_frags, &L))
    return VRS_EINVAL;
  out->frag_count = L.frag_count;
  out->sorted_keys = L.fkey1;
  out->sorted_ids = L.fval1;   // low 32 bits of each 64-bit value
  out->pyramid_pixels = L.pix_total;
  return VRS_OK;
}

namespace vrs {
vrs_status splat_impl(const float* pos, const float* radius, const uint16_t* feat,
                      const float* opacity, int64_t np, int channels, int levels,
                      const vrs_view* views, int n_views, const vrs_crop* crops, int n_crops,
                      const vrs_crop_place* place, const float* depth, const float* t_final,
                      float cov_min, float slack, const uint32_t* point_ids, float* pyramid,
                      void* ws, size_t ws_bytes, int64_t max_frags, int32_t* dev_status,
                      void* stream, const Trace* tr, const float* gaze) {
  KViews kv;
  KCrops kc;
  SplatWs L;
  if (gaze && !place) return VRS_EINVAL;
  if (channels != 4) return channels > 0 ? VRS_EUNSUPPORTED : VRS_EINVAL;
  if (!check_views(views, n_views, &kv) || !make_crops(crops, n_crops, levels, kv, &kc, place))
    return VRS_EINVAL;
  if (np < 0 || np * n_views >= (int64_t(1) << 30) ||
      (np > 0 && (!pos || !radius || !feat)))
    return VRS_EINVAL;
  if ((depth == nullptr) != (t_final == nullptr)) return VRS_EINVAL;
  if (!pyramid || !ws || max_frags < 0 || max_frags >= (int64_t(1) << 30)) return VRS_EINVAL;
  if (!splat_layout_for(np, n_views, views, crops, n_crops, levels, max_frags, &L) || ws_bytes < L.total)
    return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  PtArgs a;
  a.cov_min = cov_min;
  a.slack = slack;
  a.levels = levels;
  a.view_mask = 0;
  for (int k = 0; k < n_crops; ++k) a.view_mask |= 1u << crops[k].view;
  a.ord_side = L.surv2 ? ord_side(crops, n_crops) : 0;
  const int64_t vn = L.vn;
  uint32_t* frag_count = at<uint32_t>(ws, L.frag_count);
  trace_begin(tr, VRS_TRACE_SPLAT, st);
  if (vn == 0 || n_crops == 0) {
    if (gaze && n_crops > 0) {   // the crops are still placed for the later stages
      hipLaunchKernelGGL(k_place_crops, dim3(1), dim3(64), 0, st,
                         reinterpret_cast<const float2*>(gaze), kc,
                         reinterpret_cast<int4*>(const_cast<vrs_crop_place*>(place)));
      VRS_LAUNCH_CHECK();
    }
    if (L.pix_total > 0) {
      const int blocks = (int)std::min<int64_t>(4096, div_up(L.pix_total, 256));
      hipLaunchKernelGGL(k_zero4, dim3(blocks), dim3(256), 0, st,
                         reinterpret_cast<float4*>(pyramid), L.pix_total);
      VRS_LAUNCH_CHECK();
    }
    VRS_HIP_CHECK(fill_u32(frag_count, 0, 1, st));
    trace_end(tr, VRS_TRACE_SPLAT, st);
    return VRS_OK;
  }
  uint32_t* live = at<uint32_t>(ws, L.live);
  // Without the cull every workgroup has survivors, and what many of them wait
  // for is their atomic on the one counter (about 11 ns each): half as many of
  // them (5M points: 97 -> 72 us).  With it the reads under the points bound it
  // (two 2016 x 2240 views: 62 us, 65 with 512), and under 1M points too few
  // workgroups would be left.
  const bool wide = !t_final && np >= (int64_t(1) << 20);
  const int sel_block = wide ? 512 : 256;
  const int sel_parts = div_up(np, sel_block * kSelRounds);
  const size_t sel_lds = (size_t)kSelRounds * n_views * 256 * 8;   // (counts alone with 512)
  uint32_t* grid = at<uint32_t>(ws, L.grid);
  // Points in no spatial order read T' and depth from a cache line each.  One
  // image of the depths that hide points halves those reads; it costs 12 bytes
  // a view pixel, so it is made where at least a quarter as many points reach
  // a crop's area (2M points, four 1024 x 1024 views with a 512 crop each:
  // 93 -> 73 us with the image).  A numbering says that the points are stored
  // in spatial order: two reads then cost little more than one (5M points,
  // stereo 2016 x 2240: 63 us against 57).
  float* hide = L.hide && t_final && !point_ids ? at<float>(ws, L.hide) : nullptr;
  const int64_t pixels = (int64_t)n_views * views[0].width * views[0].height;
  {
    const int64_t cells = (int64_t)n_views * L.gx * L.gy;
    const int64_t scan_words = (int64_t)(scan_tmp_bytes(L.pix_total) / 4);
    const int64_t most = std::max(std::max<int64_t>(L.pix_total, scan_words),
                                  std::max(cells, hide ? pixels : 0));
    hipLaunchKernelGGL(k_pt_prep, dim3((unsigned)std::min<int64_t>(4096, div_up(most, 256))),
                       dim3(256), 0, st, at<uint32_t>(ws, L.pcnt), L.pix_total,
                       at<uint64_t>(ws, L.ctr), at<uint32_t>(ws, L.scan_tmp), scan_words, kc,
                       n_views, levels, L.gx, L.gy, grid, reinterpret_cast<const float2*>(gaze),
                       reinterpret_cast<int4*>(const_cast<vrs_crop_place*>(place)), depth, t_final,
                       a, hide, pixels);
    VRS_LAUNCH_CHECK();
  }
  // survivors with their fragment offsets (compaction order), then emission
  auto select = a.ord_side ? (wide ? k_pt_select<512, true> : k_pt_select<256, true>)
                           : (wide ? k_pt_select<512, false> : k_pt_select<256, false>);
  hipLaunchKernelGGL(select, dim3(sel_parts), dim3(sel_block), sel_lds, st, pos, radius, np, kv, kc,
                     a, depth, t_final, hide, grid, L.gx, L.gy, at<uint4>(ws, L.surv),
                     at<uint64_t>(ws, L.ctr), at<uint32_t>(ws, L.chunk_first), max_frags,
                     dev_status);
  VRS_LAUNCH_CHECK();
  const uint4* surv2 = L.surv2 ? at<uint4>(ws, L.surv2) : nullptr;
  const float4* at2 = at<float4>(ws, L.seg);   // the segments are filled after the emission
  if (L.surv2) {
    uint64_t* hist = at<uint64_t>(ws, L.ord_hist);
    hipLaunchKernelGGL(k_pt_ord_count, dim3(L.ord_parts), dim3(kOrdBlock), 0, st,
                       at<uint4>(ws, L.surv), live, frag_count, max_frags, L.pix_total, hist);
    VRS_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_pt_ord_scan, dim3(kOrdBuckets / 64), dim3(1024), 0, st, frag_count,
                       max_frags, L.pix_total, hist, L.ord_parts);
    VRS_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_pt_ord_move, dim3(L.ord_parts), dim3(kOrdBlock), 0, st, pos, radius, np,
                       at<uint4>(ws, L.surv), live, frag_count, max_frags, L.pix_total, hist,
                       at<uint4>(ws, L.surv2), at<float4>(ws, L.seg),
                       at<uint32_t>(ws, L.chunk_first));
    VRS_LAUNCH_CHECK();
  }
  uint32_t* pcnt = at<uint32_t>(ws, L.pcnt);
  uint32_t* poff = at<uint32_t>(ws, L.poff);
  // one workgroup per chunk of the capacity's fragment range (grid-stride
  // beyond 8192 chunks); workgroups past the counted chunks leave at once
  const int64_t emit_blocks =
      std::min<int64_t>(8192, std::max<int64_t>(1, div_up(max_frags, kEmitFrags)));
  hipLaunchKernelGGL(k_pt_emit, dim3((unsigned)emit_blocks), dim3(kEmitBlock), 0, st, pos, radius,
                     np, kv, kc, a, at<uint4>(ws, L.surv), surv2, at2, L.pix_total, live,
                     at<uint32_t>(ws, L.chunk_first),
                     frag_count, max_frags, at<uint32_t>(ws, L.fkey0), at<uint64_t>(ws, L.fval0),
                     at<uint32_t>(ws, L.fdep), at<uint32_t>(ws, L.fslot), pcnt, grid, L.gx, L.gy,
                     dev_status);
  VRS_LAUNCH_CHECK();
  // per-pixel segments, then each fragment to its place in blend order
  VRS_HIP_CHECK(exclusive_scan_u32(pcnt, nullptr, poff, poff + L.pix_total, nullptr, L.pix_total,
                                   at<void>(ws, L.scan_tmp), dev_status, st, true));
  const unsigned fb = (unsigned)std::min<int64_t>(8192, std::max<int64_t>(1, div_up(max_frags, 256)));
  hipLaunchKernelGGL(k_pt_scatter, dim3(fb), dim3(256), 0, st, at<uint32_t>(ws, L.fkey0),
                     at<uint64_t>(ws, L.fval0), at<uint32_t>(ws, L.fdep),
                     at<uint32_t>(ws, L.fslot), poff, frag_count, max_frags,
                     at<uint4>(ws, L.seg));
  VRS_LAUNCH_CHECK();
  // long lists are ranked and blended together (four workgroups per compute
  // unit, what the LDS holds), short ones by a thread per fragment and pixel
  const bool dense = max_frags > kRsDense * L.pix_total;
  if (dense) {
    const unsigned rb = (unsigned)std::min<int64_t>(4 * device_cus(), div_up(L.pix_total, kRsPix));
    hipLaunchKernelGGL(k_pt_resolve, dim3(rb), dim3(256), 0, st, at<uint4>(ws, L.seg),
                       at<uint32_t>(ws, L.fdep), poff,
                       frag_count, max_frags, L.pix_total, at<uint32_t>(ws, L.left), pcnt,
                       point_ids, feat, opacity, np, at<uint32_t>(ws, L.fkey1), at<uint64_t>(ws, L.fval1),
                       reinterpret_cast<float4*>(pyramid));
    VRS_LAUNCH_CHECK();
  }
  hipLaunchKernelGGL((dense ? k_pt_rank<true> : k_pt_rank<false>), dim3(fb), dim3(256), 0, st, at<uint4>(ws, L.seg),
                     at<uint32_t>(ws, L.fdep), poff,
                     frag_count, max_frags, L.pix_total, at<uint32_t>(ws, L.left), pcnt, point_ids,
                     at<uint32_t>(ws, L.fkey1),
                     at<uint64_t>(ws, L.fval1));
  VRS_LAUNCH_CHECK();
  const unsigned pb = (unsigned)std::min<int64_t>(8192, std::max<int64_t>(1, div_up(L.pix_total, 256)));
  hipLaunchKernelGGL((dense ? k_pt_blend<true> : k_pt_blend<false>), dim3(pb), dim3(256), 0, st, at<uint64_t>(ws, L.fval1), poff,
                     frag_count, max_frags, at<uint32_t>(ws, L.left), pcnt, feat, opacity, np,
                     L.pix_total, reinterpret_cast<float4*>(pyramid));
  VRS_LAUNCH_CHECK();
  trace_end(tr, VRS_TRACE_SPLAT, st);
  return VRS_OK;
}
}  // namespace vrs

extern "C" vrs_status vrs_splat_points(const float* pos, const float* radius,
                                       const uint16_t* feat, const float* opacity, int64_t np,
                                       int channels, int levels, const vrs_view* views,
                                       int n_views, const vrs_crop* crops, int n_crops,
                                       const vrs_crop_place* place, const float* depth,
                                       const float* t_final, float cov_min, float slack,
                                       const uint32_t* point_ids, float* pyramid, void* ws,
                                       size_t ws_bytes, int64_t max_frags, int32_t* dev_status,
                                       void* stream) {
  return splat_impl(pos, radius, feat, opacity, np, channels, levels, views, n_views, crops,
                    n_crops, place, depth, t_final, cov_min, slack, point_ids, pyramid, ws,
                    ws_bytes, max_frags, dev_status, stream, nullptr);
}

// ------------------------------------------------------------- backward
namespace vrs {

// The adjoint in two kernels.  With G = feat . dF and A the same product for
// the colour behind a fragment, a fragment's feature gradient is alpha T dF and
// its alpha's is T (G - A), T the transmittance before it.  T is a prefix
// product of 1 - alpha over the pixel's list and A a suffix composition of
// A -> alpha G + (1 - alpha) A, so 16 lanes take a pixel and scan 16 fragments
// at a time (row shifts); a fully opaque fragment (alpha >= 1) cuts both, also
// where what lies behind it is not finite.  The second kernel gathers a point's
// fragments and carries them into the point.  Both are latency-bound.  Fitting workload (2M points, four 512 crops): one
// thread walking each list took 864 us, the two take 165.
constexpr int kPbLanes = 16;

template <int CTRL>
__device__ inline float row_shift(float v, float edge) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), CTRL,
                                                    0xf, 0xf, false));
}

__global__ __launch_bounds__(256) void k_pt_scan_bwd(
    const uint64_t* __restrict__ fval, const uint32_t* __restrict__ poff,
    const uint32_t* __restrict__ total_p, int64_t max_frags, const uint16_t* __restrict__ feat,
    const float* __restrict__ opacity, int64_t np, int64_t pix_total,
    const float4* __restrict__ dpyr, float2* res) {
  if ((int64_t)*total_p > max_frags) return;
  const int lane = threadIdx.x & 63, li = lane % kPbLanes, row = lane / kPbLanes;
  // a wave looks at 64 pixels, one per lane, and takes those that hold
  // fragments four at a time, one per row of lanes (most pixels hold none)
  for (int64_t p0 = (blockIdx.x * (int64_t)256 + threadIdx.x - lane); p0 < pix_total;
       p0 += (int64_t)gridDim.x * 256) {
    const uint32_t start_l = p0 + lane < pix_total ? poff[p0 + lane] : 0u;
    const uint32_t n_l = p0 + lane < pix_total ? poff[p0 + lane + 1] - start_l : 0u;
    for (uint64_t m = __ballot(n_l > 0); m;) {
      int at = -1;
#pragma unroll
      for (int r = 0; r < 64 / kPbLanes; ++r) {
        if (row == r && m) at = __builtin_ctzll(m);
        m &= m - 1;   // (stays 0 once empty)
      }
      const uint32_t start = (uint32_t)__shfl((int)start_l, at, 64);
      const int n_at = __shfl((int)n_l, at, 64);   // by every lane: the source is any of them
      const int n = at < 0 ? 0 : n_at;
      const int64_t p = p0 + at;
      if (n == 0) continue;
      const float4 g = dpyr[p];
      const int last = (n - 1) / kPbLanes;
      // alpha, 1 - alpha (0 from an opaque one on) and T of the lane's fragment
      // in chunk c; T0: before the chunk, advanced past it
      float al = 0.0f, om = 1.0f, G = 0.0f, Tb = 0.0f, T0 = 1.0f;
      auto load = [&](int c) {
        const int j = c * kPbLanes + li;
        al = 0.0f;
        om = 1.0f;
        G = 0.0f;
        if (j < n) {
          const uint64_t v = fval[start + j];
          const uint32_t id = (uint32_t)v;
          if (id < (uint64_t)np) {
            const float w = __uint_as_float((uint32_t)(v >> 32));
            al = opacity ? w * opacity[id] : w;
            om = al >= 1.0f ? 0.0f : 1.0f - al;
            const uint2 hb = *reinterpret_cast<const uint2*>(feat + (int64_t)id * 4);
            G = h2f((uint16_t)(hb.x & 0xffffu)) * g.x + h2f((uint16_t)(hb.x >> 16)) * g.y +
                h2f((uint16_t)(hb.y & 0xffffu)) * g.z + h2f((uint16_t)(hb.y >> 16)) * g.w;
          }
        }
      };
      auto scan_T = [&]() {
        float q = om;   // inclusive products over the row: row_shr 1, 2, 4, 8
        q *= row_shift<0x111>(q, 1.0f);
        q *= row_shift<0x112>(q, 1.0f);
        q *= row_shift<0x114>(q, 1.0f);
        q *= row_shift<0x118>(q, 1.0f);
        Tb = T0 * row_shift<0x111>(q, 1.0f);
        T0 *= __shfl(q, kPbLanes - 1, kPbLanes);
      };
      // the chunks before the last leave T for the walk back
      for (int c = 0; c <= last; ++c) {
        load(c);
        scan_T();
        if (c < last) res[start + c * kPbLanes + li].x = Tb;
      }
      float Aend = 0.0f;   // A behind the chunk
      for (int c = last; c >= 0; --c) {
        if (c < last) {
          load(c);
          Tb = res[start + c * kPbLanes + li].x;
        }
        // suffix compositions of A -> b + a A over the row: row_shl 1, 2, 4, 8
        float a = om, b = al * G;
        auto over = [&](float behind) { return a == 0.0f ? b : fmaf(a, behind, b); };
        b = over(row_shift<0x101>(b, 0.0f));
        a *= row_shift<0x101>(a, 1.0f);
        b = over(row_shift<0x102>(b, 0.0f));
        a *= row_shift<0x102>(a, 1.0f);
        b = over(row_shift<0x104>(b, 0.0f));
        a *= row_shift<0x104>(a, 1.0f);
        b = over(row_shift<0x108>(b, 0.0f));
        a *= row_shift<0x108>(a, 1.0f);
        const float here = over(Aend);   // A before the lane's fragment
        const float A = row_shift<0x101>(here, Aend);
        Aend = __shfl(here, 0, kPbLanes);
        const int j = c * kPbLanes + li;
        // (behind an opaque fragment: nothing, whatever G and A are)
        if (j < n)
          res[start + j] = Tb == 0.0f ? make_float2(0.0f, 0.0f) : make_float2(al * Tb, Tb * (G - A));
      }
    }
  }
}

// A quad of lanes per survivor walks its crops and layers as the emission
// did, a lane per footprint target, so that the target's fragment is the next
// of the survivor's in emission order; its place in the sorted lists is
// fslot -> fin.  The quad's sums go out once per survivor (two atomic
// instructions) instead of eight scattered atomics per fragment, which bound
// the per-fragment form (726 us against 91).
// res: each sorted fragment's alpha T and alpha gradient.
template <int CTRL>
__device__ inline float quad_add(float v) {
  return v + __int_as_float(
                 __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ inline float quad_sum(float v) { return quad_add<0x4E>(quad_add<0xB1>(v)); }

__global__ __launch_bounds__(256) void k_pt_blend_bwd(
    const uint4* __restrict__ surv1, const uint4* __restrict__ surv2, int64_t pix_total,
    const uint32_t* __restrict__ live_p, const uint32_t* __restrict__ total_p, int64_t max_frags,
    const uint32_t* __restrict__ fslot,
    const uint32_t* __restrict__ fin, const float* __restrict__ pos,
    const float* __restrict__ radius, const float* __restrict__ opacity, int64_t np, KViews views,
    KCrops crops, PtArgs a, const uint32_t* __restrict__ grid, int gx, int gy,
    const float4* __restrict__ dpyr, const float2* __restrict__ res, float* __restrict__ d_feat,
    float* __restrict__ d_pos, float* __restrict__ d_radius, float* __restrict__ d_opacity) {
  __shared__ int s_cx0[VRS_MAX_CROPS], s_cy0[VRS_MAX_CROPS], s_cs[VRS_MAX_CROPS],
      s_pb[VRS_MAX_CROPS];
  if (threadIdx.x < crops.n) {
    s_cx0[threadIdx.x] = crop_x0(crops, threadIdx.x);
    s_cy0[threadIdx.x] = crop_y0(crops, threadIdx.x);
    s_cs[threadIdx.x] = crops.c[threadIdx.x].size;
    s_pb[threadIdx.x] = crops.c[threadIdx.x].pix_base;
  }
  __syncthreads();
  const int64_t total = *total_p, live = *live_p;
  if (total > max_frags) return;
  const uint4* __restrict__ surv =
      surv2 && pt_dense(total, max_frags, pix_total) ? surv2 : surv1;   // as the emission read them
  const int q = threadIdx.x & 3, dx = q & 1, dy = q >> 1;
  for (int64_t j = (blockIdx.x * (int64_t)256 + threadIdx.x) >> 2; j < live;
       j += (int64_t)gridDim.x * 64) {
    const uint4 sv = surv[j];
    const int v = (int)(sv.x / np);
    const int64_t i = sv.x - (int64_t)v * np;
    const KView& cv = views.v[v];
    const float x = pos[i], y = pos[np + i], z = pos[2 * np + i];
    PtGeom g;
    if (!pt_geom32(cv, x, y, z, radius[i], a.levels, g)) continue;
    const float o = opacity ? opacity[i] : 1.0f;
    float f = 0.0f;
    if (g.two) f = log2f(g.s) - (float)g.l0;
    FF ux, uy;
    pt_plane_ff(cv, x, y, z, ux, uy);
    // the lane's sums: features, the point's opacity, pixel position, size
    float df[4] = {0, 0, 0, 0}, dop = 0.0f, dpx = 0.0f, dpy = 0.0f, ds = 0.0f;
    int64_t at = sv.z;   // the survivor's next fragment
    for (uint32_t cand = pt_candidates(cv, v, crops.n, grid, gx, gy, x, y, z); cand;
         cand &= cand - 1) {
      const int k = __builtin_ctz(cand);
      const int cx0 = s_cx0[k], cy0 = s_cy0[k], size = s_cs[k];
      int lb = s_pb[k];
      int l = 0;
      for (; l < g.l0; ++l) lb += (size >> l) * (size >> l);
      for (int li = 0; li < (g.two ? 2 : 1); ++li, ++l) {
        const int Sl = size >> l;
        float xl, yl;
        int ix, iy;
        if (pt_layer32(g, cx0, cy0, l, Sl, xl, yl, ix, iy)) {
          const bool x0 = ix >= 0, x1 = ix + 1 < Sl, y0 = iy >= 0, y1 = iy + 1 < Sl;
          const int nx = (x0 ? 1 : 0) + (x1 ? 1 : 0);
          if ((dx ? x1 : x0) && (dy ? y1 : y0)) {
            const int64_t e = at + (dy && y0 ? nx : 0) + (dx && x0 ? 1 : 0);
            const uint32_t place = e < total ? fslot[e] : ~0u;
            const uint32_t at_list = place < total ? fin[place] : ~0u;
            if (at_list < total) {
              const float2 r = res[at_list];
              float4 gp = dpyr[lb + (iy + dy) * Sl + ix + dx];
              // (a fragment that is not seen takes nothing, whatever the pixel's gradient)
              if (r.x == 0.0f && r.y == 0.0f) gp = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
              df[0] = fmaf(r.x, gp.x, df[0]);
              df[1] = fmaf(r.x, gp.y, df[1]);
              df[2] = fmaf(r.x, gp.z, df[2]);
              df[3] = fmaf(r.x, gp.w, df[3]);
              const float bx = pt_frac_ff(cv.fx, ux, cv.cx, cx0, l, ix);
              const float by = pt_frac_ff(cv.fy, uy, cv.cy, cy0, l, iy);
              const float wx = dx ? bx : 1.0f - bx, wy = dy ? by : 1.0f - by;
              const float wl = g.two ? (li == 0 ? 1.0f - f : f) : 1.0f;
              const float dw = r.y * o;
              dop = fmaf(r.y, wl * (wx * wy), dop);
              // trilinear weight: layer weight x bilinear weight
              const float sc = ldexpf(1.0f, -l);
              dpx += dw * wl * wy * (dx ? sc : -sc);
              dpy += dw * wl * wx * (dy ? sc : -sc);
              if (g.two) ds += (li == 0 ? -dw : dw) * wx * wy / (g.s * 0.69314718055994531f);
            }
          }
          at += nx * ((y0 ? 1 : 0) + (y1 ? 1 : 0));
        }
        lb += Sl * Sl;
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) df[c] = quad_sum(df[c]);
    dop = quad_sum(dop);
    dpx = quad_sum(dpx);
    dpy = quad_sum(dpy);
    ds = quad_sum(ds);
    // lane q: feature q, position q (q < 3) or the radius
    if (d_feat) {
      const float m = q == 0 ? df[0] : (q == 1 ? df[1] : (q == 2 ? df[2] : df[3]));
      if (m != 0.0f) atomicAdd(&d_feat[i * 4 + q], m);
    }
    const float tz = g.t[2];
    const float dt0 = dpx * cv.fx / tz, dt1 = dpy * cv.fy / tz;
    const float dt2 = -dpx * cv.fx * g.t[0] / (tz * tz) - dpy * cv.fy * g.t[1] / (tz * tz) -
                      ds * g.s / tz;
    const int qr = q < 3 ? q : 0;
    const float m = q < 3 ? cv.R[qr] * dt0 + cv.R[3 + qr] * dt1 + cv.R[6 + qr] * dt2
                          : ds * 2.0f * cv.fx / tz;
    float* to = q < 3 ? (d_pos ? d_pos + q * np + i : nullptr)
                      : (d_radius ? d_radius + i : nullptr);
    if (to && m != 0.0f) atomicAdd(to, m);
    if (d_opacity && opacity && q == 0) atomicAdd(&d_opacity[i], dop);
  }
}

}  // namespace vrs

extern "C" vrs_status vrs_splat_points_backward(const float* pos, const float* radius,
                                                const uint16_t* feat, const float* opacity,
                                                int64_t np, int channels, int levels,
                                                const vrs_view* views, int n_views,
                                                const vrs_crop* crops, int n_crops,
                                                const vrs_crop_place* place,
                                                const float* d_pyramid, float* d_feat,
                                                float* d_pos, float* d_radius, float* d_opacity,
                                                void* ws, size_t ws_bytes, int64_t max_frags,
                                                void* stream) {
  KViews kv;
  KCrops kc;
  SplatWs L;
  if (channels != 4) return channels > 0 ? VRS_EUNSUPPORTED : VRS_EINVAL;
  if (!check_views(views, n_views, &kv) || !make_crops(crops, n_crops, levels, kv, &kc, place))
    return VRS_EINVAL;
  if (!splat_layout_for(np, n_views, views, crops, n_crops, levels, max_frags, &L) || !ws ||
      ws_bytes < L.total || !d_pyramid)
    return VRS_EINVAL;
  if (np > 0 && (!pos || !radius || !feat)) return VRS_EINVAL;
  if (np == 0 || n_crops == 0) return VRS_OK;
  PtArgs a;
  a.cov_min = 0.5f;
  a.slack = 1.05f;
  a.levels = levels;
  a.view_mask = 0;
  for (int k = 0; k < n_crops; ++k) a.view_mask |= 1u << crops[k].view;
  a.ord_side = L.surv2 ? ord_side(crops, n_crops) : 0;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the emission's weights are free: two numbers per fragment there
  float2* res = at<float2>(ws, L.fval0);
  const int sb = (int)std::min<int64_t>(16384, div_up(L.pix_total, 256));
  hipLaunchKernelGGL(k_pt_scan_bwd, dim3(sb), dim3(256), 0, st, at<uint64_t>(ws, L.fval1),
                     at<uint32_t>(ws, L.poff), at<uint32_t>(ws, L.frag_count), max_frags, feat,
                     opacity, np, L.pix_total, reinterpret_cast<const float4*>(d_pyramid), res);
  VRS_LAUNCH_CHECK();
  // no more survivors than fragments or (view, point) pairs
  const int bb = (int)std::min<int64_t>(
      8192, std::max(1, div_up(std::min<int64_t>(max_frags, L.vn), 64)));
  hipLaunchKernelGGL(k_pt_blend_bwd, dim3(bb), dim3(256), 0, st, at<uint4>(ws, L.surv),
                     L.surv2 ? at<uint4>(ws, L.surv2) : nullptr, L.pix_total,
                     at<uint32_t>(ws, L.live), at<uint32_t>(ws, L.frag_count), max_frags,
                     at<uint32_t>(ws, L.fslot), at<uint32_t>(ws, L.fdep), pos, radius, opacity, np, kv,
                     kc, a, at<uint32_t>(ws, L.grid), L.gx, L.gy,
                     reinterpret_cast<const float4*>(d_pyramid), res, d_feat, d_pos, d_radius,
                     d_opacity);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

// ------------------------------------------------------- crop placement

extern "C" vrs_status vrs_place_crops(const float* gaze, const vrs_view* views, int n_views,
                                      const vrs_crop* crops, int n_crops, vrs_crop_place* place,
                                      void* stream) {
  KViews kv;
  KCrops kc;
  if (!gaze || !place || n_crops < 1 || !check_views(views, n_views, &kv) ||
      !make_crops(crops, n_crops, 1, kv, &kc, nullptr, false))
    return VRS_EINVAL;
  hipLaunchKernelGGL(k_place_crops, dim3(1), dim3(64), 0, static_cast<hipStream_t>(stream),
                     reinterpret_cast<const float2*>(gaze), kc, reinterpret_cast<int4*>(place));
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}
