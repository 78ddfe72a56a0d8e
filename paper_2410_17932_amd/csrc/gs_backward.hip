// Peripheral 3D Gaussian splatting, backward (end-to-end fitting, Sec. 3.5).
//
//   k_gs_blend_bwd        one wave per sub-tile; every pixel replays its
//                         list back to front from its stored stop position
//                         and final transmittance (T before an entry is
//                         T after it divided by 1 - alpha), so no per-pixel
//                         lists are stored; per-entry moments of the
//                         screen-space gradient are summed over the wave
//                         and added with one atomic instruction
//   k_gs_project_bwd      one thread per Gaussian: chain rule through the
//                         conic inverse, the EWA Jacobian, the camera
//                         transform and the spherical harmonics, summed
//                         over views, accumulated into the caller's
//                         gradient planes
#include "gs_layout.h"

namespace vrs {

// Per (view, Gaussian): with s the pixel's gradient with respect to the
// exponent -d^T Q d / 2 (Q the conic), d = mean - pixel centre and u =
// -log2(e) Q d, the gradient of the opacity and the sums of s ux, s uy, s
// ux^2, s ux uy, s uy^2, and the gradients of r, g, b and z.  The position's gradient is a multiple of the
// sum of s u and the screen covariance's of s u u^T, so k_gs_project_bwd only
// scales them; sums of s d and s d d^T would still have to go through Q, which
// loses digits where Q is ill conditioned (thin Gaussians).
constexpr int kG2d = 10;

// Two values' sums over lane pairs 32 (16) lanes apart, in one register:
// the first value's in the lower 32 lanes (even rows of 16), the second's in
// the upper (odd rows).  One swap and one add for two values.
__device__ inline float pair_sum32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline float pair_sum16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sum over each row of 16 lanes, in every lane of the row.
template <int CTRL>
__device__ inline float row_rot(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ inline float row_sum(float v) {
  v += row_rot<0x128>(v);   // row_ror:8
  v += row_rot<0x124>(v);
  v += row_rot<0x122>(v);
  return v + row_rot<0x121>(v);
}

// One wave per 8 x 8 sub-tile of a tile, one pixel per lane; sub-tiles go in
// the forward's longest-list-first order.  Records are staged 64 at a time,
// one per lane, the next batch's loads issued before the current one is
// walked, and only those whose contributing ellipse may reach the sub-tile are
// walked.  Bound by vector issue (about 80 slots per record) and, where few
// tiles hold long lists, by the walk's length: four pixels per lane share the
// reduction and the atomics but were slower at every size measured (2330
// against 2099 us below, 1955 against 817 at 256 x 256).  What keeps it there:
// a pixel that does not take the entry has alpha 0, which leaves its sums as
// they are, so that only the running sum and the opacity's gradient are selected
// by the mask (all ten values where a gradient, a conic or an opacity is not
// finite, which 0 does not cancel); the colour behind an entry is needed only
// through its product with the pixel's gradient, one running sum instead of four;
// and the ten sums are reduced together, halving the registers at each exchange
// (28 instructions instead of 120), into ten lanes' one atomic instruction.  T / (1 - alpha) is the hardware reciprocal with its remainder
// put back (1 - alpha is in [0.01, 1], so no scaling is needed).
// 1M Gaussians, four 1024 x 1024 views, tile 16: 3574 us with ten reductions,
// ten atomics and all records of a tile per 64 pixels, 453 us now.
template <int TILE, bool DEPTH>
__global__ __launch_bounds__(64) void k_gs_blend_bwd(
    const uint32_t* __restrict__ order, const uint2* __restrict__ ranges,
    const uint32_t* __restrict__ ids, const float4* __restrict__ rec, int64_t n, KViews views,
    GsOpt o, int64_t tiles_x, int64_t tiles_per_view, const uint32_t* __restrict__ last_pos,
    const float* __restrict__ tfinal, const float* __restrict__ d_rgb,
    const float* __restrict__ d_depth, float* __restrict__ g2d) {
  constexpr int NQ = TILE / 8;
  __shared__ float4 s_a[64], s_b[64], s_c[64];
  __shared__ uint32_t s_id[64];
  const int64_t tglob = order[blockIdx.x / (NQ * NQ)];
  const int sub = blockIdx.x % (NQ * NQ);
  const int v = (int)(tglob / tiles_per_view);
  const int64_t tl = tglob - (int64_t)v * tiles_per_view;
  const int ty = (int)(tl / tiles_x), tx = (int)(tl - (int64_t)ty * tiles_x);
  const KView& cv = views.v[v];
  const int W = cv.W, H = cv.H, lane = threadIdx.x;
  const int sx0 = tx * TILE + sub % NQ * 8, sy0 = ty * TILE + sub / NQ * 8;
  if (sx0 >= W || sy0 >= H) return;
  const int px = sx0 + lane % 8, py = sy0 + lane / 8;
  uint32_t last = 0;
  float T = 1.0f, g0 = 0.0f, g1 = 0.0f, g2 = 0.0f, gd = 0.0f;
  if (px < W && py < H) {
    const int64_t plane = (int64_t)W * H;
    const int64_t pix = (int64_t)v * plane + (int64_t)py * W + px;
    const int64_t rp = (int64_t)v * 3 * plane + (int64_t)py * W + px;
    last = last_pos[pix];
    T = tfinal[pix];
    g0 = d_rgb[rp];
    g1 = d_rgb[rp + plane];
    g2 = d_rgb[rp + 2 * plane];
    if (DEPTH) gd = d_depth[pix];
    if (last == 0) g0 = g1 = g2 = gd = 0.0f;   // no entries: the pixel may hold anything
  }
  // the pixel's gradient times the colour behind the entry reached so far
  float A = g0 * o.bg[0] + g1 * o.bg[1] + g2 * o.bg[2];
  uint32_t most = last;
#pragma unroll
  for (int sh = 32; sh > 0; sh >>= 1) most = max(most, (uint32_t)__shfl_xor((int)most, sh, 64));
  const uint32_t stop = (uint32_t)__builtin_amdgcn_readfirstlane((int)most);
  if (stop == 0) return;
  // pixels whose gradient 0 does not cancel
  const bool wild = wave_mask(!(fabsf(g0) < INFINITY && fabsf(g1) < INFINITY &&
                                fabsf(g2) < INFINITY && fabsf(gd) < INFINITY)) != 0;
  const float aclamp = o.aclamp, amin = o.amin, inv_amin = 1.0f / amin;
  const float xc = (float)px + 0.5f, yc = (float)py + 0.5f;
  const int64_t vn = (int64_t)v * n;
  const uint32_t* list = ids + ranges[tglob].x;
  // the lane's value in the reduced layout (see the end of the record loop)
  const int l15 = lane & 15, row = lane >> 4, half = row >> 1, odd = row & 1;
  const int slot = l15 < 2 ? l15 * 4 + odd * 2 + half : 8 + half;
  const bool adds = l15 < 2 || (l15 == 2 && odd == 0 && (DEPTH || half == 0));
  // batch of positions [top - 64, top); lane l holds position top - 64 + l
  auto load_id = [&](int top) -> uint32_t {
    const int p = top - 64 + lane;
    const uint32_t id = p >= 0 ? list[p] : 0u;
    return id < (uint64_t)n ? id : 0u;
  };
  int top = (int)stop;
  uint32_t id = load_id(top);
  float4 a, b, c;
  gs_stage(rec, vn + id, a, b, c);
  uint32_t id_next = load_id(top - 64);
  for (; top > 0; top -= 64) {
    __syncthreads();
    s_a[lane] = a;
    s_b[lane] = b;
    s_c[lane] = c;
    s_id[lane] = id;
    // records whose products 0 may not cancel: a conic that is not finite or
    // overflows times a distance, an opacity that is not finite
    const float size = (fabsf(a.z) + fabsf(a.w)) + (fabsf(b.x) + fabsf(b.y));
    const uint64_t odd = wild ? ~0ull : wave_mask(!(size < 1.0e28f));
    uint64_t m;
    {
      const uint32_t lo = __float_as_uint(b.z), hi = __float_as_uint(b.w);
      const int xlo = max((int)(lo & 0xffffu), sx0), xhi = min((int)(hi & 0xffffu), sx0 + 7);
      const int ylo = max((int)(lo >> 16), sy0), yhi = min((int)(hi >> 16), sy0 + 7);
      bool reach = top - 64 + lane >= 0 && xlo <= xhi && ylo <= yhi;
      if (reach) {
        // as in the forward blend: out of reach only where every pixel's own
        // test would fail
        const float ga = -a.z, gb = -a.w, gc = -b.x;
        float thr = b.y >= amin ? __builtin_amdgcn_logf(b.y * inv_amin) * 1.001f + 1.0e-3f : -1.0f;
        if (!(ga > 0.0f && gc > 0.0f)) thr = 3.0e38f;
        const float g = box_min_quadratic(
            ga, gb, gc, 0.5f * __builtin_amdgcn_rcpf(ga), 0.5f * __builtin_amdgcn_rcpf(gc),
            a.x - ((float)xhi + 0.5f), a.x - ((float)xlo + 0.5f), a.y - ((float)yhi + 0.5f),
            a.y - ((float)ylo + 0.5f));
        reach = !(g > thr);
      }
      m = wave_mask(reach);
    }
    __syncthreads();
    id = id_next;
    if (top > 64) {
      gs_stage(rec, vn + id, a, b, c);
      id_next = load_id(top - 128);
    }
    while (m) {
      const int k = 63 - __builtin_clzll(m);
      m &= ~(1ull << k);
      const uint32_t pos = (uint32_t)(top - 64 + k);   // position in the tile list
      const float4 ka = s_a[k], kb = s_b[k], kc = s_c[k];
      const uint32_t lo = __float_as_uint(kb.z), hi = __float_as_uint(kb.w);
      const int rx0 = (int)(lo & 0xffffu), ry0 = (int)(lo >> 16);
      const float dx = ka.x - xc, dy = ka.y - yc;
      const float e = __builtin_amdgcn_exp2f(gs_exponent(ka, kb, dx, dy));
      const float oe = kb.y * e, al0 = fminf(oe, aclamp);
      const uint64_t ok = wave_mask((uint32_t)(px - rx0) <= (uint32_t)((int)(hi & 0xffffu) - rx0)) &
                          wave_mask((uint32_t)(py - ry0) <= (uint32_t)((int)(hi >> 16) - ry0)) &
                          wave_mask(al0 >= amin) & wave_mask(pos < last);
      if (ok == 0) continue;
      const bool in = lane_in(ok);
      const float al = in ? al0 : 0.0f;
      const float d = 1.0f - al;
      const float r = __builtin_amdgcn_rcpf(d);
      const float t = T * r;
      const float Tb = fmaf(fmaf(-d, t, T), r, t);
      const float w = al * Tb;
      float G = fmaf(g2, kc.z, fmaf(g1, kc.y, g0 * kc.x));
      if (DEPTH) G = fmaf(gd, kc.w, G);
      const float diff = G - A;
      A = in ? fmaf(al, diff, A) : A;   // (the colour may not be finite)
      T = Tb;
      // to the opacity and, times it, to the exponent (not by a division of the
      // latter: an opacity of 0 has a gradient where alpha_min is 0); a clamped
      // alpha carries nothing to either
      const float go = in && oe < aclamp ? (Tb * diff) * e : 0.0f;
      const float s = go * kb.y;
      const float hx = ka.z * dx;
      const float ux = fmaf(ka.w, dy, hx + hx), uy = fmaf(kb.x + kb.x, dy, ka.w * dx);
      const float sx = s * ux, sy = s * uy;
      // values 0..9 = opacity, s ux, s uy, s ux^2, s ux uy, s uy^2, r, g, b, z.
      // After the exchanges over 32 and 16 lanes, rows 0..3 of q0 hold the
      // sums of values 0, 2, 1, 3, of q1 those of 4, 6, 5, 7, of q2 8 and 9
      // in rows 0 and 2; lane 0 of each row takes q0, lane 1 q1, lane 2 q2.
      float x[10] = {go,      sx,     sy,     sx * ux, sx * uy,
                     sy * uy, w * g0, w * g1, w * g2,  DEPTH ? w * gd : 0.0f};
      if ((odd >> k) & 1)   // uniform
#pragma unroll
        for (int i = 0; i < 10; ++i) x[i] = in ? x[i] : 0.0f;
      const float p0 = pair_sum32(x[0], x[1]), p1 = pair_sum32(x[2], x[3]);
      const float p2 = pair_sum32(x[4], x[5]), p3 = pair_sum32(x[6], x[7]);
      const float p4 = pair_sum32(x[8], x[9]);
      const float q0 = row_sum(pair_sum16(p0, p1)), q1 = row_sum(pair_sum16(p2, p3));
      const float q2 = row_sum(pair_sum16(p4, 0.0f));
      const float val = l15 == 0 ? q0 : (l15 == 1 ? q1 : q2);
      if (adds) atomicAdd(g2d + (vn + s_id[k]) * kG2d + slot, val);
    }
  }
}

// derivatives of the SH basis with respect to the (unnormalised) direction
// components, contracted with dY: returns dL/d(x, y, z)
__device__ inline void sh_grad_dir(int deg, float x, float y, float z, const float* dY,
                                   float& gx, float& gy, float& gz) {
  gx = gy = gz = 0.0f;
  if (deg < 1) return;
  gy += -ShC::c1 * dY[1];
  gz += ShC::c1 * dY[2];
  gx += -ShC::c1 * dY[3];
  if (deg < 2) return;
  gx += ShC::c2a * y * dY[4];
  gy += ShC::c2a * x * dY[4];
  gy += -ShC::c2a * z * dY[5];
  gz += -ShC::c2a * y * dY[5];
  gx += -2.0f * ShC::c2b * x * dY[6];
  gy += -2.0f * ShC::c2b * y * dY[6];
  gz += 4.0f * ShC::c2b * z * dY[6];
  gx += -ShC::c2a * z * dY[7];
  gz += -ShC::c2a * x * dY[7];
  gx += 2.0f * ShC::c2c * x * dY[8];
  gy += -2.0f * ShC::c2c * y * dY[8];
  if (deg < 3) return;
  const float xx = x * x, yy = y * y, zz = z * z;
  gx += -6.0f * ShC::c3a * x * y * dY[9];
  gy += -ShC::c3a * (3.0f * xx - 3.0f * yy) * dY[9];
  gx += ShC::c3b * y * z * dY[10];
  gy += ShC::c3b * x * z * dY[10];
  gz += ShC::c3b * x * y * dY[10];
  gx += 2.0f * ShC::c3c * x * y * dY[11];
  gy += -ShC::c3c * (4.0f * zz - xx - 3.0f * yy) * dY[11];
  gz += -8.0f * ShC::c3c * y * z * dY[11];
  gx += -6.0f * ShC::c3d * x * z * dY[12];
  gy += -6.0f * ShC::c3d * y * z * dY[12];
  gz += ShC::c3d * (6.0f * zz - 3.0f * xx - 3.0f * yy) * dY[12];
  gx += -ShC::c3c * (4.0f * zz - 3.0f * xx - yy) * dY[13];
  gy += 2.0f * ShC::c3c * x * y * dY[13];
  gz += -8.0f * ShC::c3c * x * z * dY[13];
  gx += 2.0f * ShC::c3e * x * z * dY[14];
  gy += -2.0f * ShC::c3e * y * z * dY[14];
  gz += ShC::c3e * (xx - yy) * dY[14];
  gx += -ShC::c3a * (3.0f * xx - 3.0f * yy) * dY[15];
  gy += 6.0f * ShC::c3a * x * y * dY[15];
}

// HBM-bound: each attribute read once for all views (the SH coefficients stay
// in registers), the gradient planes read and written, 40 B of moments and 12
// of colour per view.  1M Gaussians of degree 3, four views: 350 us adding
// to the gradients (962 with the coefficients read twice per view under
// branches), where a Gaussian that no pixel took leaves them untouched, and
// 213 us writing them (no read of 232 MB, and none to be cleared before).
template <int DEG, bool ADD>
__global__ __launch_bounds__(256) void k_gs_project_bwd(
    const float* __restrict__ mean, const float* __restrict__ cov,
    const float* __restrict__ sh, int64_t n, KViews views, GsOpt o,
    const float4* __restrict__ rec, const float* __restrict__ g2d, float* __restrict__ d_mean,
    float* __restrict__ d_cov, float* __restrict__ d_op, float* __restrict__ d_sh) {
  constexpr int K = (DEG + 1) * (DEG + 1);
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  // the views' moments first: nothing else is read where all are zero
  bool any = false;
  for (int v = 0; v < views.n; ++v) {
    const float2* G = reinterpret_cast<const float2*>(g2d + ((int64_t)v * n + i) * kG2d);
#pragma unroll
    for (int q = 0; q < kG2d / 2; ++q) any |= G[q].x != 0.0f || G[q].y != 0.0f;
  }
  auto put = [](float& p, float v) { p = ADD ? p + v : v; };
  if (!any) {
    if (!ADD) {
#pragma unroll
      for (int k = 0; k < 3; ++k) d_mean[k * n + i] = 0.0f;
#pragma unroll
      for (int k = 0; k < 6; ++k) d_cov[k * n + i] = 0.0f;
      d_op[i] = 0.0f;
#pragma unroll
      for (int k = 0; k < 3 * K; ++k) d_sh[k * n + i] = 0.0f;
    }
    return;
  }
  const float mx = mean[i], my = mean[n + i], mz = mean[2 * n + i];
  float S6[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) S6[k] = cov[k * n + i];
  float coef[K][3];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) coef[k][ch] = sh[(k * 3 + ch) * n + i];
  float dm[3] = {0, 0, 0}, dcv[6] = {0, 0, 0, 0, 0, 0}, dopa = 0.0f;
  float dshv[K][3];
#pragma unroll
  for (int k = 0; k < K; ++k) dshv[k][0] = dshv[k][1] = dshv[k][2] = 0.0f;
  for (int v = 0; v < views.n; ++v) {
    const int64_t e = (int64_t)v * n + i;
    float G[kG2d];
#pragma unroll
    for (int q = 0; q < kG2d / 2; ++q) {
      const float2 t = reinterpret_cast<const float2*>(g2d + e * kG2d)[q];
      G[2 * q] = t.x;
      G[2 * q + 1] = t.y;
    }
    bool used = false;
#pragma unroll
    for (int q = 0; q < kG2d; ++q) used |= G[q] != 0.0f;
    if (!used) continue;
    const KView& cv = views.v[v];
    Geom g;
    if (!gs_geom32(cv, mx, my, mz, S6, o.lowpass, o.extent, g)) continue;
    // exponent -d^T Q d / 2, alpha = opacity e^exponent: dL/dd = -s Q d and,
    // with dQ = -Q dSigma Q, dL/dSigma = s (Q d) (Q d)^T / 2; u = -log2(e) Q d
    constexpr float kLn2 = 0.69314718055994531f;
    const float gpx = kLn2 * G[1], gpy = kLn2 * G[2], gz = G[9];
    dopa += G[0];
    // dL/dSigma2D as a full symmetric matrix Gs
    constexpr float h = 0.5f * kLn2 * kLn2;
    const float Gs[2][2] = {{h * G[3], h * G[4]}, {h * G[4], h * G[5]}};
    // dSigma3D = M^T Gs M ; dM = 2 Gs M Sigma
    const float S[3][3] = {{S6[0], S6[1], S6[2]}, {S6[1], S6[3], S6[4]}, {S6[2], S6[4], S6[5]}};
    float GM[2][3];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int k = 0; k < 3; ++k) GM[a][k] = Gs[a][0] * g.M[0][k] + Gs[a][1] * g.M[1][k];
    float D3[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) D3[r][k] = g.M[0][r] * GM[0][k] + g.M[1][r] * GM[1][k];
    dcv[0] += D3[0][0];
    dcv[1] += D3[0][1] + D3[1][0];
    dcv[2] += D3[0][2] + D3[2][0];
    dcv[3] += D3[1][1];
    dcv[4] += D3[1][2] + D3[2][1];
    dcv[5] += D3[2][2];
    float dM[2][3];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        dM[a][k] = 2.0f * (GM[a][0] * S[0][k] + GM[a][1] * S[1][k] + GM[a][2] * S[2][k]);
    // M0k = jx R0k + j02 R2k, M1k = jy R1k + j12 R2k
    float djx = 0, dj02 = 0, djy = 0, dj12 = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      djx += dM[0][k] * cv.R[k];
      dj02 += dM[0][k] * cv.R[6 + k];
      djy += dM[1][k] * cv.R[3 + k];
      dj12 += dM[1][k] * cv.R[6 + k];
    }
    const float tz = g.t[2];
    const float limx = 1.3f * ((0.5f * (float)cv.W) / cv.fx);
    const float limy = 1.3f * ((0.5f * (float)cv.H) / cv.fy);
    const bool inx = g.ux > -limx && g.ux < limx, iny = g.uy > -limy && g.uy < limy;
    const float cxl = clamp_f(g.ux, -limx, limx), cyl = clamp_f(g.uy, -limy, limy);
    // j02 = -jx cxl, j12 = -jy cyl
    djx += -dj02 * cxl;
    djy += -dj12 * cyl;
    float dux = inx ? -dj02 * g.jx : 0.0f;
    float duy = iny ? -dj12 * g.jy : 0.0f;
    // pixel position
    dux += gpx * cv.fx;
    duy += gpy * cv.fy;
    float dt[3];
    dt[0] = dux / tz;
    dt[1] = duy / tz;
    dt[2] = -dux * g.t[0] / (tz * tz) - duy * g.t[1] / (tz * tz) - djx * cv.fx / (tz * tz) -
            djy * cv.fy / (tz * tz) + gz;
    // colour
    float dx = mx - cv.cam[0], dy = my - cv.cam[1], dz = mz - cv.cam[2];
    const float len = sqrtf(dx * dx + dy * dy + dz * dz);
    const float rn = 1.0f / len;
    dx *= rn; dy *= rn; dz *= rn;
    float Y[16];
    sh_eval(DEG, dx, dy, dz, Y);
    float dY[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) dY[k] = 0.0f;
    // the record's colour is zero where the forward clamped it: no gradient
    const float4 r1 = rec[3 * e + 1];
    const float col[3] = {r1.z, r1.w, rec[3 * e + 2].x};
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float gc = col[ch] > 0.0f ? G[6 + ch] : 0.0f;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        dshv[k][ch] += Y[k] * gc;
        dY[k] += coef[k][ch] * gc;
      }
    }
    float gdx, gdy, gdz;
    sh_grad_dir(DEG, dx, dy, dz, dY, gdx, gdy, gdz);
    const float dot = gdx * dx + gdy * dy + gdz * dz;
    float dmv[3] = {(gdx - dx * dot) * rn, (gdy - dy * dot) * rn, (gdz - dz * dot) * rn};
    // t = R m + T
#pragma unroll
    for (int k = 0; k < 3; ++k)
      dm[k] += cv.R[k] * dt[0] + cv.R[3 + k] * dt[1] + cv.R[6 + k] * dt[2] + dmv[k];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) put(d_mean[k * n + i], dm[k]);
#pragma unroll
  for (int k = 0; k < 6; ++k) put(d_cov[k * n + i], dcv[k]);
  put(d_op[i], dopa);
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) put(d_sh[(k * 3 + ch) * n + i], dshv[k][ch]);
}

template <int TILE>
static void launch_blend_bwd(const RenderWs& L, void* ws, int64_t n, const KViews& kv,
                             const GsOpt& o, const float* tf, const float* d_rgb,
                             const float* d_depth, hipStream_t st) {
  const dim3 grid((unsigned)(L.tiles_total * (TILE / 8) * (TILE / 8)));
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(64), 0, st, at<uint32_t>(ws, L.order),
                       at<uint2>(ws, L.ranges), at<uint32_t>(ws, L.ids), at<float4>(ws, L.rec), n,
                       kv, o, L.tiles_x, L.tiles_x * L.tiles_y, at<uint32_t>(ws, L.last), tf,
                       d_rgb, d_depth, at<float>(ws, L.g2d));
  };
  if (d_depth) run(k_gs_blend_bwd<TILE, true>);
  else run(k_gs_blend_bwd<TILE, false>);
}

}  // namespace vrs

using namespace vrs;

static vrs_status render_backward(
    bool add, const float* mean, const float* cov, const float* opacity, const float* sh, int sh_degree,
    int64_t n, const vrs_view* views, int n_views, const vrs_raster_opts* ro,
    const float* t_final, const float* d_rgb, const float* d_depth, float* d_mean, float* d_cov,
    float* d_opacity, float* d_sh, void* ws, size_t ws_bytes, int64_t max_pairs, void* stream) {
  GsOpt o;
  KViews kv;
  RenderWs L;
  if (!ro || !make_views(views, n_views, &kv)) return VRS_EINVAL;
  if (ro->order != VRS_ORDER_PRIMITIVE) return VRS_EUNSUPPORTED;
  o.tile = ro->tile; o.aclamp = ro->alpha_clamp; o.amin = ro->alpha_min; o.tmin = ro->t_min;
  o.order = ro->order;
  o.lowpass = ro->lowpass; o.extent = ro->extent;
  for (int k = 0; k < 3; ++k) o.bg[k] = ro->bg[k];
  for (int i = 1; i < n_views; ++i)
    if (views[i].width != views[0].width || views[i].height != views[0].height) return VRS_EINVAL;
  if (sh_degree < 0 || sh_degree > 3 || n < 0) return VRS_EINVAL;
  if (!render_layout(n, n_views, views, o.tile, opts_radix(ro), max_pairs, &L) || !ws ||
      ws_bytes < L.total)
    return VRS_EINVAL;
  if (!t_final || !d_rgb || (n > 0 && (!mean || !cov || !opacity || !sh || !d_mean || !d_cov ||
                                       !d_opacity || !d_sh)))
    return VRS_EINVAL;
  if (n == 0) return VRS_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  VRS_HIP_CHECK(fill_u32(at<uint32_t>(ws, L.g2d), 0u, L.vn * kG2d, st));
  switch (o.tile) {
    case 8: launch_blend_bwd<8>(L, ws, n, kv, o, t_final, d_rgb, d_depth, st); break;
    case 16: launch_blend_bwd<16>(L, ws, n, kv, o, t_final, d_rgb, d_depth, st); break;
    default: launch_blend_bwd<32>(L, ws, n, kv, o, t_final, d_rgb, d_depth, st); break;
  }
  VRS_LAUNCH_CHECK();
  auto project = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(div_up(n, 256)), dim3(256), 0, st, mean, cov, sh, n,
                       kv, o, at<float4>(ws, L.rec), at<float>(ws, L.g2d), d_mean, d_cov,
                       d_opacity, d_sh);
  };
  switch (sh_degree) {
    case 0: add ? project(k_gs_project_bwd<0, true>) : project(k_gs_project_bwd<0, false>); break;
    case 1: add ? project(k_gs_project_bwd<1, true>) : project(k_gs_project_bwd<1, false>); break;
    case 2: add ? project(k_gs_project_bwd<2, true>) : project(k_gs_project_bwd<2, false>); break;
    default: add ? project(k_gs_project_bwd<3, true>) : project(k_gs_project_bwd<3, false>); break;
  }
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_render_gaussians_backward(
    const float* mean, const float* cov, const float* opacity, const float* sh, int sh_degree,
    int64_t n, const vrs_view* views, int n_views, const vrs_raster_opts* ro,
    const float* t_final, const float* d_rgb, const float* d_depth, float* d_mean, float* d_cov,
    float* d_opacity, float* d_sh, void* ws, size_t ws_bytes, int64_t max_pairs, void* stream) {
  return render_backward(true, mean, cov, opacity, sh, sh_degree, n, views, n_views, ro, t_final,
                         d_rgb, d_depth, d_mean, d_cov, d_opacity, d_sh, ws, ws_bytes, max_pairs,
                         stream);
}

extern "C" vrs_status vrs_render_gaussians_backward_write(
    const float* mean, const float* cov, const float* opacity, const float* sh, int sh_degree,
    int64_t n, const vrs_view* views, int n_views, const vrs_raster_opts* ro,
    const float* t_final, const float* d_rgb, const float* d_depth, float* d_mean, float* d_cov,
    float* d_opacity, float* d_sh, void* ws, size_t ws_bytes, int64_t max_pairs, void* stream) {
  return render_backward(false, mean, cov, opacity, sh, sh_degree, n, views, n_views, ro, t_final,
                         d_rgb, d_depth, d_mean, d_cov, d_opacity, d_sh, ws, ws_bytes, max_pairs,
                         stream);
}
