// Combination of the periphery P and the foveal images F (Sec. 3.4,
// Eqs. 2-5), its adjoint, and the L1 photometric term of the fitting loss
// (Sec. 3.5, Eq. 6).
//
// One thread per four full-frame pixels of a row (one per pixel when the
// width is not a multiple of 4): the crop table travels as a kernel argument,
// each pixel walks the crops of its view in index order.  HBM-bound: P is
// read and out written once; F is read only under the crops.  In place (out
// is P) only the four-pixel groups under some crop are read and written.
#include "vrs_common.h"

namespace vrs {

struct CompArgs {
  int n_crops, W, H, nv, mode;
  float ring, m, gamma;
  int view[VRS_MAX_CROPS], x0[VRS_MAX_CROPS], y0[VRS_MAX_CROPS], S[VRS_MAX_CROPS];
  float gx[VRS_MAX_CROPS], gy[VRS_MAX_CROPS];
  long long fbase[VRS_MAX_CROPS];
  const int4* place;   // device crop placement (x0, y0, gaze), or null
};

// Origin and gaze of crop k: the host values, or the device placement
// table's (origins clamped into the view).
// Crop origin and gaze from the host table, or from the device placement
// table `pl` (a.place, or a workgroup's copy of it in LDS).
__device__ inline int cx0(const CompArgs& a, int k, const int4* pl) {
  return pl ? clamp_origin(pl[k].x, a.W - a.S[k]) : a.x0[k];
}
__device__ inline int cy0(const CompArgs& a, int k, const int4* pl) {
  return pl ? clamp_origin(pl[k].y, a.H - a.S[k]) : a.y0[k];
}
__device__ inline float cgx(const CompArgs& a, int k, const int4* pl) {
  return pl ? __int_as_float(pl[k].z) : a.gx[k];
}
__device__ inline float cgy(const CompArgs& a, int k, const int4* pl) {
  return pl ? __int_as_float(pl[k].w) : a.gy[k];
}
__device__ inline int cx0(const CompArgs& a, int k) { return cx0(a, k, a.place); }
__device__ inline int cy0(const CompArgs& a, int k) { return cy0(a, k, a.place); }
__device__ inline float cgx(const CompArgs& a, int k) { return cgx(a, k, a.place); }
__device__ inline float cgy(const CompArgs& a, int k) { return cgy(a, k, a.place); }

__device__ inline float clamp01(float x) { return x < 0.0f ? 0.0f : (x > 1.0f ? 1.0f : x); }

__device__ inline float gray_at(const float* F, int S, int x, int y) {
  x = x < 0 ? 0 : (x > S - 1 ? S - 1 : x);
  y = y < 0 ? 0 : (y > S - 1 ? S - 1 : y);
  const long long pl = (long long)S * S, o = (long long)y * S + x;
  return (F[o] + F[pl + o] + F[2 * pl + o]) * (1.0f / 3.0f);
}

// Sobel gradients of the channel-mean image at (x, y), replicated borders.
__device__ inline void sobel(const float* F, int S, int x, int y, float& gx, float& gy) {
  const float a = gray_at(F, S, x - 1, y - 1), b = gray_at(F, S, x, y - 1),
              c = gray_at(F, S, x + 1, y - 1), d = gray_at(F, S, x - 1, y),
              e = gray_at(F, S, x + 1, y), f = gray_at(F, S, x - 1, y + 1),
              g = gray_at(F, S, x, y + 1), h = gray_at(F, S, x + 1, y + 1);
  gx = (c + 2.0f * e + h) - (a + 2.0f * d + f);
  gy = (f + 2.0f * g + h) - (a + 2.0f * b + c);
}

__device__ inline float smootherstep(float x) { return x * x * x * (x * (6.0f * x - 15.0f) + 10.0f); }
__device__ inline float smootherstep_d(float x) { return 30.0f * x * x * (x - 1.0f) * (x - 1.0f); }

// Blend mask c of crop k at crop pixel (lx, ly); u_out = argument of S2
// (PAPER mode), fe_out = edge term.
__device__ inline float blend_mask(const CompArgs& a, int k, const float* F, int lx, int ly,
                                   float& u_out, float& gx, float& gy, const int4* pl) {
  const float dx = (float)(cx0(a, k, pl) + lx) + 0.5f - cgx(a, k, pl);
  const float dy = (float)(cy0(a, k, pl) + ly) + 0.5f - cgy(a, k, pl);
  const float r = sqrtf(dx * dx + dy * dy);
  const float df = 0.5f * (float)a.S[k];
  if (a.mode == VRS_BLEND_LINEAR) {
    u_out = 0.0f;
    gx = gy = 0.0f;
    return clamp01((df - r) / a.ring);
  }
  const float rn = clamp01(r / df);
  const float fp = (rn - a.m) / (1.0f - a.m);
  // gamma = 0: Eq. 5 without the edge term (Eq. 4), no Sobel work
  gx = gy = 0.0f;
  if (a.gamma != 0.0f) sobel(F, a.S[k], lx, ly, gx, gy);
  const float fe = 0.25f * sqrtf(gx * gx + gy * gy);
  u_out = fp + a.gamma * fe;
  return 1.0f - smootherstep(clamp01(u_out));
}

__global__ __launch_bounds__(256) void k_composite(CompArgs a, const float* P,
                                                   const float* __restrict__ F, float* out) {
  const long long plane = (long long)a.W * a.H;
  const long long total = plane * a.nv;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int v = (int)(i / plane);
    const long long pi = i - v * plane;
    const int y = (int)(pi / a.W), x = (int)(pi - (long long)y * a.W);
    const long long base = (long long)v * 3 * plane + pi;
    float o0 = P[base], o1 = P[base + plane], o2 = P[base + 2 * plane];
    for (int k = 0; k < a.n_crops; ++k) {
      if (a.view[k] != v) continue;
      const int lx = x - cx0(a, k), ly = y - cy0(a, k), S = a.S[k];
      if (lx < 0 || ly < 0 || lx >= S || ly >= S) continue;
      {
        // outside the crop's inscribed circle the mask is 0 in both modes
        const float dx = (float)(cx0(a, k) + lx) + 0.5f - cgx(a, k);
        const float dy = (float)(cy0(a, k) + ly) + 0.5f - cgy(a, k);
        if (!(sqrtf(dx * dx + dy * dy) < 0.5f * (float)S)) continue;
      }
      const float* Fk = F + a.fbase[k];
      float u, gx, gy;
      const float c = blend_mask(a, k, Fk, lx, ly, u, gx, gy, a.place);
      const long long fp = (long long)S * S, fo = (long long)ly * S + lx;
      o0 = (1.0f - c) * o0 + c * Fk[fo];
      o1 = (1.0f - c) * o1 + c * Fk[fp + fo];
      o2 = (1.0f - c) * o2 + c * Fk[2 * fp + fo];
    }
    out[base] = o0;
    out[base + plane] = o1;
    out[base + 2 * plane] = o2;
  }
}

// Same per pixel as k_composite, four consecutive pixels of a row per thread
// (W % 4 == 0): 16-byte loads and stores of P and out, crops rejected once
// per four pixels.
// Four pixels (v, y, x..x+3) of a row: their crop chain from P into out
// (which may be P: every read comes before the writes).
// cand: the crops that may cover the quad (bit k), walked in crop order.
__device__ inline void comp_quad(const CompArgs& a, const float* P, const float* __restrict__ F,
                                 float* out, int v, int y, int x, const int4* pl, uint32_t cand) {
  const long long plane = (long long)a.W * a.H;
  const long long base = (long long)v * 3 * plane + (long long)y * a.W + x;
  float4 c4[3] = {*reinterpret_cast<const float4*>(P + base),
                  *reinterpret_cast<const float4*>(P + base + plane),
                  *reinterpret_cast<const float4*>(P + base + 2 * plane)};
  float o[3][4];
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) {
    o[ch][0] = c4[ch].x; o[ch][1] = c4[ch].y; o[ch][2] = c4[ch].z; o[ch][3] = c4[ch].w;
  }
  while (cand) {
    const int k = __builtin_ctz(cand);
    cand &= cand - 1;
    if (a.view[k] != v) continue;
    const int S = a.S[k], ly = y - cy0(a, k, pl);
    if (ly < 0 || ly >= S || x + 3 < cx0(a, k, pl) || x >= cx0(a, k, pl) + S) continue;
    const float* Fk = F + a.fbase[k];
    const long long fp = (long long)S * S;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int lx = x + j - cx0(a, k, pl);
      if (lx < 0 || lx >= S) continue;
      {
        // outside the crop's inscribed circle the mask is 0 in both modes
        // (the same operations as blend_mask): the pixel keeps its value
        const float dx = (float)(cx0(a, k, pl) + lx) + 0.5f - cgx(a, k, pl);
        const float dy = (float)(cy0(a, k, pl) + ly) + 0.5f - cgy(a, k, pl);
        if (!(sqrtf(dx * dx + dy * dy) < 0.5f * (float)S)) continue;
      }
      float u, gx, gy;
      const float c = blend_mask(a, k, Fk, lx, ly, u, gx, gy, pl);
      const long long fo = (long long)ly * S + lx;
      o[0][j] = (1.0f - c) * o[0][j] + c * Fk[fo];
      o[1][j] = (1.0f - c) * o[1][j] + c * Fk[fp + fo];
      o[2][j] = (1.0f - c) * o[2][j] + c * Fk[2 * fp + fo];
    }
  }
#pragma unroll
  for (int ch = 0; ch < 3; ++ch)
    *reinterpret_cast<float4*>(out + base + ch * plane) =
        make_float4(o[ch][0], o[ch][1], o[ch][2], o[ch][3]);
}

__global__ __launch_bounds__(256) void k_composite4(CompArgs a, const float* __restrict__ P,
                                                    const float* __restrict__ F,
                                                    float* __restrict__ out) {
  const long long plane = (long long)a.W * a.H, qplane = plane / 4;
  const long long total = qplane * a.nv;
  for (long long q = blockIdx.x * (long long)blockDim.x + threadIdx.x; q < total;
       q += (long long)gridDim.x * blockDim.x) {
    const int v = (int)(q / qplane);
    const long long pi = (q - v * qplane) * 4;
    const int y = (int)(pi / a.W), x = (int)(pi - (long long)y * a.W);
    comp_quad(a, P, F, out, v, y, x, a.place, a.n_crops >= 32 ? ~0u : (1u << a.n_crops) - 1u);
  }
}

// In place: workgroup (b, k) takes crop k's four-pixel groups [256 b,
// 256 b + 256) in row order over the crop's rows and the groups its columns
// touch; a group under several crops is done once, by the first of them,
// with the whole crop chain.  Pixels under no crop are not touched.
__global__ __launch_bounds__(256) void k_composite4_inplace(CompArgs a, float* io,
                                                            const float* __restrict__ F) {
  // the device placement table read once per workgroup: every pixel walks
  // the crop chain, which would otherwise wait on a load per crop
  __shared__ int4 s_pl[VRS_MAX_CROPS];
  __shared__ uint32_t s_near;
  const int4* pl = nullptr;
  if (a.place) {   // uniform
    if (threadIdx.x < a.n_crops) s_pl[threadIdx.x] = a.place[threadIdx.x];
    __syncthreads();
    pl = s_pl;
  }
  const int kc = blockIdx.y;
  const int S = a.S[kc], v = a.view[kc];
  const int gx0 = cx0(a, kc, pl) >> 2, ng = ((cx0(a, kc, pl) + S - 1) >> 2) - gx0 + 1;
  // the crops whose square meets this crop's four-pixel groups: the only
  // ones any of the workgroup's groups can lie under (crop kc among them)
  if (threadIdx.x < 64) {
    const int k = threadIdx.x;
    bool near = false;
    if (k < a.n_crops && a.view[k] == v) {
      const int kx = cx0(a, k, pl), ky = cy0(a, k, pl), ks = a.S[k];
      const int ky0 = cy0(a, kc, pl);
      near = kx < (gx0 + ng) * 4 && kx + ks > gx0 * 4 && ky < ky0 + S && ky + ks > ky0;
    }
    const uint64_t m = __ballot(near);
    if (threadIdx.x == 0) s_near = (uint32_t)m;
  }
  __syncthreads();
  const uint32_t near = s_near;
  const long long i = blockIdx.x * 256LL + threadIdx.x;
  if (i >= (long long)S * ng) return;
  const int ly = (int)(i / ng);
  const int y = cy0(a, kc, pl) + ly, x = (gx0 + (int)(i - (long long)ly * ng)) * 4;
  for (uint32_t e = near & ((1u << kc) - 1u); e; e &= e - 1) {
    const int k = __builtin_ctz(e);
    if (a.view[k] == v && y >= cy0(a, k, pl) && y < cy0(a, k, pl) + a.S[k] &&
        x + 3 >= cx0(a, k, pl) && x < cx0(a, k, pl) + a.S[k])
      return;   // an earlier crop's group
  }
  comp_quad(a, io, F, io, v, y, x, pl, near);
}

// Adjoint.  With g the gradient of the image after crop k's blend,
//   dF_k += c_k g,  dc_k = <g, F_k - out_{k-1}>,  g <- (1 - c_k) g,  dP += g.
// In PAPER mode dc_k also flows into F_k through the Sobel edge term.  Two
// kernels: the periphery's gradient per view pixel, and each crop's per crop
// pixel (one thread owns each gradient element, so nothing is atomic).  A
// pixel under several crops walks those, and recomputes their masks, in both;
// where many crops lie over one another, with the edge term, k_composite_bwd
// walks each view pixel's chain once instead (see kCompChain).
// Four 1024 x 1024 views with a 512 crop each, with the edge term: 48 us and 28
// us, 40 and 24 written instead of added (together 155 with per-pixel chains in
// scratch memory and 27 atomics per edge pixel).

// The crops of view v over pixel (x, y), as bits (of those in `cand`).
__device__ inline uint32_t comp_over(const CompArgs& a, int v, int x, int y, uint32_t cand) {
  uint32_t m = 0;
  for (; cand; cand &= cand - 1) {
    const int k = __builtin_ctz(cand);
    if (a.view[k] != v) continue;
    const int lx = x - cx0(a, k), ly = y - cy0(a, k);
    if (lx >= 0 && ly >= 0 && lx < a.S[k] && ly < a.S[k]) m |= 1u << k;
  }
  return m;
}
// Whether the mask may be non-zero at distance r from the gaze: inside the
// inscribed circle, where the edge term can only raise S2's argument.
__device__ inline bool comp_inside(const CompArgs& a, int k, float r) {
  return r < 0.5f * (float)a.S[k] || (a.mode == VRS_BLEND_PAPER && a.gamma < 0.0f);
}
// Blend mask of crop k at view pixel (x, y); no Sobel work where it is 0.
__device__ inline float comp_mask(const CompArgs& a, int k, const float* __restrict__ F, int x,
                                  int y) {
  const float dx = (float)x + 0.5f - cgx(a, k), dy = (float)y + 0.5f - cgy(a, k);
  if (!comp_inside(a, k, sqrtf(dx * dx + dy * dy))) return 0.0f;
  float u, gx, gy;
  return blend_mask(a, k, F + a.fbase[k], x - cx0(a, k), y - cy0(a, k), u, gx, gy, a.place);
}

// VEC pixels of a row per thread (4 where rows and pointers allow).
// ADD: added to dP, else written.
template <int VEC, bool ADD>
__global__ __launch_bounds__(256) void k_composite_bwd_p(CompArgs a, const float* __restrict__ F,
                                                         const float* __restrict__ dout,
                                                         float* __restrict__ dP) {
  const long long plane = (long long)a.W * a.H, per = plane / VEC;
  const uint32_t all = a.n_crops >= 32 ? ~0u : (1u << a.n_crops) - 1u;
  const int v = blockIdx.y;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < per; i += (long long)gridDim.x * 256) {
    const long long pi = i * VEC;
    const int y = plane >> 32 ? (int)(pi / a.W) : (int)((uint32_t)pi / (uint32_t)a.W);
    const int x = (int)(pi - (long long)y * a.W);
    // the crops over any of the pixels
    uint32_t near = 0;
    for (int k = 0; k < a.n_crops; ++k) {
      if (a.view[k] != v) continue;
      const int lx = x - cx0(a, k), ly = y - cy0(a, k);
      if (ly >= 0 && ly < a.S[k] && lx + VEC > 0 && lx < a.S[k]) near |= 1u << k;
    }
    near &= all;
    float f[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) {
      f[j] = 1.0f;
      if (near)
        for (uint32_t m = comp_over(a, v, x + j, y, near); m;) {   // last crop first
          const int k = 31 - __builtin_clz(m);
          m &= ~(1u << k);
          f[j] *= 1.0f - comp_mask(a, k, F, x + j, y);
        }
    }
    const long long base = (long long)v * 3 * plane + pi;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float* o = dP + base + c * plane;
      const float* g = dout + base + c * plane;
      if constexpr (VEC == 4) {
        const float4 d = ADD ? *reinterpret_cast<const float4*>(o) : make_float4(0, 0, 0, 0);
        const float4 e = *reinterpret_cast<const float4*>(g);
        *reinterpret_cast<float4*>(o) = make_float4(fmaf(f[0], e.x, d.x), fmaf(f[1], e.y, d.y),
                                                    fmaf(f[2], e.z, d.z), fmaf(f[3], e.w, d.w));
      } else {
        *o = fmaf(f[0], *g, ADD ? *o : 0.0f);
      }
    }
  }
}

// One 16 x 16 tile of crop blockIdx.y.  EDGE (PAPER mode with gamma): the
// tile's grey values with two pixels around, the edge term's gradient in the
// Sobel sums of every pixel with one around, gathered by the pixels it flows
// into: tap (ox, oy) of pixel p lands on the pixel at p + o clamped into the
// crop, so a border pixel also takes its own outward taps.
template <bool EDGE, bool ADD>
__global__ __launch_bounds__(256) void k_composite_bwd_f(CompArgs a, const float* __restrict__ P,
                                                         const float* __restrict__ F,
                                                         const float* __restrict__ dout,
                                                         float* __restrict__ dF) {
  constexpr int N = EDGE ? 18 : 16, OFF = EDGE ? 1 : 0;
  __shared__ float s_gray[EDGE ? 20 : 1][21];
  __shared__ float s_wx[EDGE ? 18 : 1][19], s_wy[EDGE ? 18 : 1][19];
  __shared__ float s_d[3][16][17];
  const int k = blockIdx.y, S = a.S[k], v = a.view[k];
  const int nt = (S + 15) / 16;
  if ((int)blockIdx.x >= nt * nt) return;
  const int X0 = (int)blockIdx.x % nt * 16, Y0 = (int)blockIdx.x / nt * 16;
  const int tid = threadIdx.x, ox0 = cx0(a, k), oy0 = cy0(a, k);
  const long long plane = (long long)a.W * a.H, fp = (long long)S * S;
  const float* Fk = F + a.fbase[k];
  if constexpr (EDGE) {
    for (int i = tid; i < 400; i += 256) s_gray[i / 20][i % 20] = gray_at(Fk, S, X0 + i % 20 - 2, Y0 + i / 20 - 2);
    __syncthreads();
  }
  const uint32_t all = a.n_crops >= 32 ? ~0u : (1u << a.n_crops) - 1u;
  for (int i = tid; i < N * N; i += 256) {
    const int hx = i % N, hy = i / N;
    const int lx = X0 + hx - OFF, ly = Y0 + hy - OFF;
    float wx = 0.0f, wy = 0.0f, d[3] = {0, 0, 0};
    if (lx >= 0 && ly >= 0 && lx < S && ly < S) {
      const int x = ox0 + lx, y = oy0 + ly;
      const long long base = (long long)v * 3 * plane + (long long)y * a.W + x;
      float g[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) g[c] = dout[base + c * plane];
      const uint32_t over = comp_over(a, v, x, y, all);
      for (uint32_t m = over & ~((2u << k) - 1u); m;) {   // the later crops, last first
        const int q = 31 - __builtin_clz(m);
        m &= ~(1u << q);
        const float f = 1.0f - comp_mask(a, q, F, x, y);
#pragma unroll
        for (int c = 0; c < 3; ++c) g[c] *= f;
      }
      const long long fo = (long long)ly * S + lx;
      if constexpr (!EDGE) {
        const float c = comp_mask(a, k, F, x, y);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) d[ch] = c * g[ch];
      } else {
        const float dx = (float)x + 0.5f - cgx(a, k), dy = (float)y + 0.5f - cgy(a, k);
        const float r = sqrtf(dx * dx + dy * dy), df = 0.5f * (float)S;
        if (comp_inside(a, k, r)) {
          auto gr = [&](int ex, int ey) { return s_gray[hy + 1 + ey][hx + 1 + ex]; };
          const float gx = (gr(1, -1) + 2.0f * gr(1, 0) + gr(1, 1)) -
                           (gr(-1, -1) + 2.0f * gr(-1, 0) + gr(-1, 1));
          const float gy = (gr(-1, 1) + 2.0f * gr(0, 1) + gr(1, 1)) -
                           (gr(-1, -1) + 2.0f * gr(0, -1) + gr(1, -1));
          const float mag = sqrtf(gx * gx + gy * gy);
          const float u = (clamp01(r / df) - a.m) / (1.0f - a.m) + a.gamma * (0.25f * mag);
          const float c = 1.0f - smootherstep(clamp01(u));
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) d[ch] = c * g[ch];
          if (u > 0.0f && u < 1.0f && mag > 0.0f) {
            // the image before crop k
            float o[3];
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) o[ch] = P[base + ch * plane];
            for (uint32_t m = over & ((1u << k) - 1u); m; m &= m - 1) {
              const int q = __builtin_ctz(m), Sq = a.S[q];
              const float cq = comp_mask(a, q, F, x, y);
              const float* Fq = F + a.fbase[q];
              const long long qo = (long long)(y - cy0(a, q)) * Sq + (x - cx0(a, q));
#pragma unroll
              for (int ch = 0; ch < 3; ++ch)
                o[ch] = (1.0f - cq) * o[ch] + cq * Fq[ch * (long long)Sq * Sq + qo];
            }
            const float dc = g[0] * (Fk[fo] - o[0]) + g[1] * (Fk[fp + fo] - o[1]) +
                             g[2] * (Fk[2 * fp + fo] - o[2]);
            // c = 1 - S2(u), u = fp + gamma |grad| / 4; d|g|/dg = g/|g|; grey = mean / 3
            const float s = -smootherstep_d(u) * a.gamma * dc * 0.25f / mag / 3.0f;
            wx = s * gx;
            wy = s * gy;
          }
        }
      }
    }
    if constexpr (EDGE) {
      s_wx[hy][hx] = wx;
      s_wy[hy][hx] = wy;
    }
    const int cx = hx - OFF, cy = hy - OFF;
    if (cx >= 0 && cy >= 0 && cx < 16 && cy < 16)
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) s_d[ch][cy][cx] = d[ch];
  }
  __syncthreads();
  const int cx = tid & 15, cy = tid >> 4, lx = X0 + cx, ly = Y0 + cy;
  if (lx >= S || ly >= S) return;
  float e = 0.0f;
  if constexpr (EDGE) {
    // Sobel factors of the taps that land here from the pixel at offset d on
    // one axis: the derivative's (-1, 0, 1) and the smoothing's (1, 2, 1)
    auto deriv = [&](int d, int t) {
      return d ? (float)-d : (t == S - 1 ? 1.0f : 0.0f) - (t == 0 ? 1.0f : 0.0f);
    };
    auto smooth = [&](int d, int t) {
      return d ? 1.0f : 2.0f + (t == S - 1 ? 1.0f : 0.0f) + (t == 0 ? 1.0f : 0.0f);
    };
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy)
#pragma unroll
      for (int dx = -1; dx <= 1; ++dx)   // (pixels outside the crop hold zeros)
        e += deriv(dx, lx) * smooth(dy, ly) * s_wx[cy + 1 + dy][cx + 1 + dx] +
             smooth(dx, lx) * deriv(dy, ly) * s_wy[cy + 1 + dy][cx + 1 + dx];
  }
  float* o = dF + a.fbase[k] + (long long)ly * S + lx;
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) o[ch * fp] = (ADD ? o[ch * fp] : 0.0f) + (s_d[ch][cy][cx] + e);
}

// The adjoint per view pixel: the crop chain is replayed forward to recover the
// intermediate images (each crop's mask computed once), then walked backwards.
// In PAPER mode the edge term is scattered to the 3x3 neighbourhood with
// atomics.
__global__ __launch_bounds__(256) void k_composite_bwd(CompArgs a, const float* __restrict__ P,
                                                       const float* __restrict__ F,
                                                       const float* __restrict__ dout,
                                                       float* __restrict__ dP,
                                                       float* __restrict__ dF) {
  const long long plane = (long long)a.W * a.H;
  const long long total = plane * a.nv;
  for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < total;
       i += (long long)gridDim.x * blockDim.x) {
    const int v = (int)(i / plane);
    const long long pi = i - v * plane;
    const int y = (int)(pi / a.W), x = (int)(pi - (long long)y * a.W);
    const long long base = (long long)v * 3 * plane + pi;
    int ks[VRS_MAX_CROPS];
    int nk = 0;
    for (int k = 0; k < a.n_crops; ++k) {
      if (a.view[k] != v) continue;
      const int lx = x - cx0(a, k), ly = y - cy0(a, k);
      if (lx < 0 || ly < 0 || lx >= a.S[k] || ly >= a.S[k]) continue;
      ks[nk++] = k;
    }
    float g0 = dout[base], g1 = dout[base + plane], g2 = dout[base + 2 * plane];
    if (nk > 0) {
      // forward replay: o_j = image after crop j
      float o[VRS_MAX_CROPS + 1][3];
      float cs[VRS_MAX_CROPS], us[VRS_MAX_CROPS], gxs[VRS_MAX_CROPS], gys[VRS_MAX_CROPS];
      o[0][0] = P[base]; o[0][1] = P[base + plane]; o[0][2] = P[base + 2 * plane];
      for (int j = 0; j < nk; ++j) {
        const int k = ks[j], S = a.S[k];
        const int lx = x - cx0(a, k), ly = y - cy0(a, k);
        const float* Fk = F + a.fbase[k];
        cs[j] = blend_mask(a, k, Fk, lx, ly, us[j], gxs[j], gys[j], a.place);
        const long long fp = (long long)S * S, fo = (long long)ly * S + lx;
        for (int ch = 0; ch < 3; ++ch)
          o[j + 1][ch] = (1.0f - cs[j]) * o[j][ch] + cs[j] * Fk[ch * fp + fo];
      }
      for (int j = nk - 1; j >= 0; --j) {
        const int k = ks[j], S = a.S[k];
        const int lx = x - cx0(a, k), ly = y - cy0(a, k);
        const float* Fk = F + a.fbase[k];
        const long long fp = (long long)S * S, fo = (long long)ly * S + lx;
        const float c = cs[j];
        const float f0 = Fk[fo], f1 = Fk[fp + fo], f2 = Fk[2 * fp + fo];
        const float dc = g0 * (f0 - o[j][0]) + g1 * (f1 - o[j][1]) + g2 * (f2 - o[j][2]);
        if (dF) {
          float* dFk = dF + a.fbase[k];
          if (a.mode == VRS_BLEND_PAPER) {
            // neighbours scatter into this crop pixel too (edge term)
            atomicAdd(&dFk[fo], c * g0);
            atomicAdd(&dFk[fp + fo], c * g1);
            atomicAdd(&dFk[2 * fp + fo], c * g2);
          } else {
            dFk[fo] += c * g0;
            dFk[fp + fo] += c * g1;
            dFk[2 * fp + fo] += c * g2;
          }
          const float u = us[j];
          if (a.mode == VRS_BLEND_PAPER && u > 0.0f && u < 1.0f) {
            // c = 1 - S2(u), u = fp + gamma |grad|/4
            const float mag = sqrtf(gxs[j] * gxs[j] + gys[j] * gys[j]);
            if (mag > 0.0f) {
              const float dfe = -smootherstep_d(u) * a.gamma * dc;
              const float s = dfe * 0.25f / mag / 3.0f;  // d|g|/dg = g/|g|; gray = mean/3
              const float wx = s * gxs[j], wy = s * gys[j];
              // Sobel taps: gx weights (+1,+2,+1 on x+1; -1,-2,-1 on x-1),
              // gy weights (+1,+2,+1 on y+1; -1,-2,-1 on y-1)
              for (int oy = -1; oy <= 1; ++oy)
                for (int ox = -1; ox <= 1; ++ox) {
                  const float kx = (float)ox * (oy == 0 ? 2.0f : 1.0f);
                  const float ky = (float)oy * (ox == 0 ? 2.0f : 1.0f);
                  const float wgt = kx * wx + ky * wy;
                  if (wgt == 0.0f) continue;
                  int sx = lx + ox, sy = ly + oy;
                  sx = sx < 0 ? 0 : (sx > S - 1 ? S - 1 : sx);
                  sy = sy < 0 ? 0 : (sy > S - 1 ? S - 1 : sy);
                  const long long so = (long long)sy * S + sx;
                  atomicAdd(&dFk[so], wgt);
                  atomicAdd(&dFk[fp + so], wgt);
                  atomicAdd(&dFk[2 * fp + so], wgt);
                }
            }
          }
        }
        g0 *= 1.0f - c;
        g1 *= 1.0f - c;
        g2 *= 1.0f - c;
      }
    }
    if (dP) {
      dP[base] += g0;
      dP[base + plane] += g1;
      dP[base + 2 * plane] += g2;
    }
  }
}

// The mean number of other crops over a crop's pixel.  k_composite_bwd_f computes
// all of their masks again for each crop, each a Sobel of 24 reads, so it grows
// with the square of the crops over one another; k_composite_bwd pays atomics
// and per-crop arrays in scratch, but each mask once.  One 1024 x 1024 view, 512
// crops over one another, with the edge term, the two kernels against
// k_composite_bwd: 2 crops 52 us and 58, 4 124 and 97, 8 366 and 175, 32 4357
// and 639 (without it the two are faster throughout).  Origins read on the
// device are not known here: such crops are taken to lie over one another.
constexpr double kCompChain = 1.5;
static double comp_overlap(const vrs_crop* crops, int n, bool placed) {
  double area = 0.0, over = 0.0;
  for (int k = 0; k < n; ++k) {
    const vrs_crop& c = crops[k];
    area += (double)c.size * c.size;
    for (int q = 0; q < n; ++q) {
      const vrs_crop& d = crops[q];
      if (q == k || d.view != c.view) continue;
      double w = std::min(c.size, d.size), h = w;
      if (!placed) {
        w = std::min(c.x0 + c.size, d.x0 + d.size) - std::max(c.x0, d.x0);
        h = std::min(c.y0 + c.size, d.y0 + d.size) - std::max(c.y0, d.y0);
      }
      if (w > 0.0 && h > 0.0) over += w * h;
    }
  }
  return area > 0.0 ? over / area : 0.0;
}

// L1: block partial sums of |pred - target| atomically added to loss[0]
// (zeroed by the preceding fill), gradient scale*sign(pred - target)/n.
// HBM-bound; two workgroups per compute unit, since every one ends with an
// atomic on the same word (about 11 ns each: 12.6M elements in 4096
// workgroups took 65 us, 35 now, 26 without the gradient).
template <int VEC>
__global__ __launch_bounds__(256) void k_l1(const float* __restrict__ pred,
                                            const float* __restrict__ target, long long n,
                                            float* loss, float* __restrict__ dpred, float scale) {
  __shared__ double s_part[4];
  double acc = 0.0;
  const float inv = 1.0f / (float)n, step = scale * inv;
  const long long vn = n / VEC;
  auto one = [&](float p, float t, float& g) {
    const float d = p - t;
    g = d > 0.0f ? step : (d < 0.0f ? -step : 0.0f);
    return fabsf(d);
  };
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < vn; i += (long long)gridDim.x * 256) {
    if constexpr (VEC == 4) {
      const float4 p = reinterpret_cast<const float4*>(pred)[i];
      const float4 t = reinterpret_cast<const float4*>(target)[i];
      float4 g;
      acc += (double)((one(p.x, t.x, g.x) + one(p.y, t.y, g.y)) +
                      (one(p.z, t.z, g.z) + one(p.w, t.w, g.w)));
      if (dpred) {
        float4 o = reinterpret_cast<float4*>(dpred)[i];
        o.x += g.x; o.y += g.y; o.z += g.z; o.w += g.w;
        reinterpret_cast<float4*>(dpred)[i] = o;
      }
    } else {
      float g;
      acc += (double)one(pred[i], target[i], g);
      if (dpred) dpred[i] += g;
    }
  }
  const long long tail = vn * VEC + blockIdx.x * 256LL + threadIdx.x;
  if (tail < n) {   // fewer than VEC elements
    float g;
    acc += (double)one(pred[tail], target[tail], g);
    if (dpred) dpred[tail] += g;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) s_part[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicAdd(loss, (float)((s_part[0] + s_part[1] + s_part[2] + s_part[3]) / (double)n));
}

__global__ void k_zero1(float* p) { *p = 0.0f; }

// The gradient alone, written: d_loss sign(pred - target) / n with d_loss a
// device scalar, so the caller need not wait for it, and nothing is read back
// or cleared first (12.6M elements: 24 us; 45 adding
// to cleared gradients).
template <int VEC>
__global__ __launch_bounds__(256) void k_l1_bwd(const float* __restrict__ pred,
                                                const float* __restrict__ target, long long n,
                                                const float* __restrict__ d_loss,
                                                float* __restrict__ dpred) {
  const float step = (d_loss ? *d_loss : 1.0f) * (1.0f / (float)n);
  auto one = [&](float p, float t) {
    const float d = p - t;
    return d > 0.0f ? step : (d < 0.0f ? -step : 0.0f);
  };
  const long long vn = n / VEC;
  for (long long i = blockIdx.x * 256LL + threadIdx.x; i < vn; i += (long long)gridDim.x * 256) {
    if constexpr (VEC == 4) {
      const float4 p = reinterpret_cast<const float4*>(pred)[i];
      const float4 t = reinterpret_cast<const float4*>(target)[i];
      reinterpret_cast<float4*>(dpred)[i] =
          make_float4(one(p.x, t.x), one(p.y, t.y), one(p.z, t.z), one(p.w, t.w));
    } else {
      dpred[i] = one(pred[i], target[i]);
    }
  }
  const long long tail = vn * VEC + blockIdx.x * 256LL + threadIdx.x;
  if (tail < n) dpred[tail] = one(pred[tail], target[tail]);
}

static bool comp_args(int nv, int W, int H, const vrs_crop* crops, int n_crops, int mode,
                      float ring, float m, float gamma, const vrs_crop_place* place,
                      CompArgs* a) {
  if (nv < 1 || nv > VRS_MAX_VIEWS || W < 1 || H < 1 || n_crops < 0 || n_crops > VRS_MAX_CROPS ||
      (n_crops > 0 && !crops))
    return false;
  if (mode != VRS_BLEND_LINEAR && mode != VRS_BLEND_PAPER) return false;
  if (mode == VRS_BLEND_LINEAR && !(ring > 0)) return false;
  if (mode == VRS_BLEND_PAPER && !(m < 1.0f)) return false;
  a->n_crops = n_crops;
  a->W = W;
  a->H = H;
  a->nv = nv;
  a->mode = mode;
  a->ring = ring;
  a->m = m;
  a->gamma = gamma;
  a->place = reinterpret_cast<const int4*>(place);
  long long fb = 0;
  for (int k = 0; k < n_crops; ++k) {
    const vrs_crop& c = crops[k];
    if (c.view < 0 || c.view >= nv || c.size < 1 || c.size > W || c.size > H) return false;
    if (!place && (c.x0 < 0 || c.y0 < 0 || c.x0 + c.size > W || c.y0 + c.size > H)) return false;
    a->view[k] = c.view;
    a->x0[k] = c.x0;
    a->y0[k] = c.y0;
    a->S[k] = c.size;
    a->gx[k] = c.gaze_x;
    a->gy[k] = c.gaze_y;
    a->fbase[k] = fb;
    fb += 3LL * c.size * c.size;
  }
  return true;
}

}  // namespace vrs

using namespace vrs;

namespace vrs {
vrs_status composite_impl(const float* rgb_periphery, int n_views, int width, int height,
                          const float* fovea_rgb, const vrs_crop* crops, int n_crops,
                          const vrs_crop_place* place, int mode, float ring, float m, float gamma,
                          float* out, void* stream, const Trace* tr) {
  CompArgs a;
  if (!comp_args(n_views, width, height, crops, n_crops, mode, ring, m, gamma, place, &a))
    return VRS_EINVAL;
  if (!rgb_periphery || !out || (n_crops > 0 && !fovea_rgb)) return VRS_EINVAL;
  const long long total = (long long)width * height * n_views;
  trace_begin(tr, VRS_TRACE_COMPOSITE, static_cast<hipStream_t>(stream));
  const bool vec4 = width % 4 == 0 && (reinterpret_cast<uintptr_t>(rgb_periphery) & 15) == 0 &&
                    (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  if (vec4 && out == rgb_periphery) {
    // four-pixel groups of the largest crop (for origins read on the
    // device, as many as any origin can give: ((S + 2) >> 2) + 1 per row)
    long long most = 0;
    for (int k = 0; k < n_crops; ++k) {
      const int S = crops[k].size;
      const long long row = place ? ((S + 2) >> 2) + 1
                                  : ((crops[k].x0 + S - 1) >> 2) - (crops[k].x0 >> 2) + 1;
      most = std::max<long long>(most, (long long)S * row);
    }
    if (n_crops > 0)
      hipLaunchKernelGGL(k_composite4_inplace, dim3((unsigned)((most + 255) / 256), n_crops),
                         dim3(256), 0, static_cast<hipStream_t>(stream), a, out, fovea_rgb);
  } else if (vec4) {
    const int blocks = (int)std::min<long long>(16384, (total / 4 + 255) / 256);
    hipLaunchKernelGGL(k_composite4, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                       a, rgb_periphery, fovea_rgb, out);
  } else {
    const int blocks = (int)std::min<long long>(16384, (total + 255) / 256);
    hipLaunchKernelGGL(k_composite, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                       a, rgb_periphery, fovea_rgb, out);
  }
  VRS_LAUNCH_CHECK();
  trace_end(tr, VRS_TRACE_COMPOSITE, static_cast<hipStream_t>(stream));
  return VRS_OK;
}
}  // namespace vrs

extern "C" vrs_status vrs_composite_frame(const float* rgb_periphery, int n_views, int width,
                                          int height, const float* fovea_rgb,
                                          const vrs_crop* crops, int n_crops,
                                          const vrs_crop_place* place, int mode, float ring,
                                          float m, float gamma, float* out, void* stream) {
  return composite_impl(rgb_periphery, n_views, width, height, fovea_rgb, crops, n_crops, place,
                        mode, ring, m, gamma, out, stream, nullptr);
}

template <bool ADD>
static vrs_status composite_backward(const float* rgb_periphery, int n_views,
                                                   int width, int height, const float* fovea_rgb,
                                                   const vrs_crop* crops, int n_crops,
                                                   const vrs_crop_place* place, int mode,
                                                   float ring, float m, float gamma,
                                                   const float* d_out, float* d_rgb_periphery,
                                                   float* d_fovea, void* stream) {
  CompArgs a;
  if (!comp_args(n_views, width, height, crops, n_crops, mode, ring, m, gamma, place, &a))
    return VRS_EINVAL;
  if (!rgb_periphery || !d_out || (n_crops > 0 && !fovea_rgb)) return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const bool edge = mode == VRS_BLEND_PAPER && gamma != 0.0f;
  if (d_fovea && edge && comp_overlap(crops, n_crops, place != nullptr) > kCompChain) {
    const long long total = (long long)width * height * n_views;
    if (!ADD) {
      if (d_rgb_periphery)
        VRS_HIP_CHECK(fill_u32(reinterpret_cast<uint32_t*>(d_rgb_periphery), 0u, 3 * total, st));
      int64_t n = 0;
      for (int k = 0; k < n_crops; ++k) n += (int64_t)3 * crops[k].size * crops[k].size;
      VRS_HIP_CHECK(fill_u32(reinterpret_cast<uint32_t*>(d_fovea), 0u, n, st));
    }
    const int blocks = (int)std::min<long long>(16384, (total + 255) / 256);
    hipLaunchKernelGGL(k_composite_bwd, dim3(blocks), dim3(256), 0, st, a, rgb_periphery,
                       fovea_rgb, d_out, d_rgb_periphery, d_fovea);
    VRS_LAUNCH_CHECK();
    return VRS_OK;
  }
  if (d_rgb_periphery) {
    const bool vec4 = width % 4 == 0 && ((reinterpret_cast<uintptr_t>(d_out) |
                                          reinterpret_cast<uintptr_t>(d_rgb_periphery)) & 15) == 0;
    const long long per = (long long)width * height / (vec4 ? 4 : 1);
    const dim3 grid((unsigned)std::min<long long>(8192, (per + 255) / 256), n_views);
    hipLaunchKernelGGL((vec4 ? k_composite_bwd_p<4, ADD> : k_composite_bwd_p<1, ADD>), grid,
                       dim3(256), 0, st, a, fovea_rgb, d_out, d_rgb_periphery);
    VRS_LAUNCH_CHECK();
  }
  if (d_fovea && n_crops > 0) {
    int most = 0;
    for (int k = 0; k < n_crops; ++k) most = std::max(most, (crops[k].size + 15) / 16);
    const dim3 grid((unsigned)(most * most), n_crops);
    hipLaunchKernelGGL((edge ? k_composite_bwd_f<true, ADD> : k_composite_bwd_f<false, ADD>), grid,
                       dim3(256), 0, st, a, rgb_periphery, fovea_rgb, d_out, d_fovea);
    VRS_LAUNCH_CHECK();
  }
  return VRS_OK;
}

extern "C" vrs_status vrs_composite_frame_backward(const float* rgb_periphery, int n_views,
                                                   int width, int height, const float* fovea_rgb,
                                                   const vrs_crop* crops, int n_crops,
                                                   const vrs_crop_place* place, int mode,
                                                   float ring, float m, float gamma,
                                                   const float* d_out, float* d_rgb_periphery,
                                                   float* d_fovea, void* stream) {
  return composite_backward<true>(rgb_periphery, n_views, width, height, fovea_rgb, crops, n_crops, place, mode, ring, m, gamma, d_out, d_rgb_periphery, d_fovea, stream);
}

extern "C" vrs_status vrs_composite_frame_backward_write(const float* rgb_periphery, int n_views,
                                                   int width, int height, const float* fovea_rgb,
                                                   const vrs_crop* crops, int n_crops,
                                                   const vrs_crop_place* place, int mode,
                                                   float ring, float m, float gamma,
                                                   const float* d_out, float* d_rgb_periphery,
                                                   float* d_fovea, void* stream) {
  return composite_backward<false>(rgb_periphery, n_views, width, height, fovea_rgb, crops, n_crops, place, mode, ring, m, gamma, d_out, d_rgb_periphery, d_fovea, stream);
}

extern "C" vrs_status vrs_l1_loss(const float* pred, const float* target, int64_t n, float* loss,
                                  float* d_pred, float scale, void* stream) {
  if (!pred || !target || !loss || n < 1) return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_zero1, dim3(1), dim3(1), 0, st, loss);
  const bool vec4 = ((reinterpret_cast<uintptr_t>(pred) | reinterpret_cast<uintptr_t>(target) |
                      reinterpret_cast<uintptr_t>(d_pred)) & 15) == 0;
  const int blocks =
      (int)std::min<int64_t>(2 * device_cus(), ((vec4 ? (n + 3) / 4 : n) + 255) / 256);
  if (vec4)
    hipLaunchKernelGGL(k_l1<4>, dim3(blocks), dim3(256), 0, st, pred, target, (long long)n, loss,
                       d_pred, scale);
  else
    hipLaunchKernelGGL(k_l1<1>, dim3(blocks), dim3(256), 0, st, pred, target, (long long)n, loss,
                       d_pred, scale);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_l1_loss_backward(const float* pred, const float* target, int64_t n,
                                           const float* d_loss, float* d_pred, void* stream) {
  if (!pred || !target || !d_pred || n < 1) return VRS_EINVAL;
  const bool vec4 = ((reinterpret_cast<uintptr_t>(pred) | reinterpret_cast<uintptr_t>(target) |
                      reinterpret_cast<uintptr_t>(d_pred)) & 15) == 0;
  const int blocks = (int)std::min<int64_t>(8192, ((vec4 ? (n + 3) / 4 : n) + 255) / 256);
  hipLaunchKernelGGL((vec4 ? k_l1_bwd<4> : k_l1_bwd<1>), dim3(blocks), dim3(256), 0,
                     static_cast<hipStream_t>(stream), pred, target, (long long)n, d_loss, d_pred);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}
