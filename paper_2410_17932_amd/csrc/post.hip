// After the combination: tone mapping (Sec. 3.4, the ADOP camera model, in
// the reading stated in vrsplat.h) and the training objective's kernels
// (Sec. 3.5, Eqs. 6-7): D-SSIM, the regulariser R, and the Adam step.
//
// All of them stream their images once (SSIM's strips and tiles re-read a 5-pixel
// halo), so each is bound by HBM bandwidth.  Sums over an image are
// deterministic (per-block partials reduced in a fixed order), except the
// gradient of a response curve of more than kTmLaneSamples samples, accumulated
// per block with LDS atomics.
#include <cmath>

#include "vrs_common.h"

namespace vrs {
namespace {

// ------------------------------------------------------------ tone mapping
constexpr int kTmFixed = 7, kTmMaxResp = 256;
constexpr int kTmBlock = 256, kTmBlocksPerView = 1024, kTmBwdBlocks = 512;

struct TmView {
  float cx, cy, inv_d2;   // principal point, rounded 1 / half-diagonal^2
};
struct TmArgs {
  TmView v[VRS_MAX_VIEWS];
  int nv, W, H, n;        // views, size, response samples
};

bool tm_args(const vrs_view* views, int nv, int n, TmArgs* a) {
  if (!views || nv < 1 || nv > VRS_MAX_VIEWS || n < 2 || n > kTmMaxResp) return false;
  const int W = views[0].width, H = views[0].height;
  if (W < 1 || H < 1) return false;
  for (int i = 0; i < nv; ++i) {
    if (views[i].width != W || views[i].height != H) return false;
    const double hd2 = (W / 2.0) * (W / 2.0) + (H / 2.0) * (H / 2.0);
    a->v[i] = TmView{views[i].cx, views[i].cy, (float)(1.0 / hd2)};
  }
  a->nv = nv;
  a->W = W;
  a->H = H;
  a->n = n;
  return true;
}

// Per-block view constants: 2^-ev rounded from double precision, white
// balance, vignetting coefficients, the response samples in LDS.
struct TmShared {
  float e, wb[3], k[3];
  float resp[kTmMaxResp];
};

__device__ inline void tm_load(TmShared& sh, const float* __restrict__ par, int n) {
  if (threadIdx.x == 0) {
    sh.e = (float)exp2(-(double)par[0]);
    for (int c = 0; c < 3; ++c) {
      sh.wb[c] = par[1 + c];
      sh.k[c] = par[4 + c];
    }
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) sh.resp[i] = par[kTmFixed + i];
  __syncthreads();
}

// Squared normalised radius and vignetting factor of pixel (x, y), in the
// documented single-precision order.
__device__ inline void tm_vig(const TmView& tv, const TmShared& sh, int x, int y, float& r2,
                              float& vig) {
#pragma clang fp contract(off)
  const float dx = ((float)x + 0.5f) - tv.cx, dy = ((float)y + 0.5f) - tv.cy;
  r2 = (dy * dy + dx * dx) * tv.inv_d2;
  vig = ((sh.k[2] * r2 + sh.k[1]) * r2 + sh.k[0]) * r2 + 1.0f;
}

// t, its segment i and fraction f, and whether t is inside (0, 1).
__device__ inline float tm_t(float x, float e, float wb, float vig) {
#pragma clang fp contract(off)
  return ((x * e) * wb) * vig;
}
__device__ inline int tm_seg(float t, int n, float& f) {
#pragma clang fp contract(off)
  const float s = fminf(fmaxf(t, 0.0f), 1.0f) * (float)(n - 1);
  const int i = min((int)floorf(s), n - 2);
  f = s - (float)i;
  return i;
}

__global__ __launch_bounds__(kTmBlock) void k_tonemap(const float* __restrict__ in,
                                                      const float* __restrict__ params, TmArgs a,
                                                      float* __restrict__ out) {
  __shared__ TmShared sh;
  const int v = blockIdx.y;
  const int P = kTmFixed + a.n;
  tm_load(sh, params + (int64_t)v * P, a.n);
  const int64_t plane = (int64_t)a.W * a.H;
  const float* src = in + (int64_t)v * 3 * plane;
  float* dst = out + (int64_t)v * 3 * plane;
  for (int64_t p = blockIdx.x * (int64_t)kTmBlock + threadIdx.x; p < plane;
       p += (int64_t)gridDim.x * kTmBlock) {
    const int y = (int)(p / a.W), x = (int)(p - (int64_t)y * a.W);
    float r2, vig;
    tm_vig(a.v[v], sh, x, y, r2, vig);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float t = tm_t(src[c * plane + p], sh.e, sh.wb[c], vig);
      float f;
      const int i = tm_seg(t, a.n, f);
      dst[c * plane + p] = fmaf(f, sh.resp[i + 1] - sh.resp[i], sh.resp[i]);
    }
  }
}

// Row and column of element p of a W-wide plane (32-bit division wherever
// the plane allows it).
__device__ inline void tm_xy(int64_t p, int64_t plane, int W, int& x, int& y) {
  if (plane >> 32) {
    y = (int)(p / W);
  } else {
    y = (int)((uint32_t)p / (uint32_t)W);
  }
  x = (int)(p - (int64_t)y * W);
}

// Adjoint: d_in written; per block partial sums of the parameters'
// gradients, [view][block][7 + n].  HBM-bound (12 B per element) once the
// response's gradient leaves the LDS atomics: those run at about one lane per
// four clocks, however the samples are spread, and held the kernel at 148 us
// for four 1024 x 1024 views.  Up to kTmLaneSamples samples every lane has a
// column of its own instead and adds to it by plain reads and writes
// (39 us); longer responses, whose columns would leave few waves in
// flight, keep atomics on one copy.
constexpr int kTmLaneSamples = 48;   // 12 KB of LDS per wave
__host__ __device__ constexpr bool tm_lanes(int n) { return n <= kTmLaneSamples; }
__host__ constexpr int tm_lds(int n) {
  return (tm_lanes(n) ? n * kTmBlock : n) * (int)sizeof(float);
}

template <bool LANES>
__global__ __launch_bounds__(kTmBlock) void k_tonemap_bwd(
    const float* __restrict__ in, const float* __restrict__ params, TmArgs a,
    const float* __restrict__ d_out, float* __restrict__ d_in, float* __restrict__ partial) {
  __shared__ TmShared sh;
  __shared__ float s_red[kTmBlock / 64][kTmFixed];
  extern __shared__ float s_dr[];   // LANES: [n][kTmBlock], else [n]
  const int v = blockIdx.y;
  const int P = kTmFixed + a.n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int i = threadIdx.x; i < (LANES ? a.n * kTmBlock : a.n); i += kTmBlock) s_dr[i] = 0.0f;
  tm_load(sh, params + (int64_t)v * P, a.n);
  const int64_t plane = (int64_t)a.W * a.H;
  const float* src = in + (int64_t)v * 3 * plane;
  const float* g = d_out + (int64_t)v * 3 * plane;
  float* dst = d_in ? d_in + (int64_t)v * 3 * plane : nullptr;
  float acc[kTmFixed] = {0, 0, 0, 0, 0, 0, 0};
  auto pixel = [&](int x, int y, const float xi[3], const float gi[3], float di[3]) {
    float r2, vig;
    tm_vig(a.v[v], sh, x, y, r2, vig);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float t = tm_t(xi[c], sh.e, sh.wb[c], vig);
      float f;
      const int i = tm_seg(t, a.n, f);
      if constexpr (LANES) {
        float* col = s_dr + i * kTmBlock + threadIdx.x;
        col[0] += gi[c] * (1.0f - f);
        col[kTmBlock] += gi[c] * f;
      } else {
        atomicAdd(&s_dr[i], gi[c] * (1.0f - f));
        atomicAdd(&s_dr[i + 1], gi[c] * f);
      }
      const bool inside = t > 0.0f && t < 1.0f;
      const float dt = inside ? gi[c] * (sh.resp[i + 1] - sh.resp[i]) * (float)(a.n - 1) : 0.0f;
      di[c] = dt * sh.e * sh.wb[c] * vig;
      acc[0] += dt * t;
      acc[1 + c] += dt * xi[c] * sh.e * vig;
      const float base = dt * xi[c] * sh.e * sh.wb[c];
      acc[4] += base * r2;
      acc[5] += base * r2 * r2;
      acc[6] += base * r2 * r2 * r2;
    }
  };
  const bool quads = plane % 4 == 0 && ((reinterpret_cast<uintptr_t>(in) |
                                         reinterpret_cast<uintptr_t>(d_out) |
                                         reinterpret_cast<uintptr_t>(d_in)) & 15) == 0;
  if (quads) {   // four elements of each plane at a time (uniform)
    for (int64_t p = 4 * (blockIdx.x * (int64_t)kTmBlock + threadIdx.x); p < plane;
         p += 4 * (int64_t)gridDim.x * kTmBlock) {
      float xi[4][3], gi[4][3], di[4][3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float4 u = *reinterpret_cast<const float4*>(src + c * plane + p);
        const float4 w = *reinterpret_cast<const float4*>(g + c * plane + p);
        xi[0][c] = u.x; xi[1][c] = u.y; xi[2][c] = u.z; xi[3][c] = u.w;
        gi[0][c] = w.x; gi[1][c] = w.y; gi[2][c] = w.z; gi[3][c] = w.w;
      }
      int x, y;
      tm_xy(p, plane, a.W, x, y);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        pixel(x, y, xi[j], gi[j], di[j]);
        if (++x == a.W) {
          x = 0;
          ++y;
        }
      }
      if (dst)
#pragma unroll
        for (int c = 0; c < 3; ++c)
          *reinterpret_cast<float4*>(dst + c * plane + p) =
              make_float4(di[0][c], di[1][c], di[2][c], di[3][c]);
    }
  } else {
    for (int64_t p = blockIdx.x * (int64_t)kTmBlock + threadIdx.x; p < plane;
         p += (int64_t)gridDim.x * kTmBlock) {
      int x, y;
      tm_xy(p, plane, a.W, x, y);
      float xi[3], gi[3], di[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        xi[c] = src[c * plane + p];
        gi[c] = g[c * plane + p];
      }
      pixel(x, y, xi, gi, di);
      if (dst)
#pragma unroll
        for (int c = 0; c < 3; ++c) dst[c * plane + p] = di[c];
    }
  }
  acc[0] *= -0.69314718055994531f;   // d t / d ev = -ln 2 t
#pragma unroll
  for (int q = 0; q < kTmFixed; ++q) {
    float s = acc[q];
#pragma unroll
    for (int sh2 = 32; sh2 > 0; sh2 >>= 1) s += __shfl_xor(s, sh2, 64);
    if (lane == 0) s_red[wave][q] = s;
  }
  __syncthreads();
  if (!partial) return;
  float* out = partial + ((int64_t)v * gridDim.x + blockIdx.x) * P;
  if (threadIdx.x < kTmFixed) {
    float s = 0.0f;
    for (int w = 0; w < kTmBlock / 64; ++w) s += s_red[w][threadIdx.x];
    out[threadIdx.x] = s;
  }
  if constexpr (!LANES) {
    for (int i = threadIdx.x; i < a.n; i += kTmBlock) out[kTmFixed + i] = s_dr[i];
  } else {
    for (int i = wave; i < a.n; i += kTmBlock / 64) {
      float s = 0.0f;
#pragma unroll
      for (int w = 0; w < kTmBlock / 64; ++w) s += s_dr[i * kTmBlock + 64 * w + lane];
#pragma unroll
      for (int sh2 = 32; sh2 > 0; sh2 >>= 1) s += __shfl_xor(s, sh2, 64);
      if (lane == 0) out[kTmFixed + i] = s;
    }
  }
}

// d_params[v][q] += sum over blocks of partial[v][b][q], in a fixed order.
__global__ __launch_bounds__(256) void k_reduce_partials(const float* __restrict__ partial,
                                                         int nb, int P,
                                                         float* __restrict__ d_params) {
  __shared__ float s[256];
  const int q = blockIdx.x, v = blockIdx.y;
  float acc = 0.0f;
  for (int b = threadIdx.x; b < nb; b += 256) acc += partial[((int64_t)v * nb + b) * P + q];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) d_params[(int64_t)v * P + q] += s[0];
}

int tm_blocks(const TmArgs& a) {
  return std::max(1, std::min(kTmBlocksPerView, div_up((int64_t)a.W * a.H, kTmBlock)));
}
// The adjoint ends each workgroup with a reduction of the response columns,
// so it takes fewer: for one view two per compute unit.
int tm_bwd_blocks(const TmArgs& a) {
  return std::max(1, std::min(kTmBwdBlocks, div_up((int64_t)a.W * a.H, kTmBlock)));
}

// ------------------------------------------------------------------- SSIM
constexpr int kSsHalo = 5, kSsTaps = 2 * kSsHalo + 1;
constexpr int kSsBlock = 128, kSsOut = 116;   // threads (input columns), output columns
constexpr int kSsRow = 132;                   // LDS row: reads of 16 from any multiple of 4

struct SsArgs {
  int planes, W, H;
  int tiles_x, tiles_y;
  int rows, groups;   // output rows per workgroup; input row groups of kSsTaps
  bool tile;          // 32 x 32 tiles (small images) instead of strips
  float w[kSsTaps];   // the window's 1-D taps, rounded from double precision
};

// Separable 11-tap blur of NM maps computed from NL input planes, over a
// strip of kSsOut columns.  Vertical first: each thread walks down one input
// column and adds its row's NM values to the 11 output rows under way, kept
// in registers (11 input rows per unrolled group, so that every register
// index is a constant); the 11 finished rows go through LDS for the
// horizontal pass, four output columns per item.  Per output about 11 NM
// fused multiply-adds each way and 5 NM 16-byte LDS reads per item: bound by
// vector issue, where 32 x 32 tiles with both passes through LDS read 22 NM
// floats per output.  in(x, y, v): the input values at a pixel of the image;
// maps(v, m): the NM maps' values; out(x, y, o): four outputs from column x.
template <int NM, int NL, class In, class Maps, class Out>
__device__ inline void ss_blur(const SsArgs& a, int X0, int Y0, float (*s_v)[NM][kSsRow], In in,
                               Maps maps, Out out) {
  const int tid = threadIdx.x, x = X0 - kSsHalo + tid;
  const int y1 = min(Y0 + a.rows, a.H);   // end of the output rows
  float acc[kSsTaps][NM], cur[kSsTaps][NL];
  auto load = [&](int g) {
#pragma unroll
    for (int s = 0; s < kSsTaps; ++s) {
      const int y = Y0 - kSsHalo + g * kSsTaps + s;
#pragma unroll
      for (int l = 0; l < NL; ++l) cur[s][l] = 0.0f;
      if (x >= 0 && x < a.W && y >= 0 && y < a.H) in(x, y, cur[s]);
    }
  };
#pragma unroll
  for (int k = 0; k < kSsTaps; ++k)
#pragma unroll
    for (int m = 0; m < NM; ++m) acc[k][m] = 0.0f;
  load(0);
  for (int g = 0; g < a.groups; ++g) {
#pragma unroll
    for (int s = 0; s < kSsTaps; ++s) {
      float v[NM];
      maps(cur[s], v);
      // input row i = 11 g + s is tap i - o of output row o = i - 10 .. i; row
      // o is summed in slot o mod 11, row i entering slot s afresh
#pragma unroll
      for (int k = 0; k < kSsTaps; ++k)
#pragma unroll
        for (int m = 0; m < NM; ++m)
          acc[k][m] = k == s ? a.w[0] * v[m]
                             : fmaf(a.w[(s - k + kSsTaps) % kSsTaps], v[m], acc[k][m]);
#pragma unroll
      for (int m = 0; m < NM; ++m) s_v[s][m][tid] = acc[(s + 1) % kSsTaps][m];
    }
    if (g + 1 < a.groups) load(g + 1);
    __syncthreads();
    for (int it = tid; it < kSsTaps * (kSsOut / 4); it += kSsBlock) {
      const int r = it / (kSsOut / 4), q = it - r * (kSsOut / 4);
      const int o = g * kSsTaps + r - 2 * kSsHalo;   // output row of the strip
      if (o < 0 || Y0 + o >= y1 || X0 + 4 * q >= a.W) continue;
      float b[NM][4];
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        float t[16];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float4 f = *reinterpret_cast<const float4*>(&s_v[r][m][4 * (q + k)]);
          t[4 * k] = f.x; t[4 * k + 1] = f.y; t[4 * k + 2] = f.z; t[4 * k + 3] = f.w;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float u = 0.0f;
#pragma unroll
          for (int j = 0; j < kSsTaps; ++j) u = fmaf(a.w[j], t[c + j], u);
          b[m][c] = u;
        }
      }
      out(X0 + 4 * q, Y0 + o, b);
    }
    __syncthreads();
  }
}

// One pixel's SSIM from five blurred moments of x, y and e = x - y (mu_x, mu_y, E[xy],
// D = mu_e, E[e^2]; s_xy is taken from E[xy] itself, since a difference of
// larger moments would lose it where either image is dark).  With a1 = 2 mu_x
// mu_y + C1, a2 = 2 s_xy + C2, b1 = a1 + D^2 (= mu_x^2 + mu_y^2 + C1), b2 = a2
// + v_e (= s_xx + s_yy + C2, v_e = E[e^2] - D^2), the map's complement is 1 - SSIM = (b1 v_e + D^2 a2) / (b1 b2): no difference of
// nearly equal terms where x and y agree.  MAPS: writes the map's partials
// in (mu_x, E[x^2]) and their combination with E[xy]'s, in the same
// difference form (A, B, C' = C + 2B: A = -2 a2 D (mu_y (mu_x + mu_y) + C1)
// / (b1^2 b2) + 2 a1 (D a2 - mu_y v_e) / (b1 b2^2), B = -SSIM / b2,
// C' = 2 a1 v_e / (b1 b2^2)) to maps [3][planes][H][W].  SUM: the block's sum
// of 1 - SSIM to partial[block].  Twelve 1024 x 1024 planes: 89 us,
// 116 the maps, 119 both in one pass (141 and 165 with 32 x 32 tiles).
// (No contraction beyond the fused operations written, so that every variant
// gives the same bits.)
struct SsPoint {
  float my, mxy, D, ve, a1, a2, b1, b2, inv;
  __device__ SsPoint(float mx, float my_, float exy, float D_, float ee) : my(my_), D(D_) {
#pragma clang fp contract(off)
    const float C1 = 0.01f * 0.01f, C2 = 0.03f * 0.03f;
    mxy = mx + my;
    const float sxy = fmaf(-mx, my, exy);
    ve = fmaf(-D, D, ee);
    a1 = fmaf(2.0f * mx, my, C1);
    a2 = fmaf(2.0f, sxy, C2);
    b1 = fmaf(D, D, a1);
    b2 = a2 + ve;
    inv = 1.0f / (b1 * b2);
  }
  __device__ float loss() const {
#pragma clang fp contract(off)
    return fmaf(b1, ve, D * D * a2) * inv;
  }
  __device__ void maps(float* __restrict__ m, int64_t at, int64_t all) const {
#pragma clang fp contract(off)
    const float C1 = 0.01f * 0.01f;
    const float s = a1 * a2 * inv;
    const float u = -2.0f * a2 * D * fmaf(my, mxy, C1) * inv / b1;
    const float v = 2.0f * a1 * fmaf(D, a2, -(my * ve)) * inv;
    m[at] = u + v / b2;
    m[all + at] = -s / b2;
    m[2 * all + at] = 2.0f * a1 * ve * inv / b2;
  }
};

// The workgroup's sum to partial[its place].
template <int BLOCK>
__device__ inline void ss_block_sum(const SsArgs& a, float sum, float* s_red,
                                    float* __restrict__ partial) {
#pragma unroll
  for (int sh = 32; sh > 0; sh >>= 1) sum += __shfl_xor(sum, sh, 64);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.0f;
    for (int w = 0; w < BLOCK / 64; ++w) t += s_red[w];
    partial[((int64_t)blockIdx.z * a.tiles_y + blockIdx.y) * a.tiles_x + blockIdx.x] = t;
  }
}

template <bool MAPS, bool SUM>
__global__ __launch_bounds__(kSsBlock) void k_ssim(const float* __restrict__ x,
                                                   const float* __restrict__ y, SsArgs a,
                                                   float* __restrict__ maps,
                                                   float* __restrict__ partial) {
  __shared__ __align__(16) float s_v[kSsTaps][5][kSsRow];
  __shared__ float s_red[kSsBlock / 64];
  const int pl = blockIdx.z;
  const int64_t plane = (int64_t)a.W * a.H;
  const float *xp = x + pl * plane, *yp = y + pl * plane;
  float sum = 0.0f;
  ss_blur<5, 2>(
      a, blockIdx.x * kSsOut, blockIdx.y * a.rows, s_v,
      [&](int px, int py, float* v) {
        const int64_t i = (int64_t)py * a.W + px;
        v[0] = xp[i];
        v[1] = yp[i];
      },
      [&](const float* v, float* m) {
        const float e = v[0] - v[1];
        m[0] = v[0];
        m[1] = v[1];
        m[2] = v[0] * v[1];
        m[3] = e;
        m[4] = e * e;
      },
      [&](int px, int py, const float (*o)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (px + c >= a.W) continue;
          const SsPoint v(o[0][c], o[1][c], o[2][c], o[3][c], o[4][c]);
          if (MAPS)
            v.maps(maps, pl * plane + (int64_t)py * a.W + px + c, (int64_t)a.planes * plane);
          if (SUM) sum += v.loss();
        }
      });
  if (SUM) ss_block_sum<kSsBlock>(a, sum, s_red, partial);
}

// d_x += scale (blur(A) + 2 (x - y) blur(B) + y blur(C')), scale =
// -d_loss / N (the partials' adjoint: A + 2 x B + y C with C = C' - 2B).
// Twelve 1024 x 1024 planes: 114 us, 95 written (129 with 32 x 32 tiles; its 350 MB take
// 74 at a copy's rate).
template <bool ADD>   // else written
__global__ __launch_bounds__(kSsBlock) void k_ssim_bwd(const float* __restrict__ x,
                                                       const float* __restrict__ y, SsArgs a,
                                                       const float* __restrict__ maps,
                                                       const float* __restrict__ d_loss,
                                                       float inv_n, float* __restrict__ d_x) {
  __shared__ __align__(16) float s_v[kSsTaps][3][kSsRow];
  const int pl = blockIdx.z;
  const int64_t plane = (int64_t)a.W * a.H;
  const int64_t all = (int64_t)a.planes * plane;
  const float* mp = maps + pl * plane;
  const float scale = -(d_loss ? *d_loss : 1.0f) * inv_n;
  ss_blur<3, 3>(
      a, blockIdx.x * kSsOut, blockIdx.y * a.rows, s_v,
      [&](int px, int py, float* v) {
        const int64_t i = (int64_t)py * a.W + px;
#pragma unroll
        for (int l = 0; l < 3; ++l) v[l] = mp[l * all + i];
      },
      [&](const float* v, float* m) {
#pragma unroll
        for (int l = 0; l < 3; ++l) m[l] = v[l];
      },
      [&](int px, int py, const float (*o)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (px + c >= a.W) continue;
          const int64_t i = pl * plane + (int64_t)py * a.W + px + c;
          const float yi = y[i];
          const float g = o[0][c] + 2.0f * (x[i] - yi) * o[1][c] + yi * o[2][c];
          d_x[i] = ADD ? d_x[i] + scale * g : scale * g;
        }
      });
}

// The same over 32 x 32 tiles, both passes through LDS: every thread of a
// small image's workgroup has work, and one is done in fewer steps (see
// ss_tiles for where).
constexpr int kStTile = 32, kStIn = kStTile + 2 * kSsHalo, kStBlock = 256;

// NM planes' halo tiles (zero outside the image) to LDS.
template <int NM>
__device__ inline void st_stage(const float* const src[NM], const SsArgs& a, int X0, int Y0,
                                float (*in)[kStIn][kStIn + 1]) {
  for (int i = threadIdx.x; i < kStIn * kStIn; i += kStBlock) {
    const int r = i / kStIn, c = i - r * kStIn;
    const int y = Y0 + r - kSsHalo, x = X0 + c - kSsHalo;
    const bool ok = x >= 0 && x < a.W && y >= 0 && y < a.H;
#pragma unroll
    for (int m = 0; m < NM; ++m) in[m][r][c] = ok ? src[m][(int64_t)y * a.W + x] : 0.0f;
  }
  __syncthreads();
}
// Vertical pass: thread (tx, ty) the rows ty + 8 q of column tx.
template <int NM>
__device__ inline void st_column(const SsArgs& a, float (*h)[kStIn][kStTile + 1], int tx, int r,
                                 float o[NM]) {
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < kSsTaps; ++j) s = fmaf(a.w[j], h[m][r + j][tx], s);
    o[m] = s;
  }
}

template <bool MAPS, bool SUM>
__global__ __launch_bounds__(kStBlock) void k_ssim_tile(const float* __restrict__ x,
                                                        const float* __restrict__ y, SsArgs a,
                                                        float* __restrict__ maps,
                                                        float* __restrict__ partial) {
  __shared__ float s_in[2][kStIn][kStIn + 1];
  __shared__ float s_h[5][kStIn][kStTile + 1];
  __shared__ float s_red[kStBlock / 64];
  const int pl = blockIdx.z, X0 = blockIdx.x * kStTile, Y0 = blockIdx.y * kStTile;
  const int64_t plane = (int64_t)a.W * a.H;
  const float* src[2] = {x + pl * plane, y + pl * plane};
  st_stage<2>(src, a, X0, Y0, s_in);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < kStIn; r += 8) {
    float h[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < kSsTaps; ++j) {
      const float w = a.w[j], u = s_in[0][r][tx + j], v = s_in[1][r][tx + j], e = u - v;
      h[0] = fmaf(w, u, h[0]);
      h[1] = fmaf(w, v, h[1]);
      h[2] = fmaf(w, u * v, h[2]);
      h[3] = fmaf(w, e, h[3]);
      h[4] = fmaf(w, e * e, h[4]);
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) s_h[m][r][tx] = h[m];
  }
  __syncthreads();
  float sum = 0.0f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = ty + 8 * q, px = X0 + tx, py = Y0 + r;
    float o[5];
    st_column<5>(a, s_h, tx, r, o);
    if (px >= a.W || py >= a.H) continue;
    const SsPoint v(o[0], o[1], o[2], o[3], o[4]);
    if (MAPS) v.maps(maps, pl * plane + (int64_t)py * a.W + px, (int64_t)a.planes * plane);
    if (SUM) sum += v.loss();
  }
  if (SUM) ss_block_sum<kStBlock>(a, sum, s_red, partial);
}

template <bool ADD>
__global__ __launch_bounds__(kStBlock) void k_ssim_bwd_tile(const float* __restrict__ x,
                                                            const float* __restrict__ y, SsArgs a,
                                                            const float* __restrict__ maps,
                                                            const float* __restrict__ d_loss,
                                                            float inv_n, float* __restrict__ d_x) {
  __shared__ float s_in[3][kStIn][kStIn + 1];
  __shared__ float s_h[3][kStIn][kStTile + 1];
  const int pl = blockIdx.z, X0 = blockIdx.x * kStTile, Y0 = blockIdx.y * kStTile;
  const int64_t plane = (int64_t)a.W * a.H, all = (int64_t)a.planes * plane;
  const float* src[3] = {maps + pl * plane, maps + all + pl * plane, maps + 2 * all + pl * plane};
  st_stage<3>(src, a, X0, Y0, s_in);
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  for (int r = ty; r < kStIn; r += 8)
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      float s = 0.0f;
#pragma unroll
      for (int j = 0; j < kSsTaps; ++j) s = fmaf(a.w[j], s_in[m][r][tx + j], s);
      s_h[m][r][tx] = s;
    }
  __syncthreads();
  const float scale = -(d_loss ? *d_loss : 1.0f) * inv_n;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = ty + 8 * q, px = X0 + tx, py = Y0 + r;
    float o[3];
    st_column<3>(a, s_h, tx, r, o);
    if (px >= a.W || py >= a.H) continue;
    const int64_t i = pl * plane + (int64_t)py * a.W + px;
    const float yi = y[i];
    const float g = o[0] + 2.0f * (x[i] - yi) * o[1] + yi * o[2];
    d_x[i] = ADD ? d_x[i] + scale * g : scale * g;
  }
}

// out[0] = sum(partial) / N (the blocks' sums of 1 - SSIM), in a fixed
// order.
__global__ __launch_bounds__(256) void k_dssim_finish(const float* __restrict__ partial,
                                                      int64_t nb, double inv_n,
                                                      float* __restrict__ out) {
  __shared__ double s[256];
  double acc = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += 256) acc += (double)partial[b];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[0] = (float)(s[0] * inv_n);
}

// Strips of 11 (groups - 1) + 1 rows at most: ten input rows of each are
// halo, so tall ones compute less, short ones fill the chip.  The number of
// groups that gives the fewest passes of `resident` workgroups per compute
// unit over it, times the groups of each (twelve 1024 x 1024 planes: 5 groups
// in two passes for the moments, 90 us against 99 with 7 and 94 with 10; 7 in
// one pass for the gradient, 114 us against 127 with 5 and 118 with 10).
constexpr int kSsResident = 5, kSsResidentBwd = 8;   // by LDS; by registers
bool ss_ok(int planes, int W, int H) {
  return planes >= 1 && W >= 1 && H >= 1 && planes <= 65535 && div_up(H, 32) <= 65535;
}
// Tiles where there are few of them (a strip's workgroup takes as many steps
// however small the image) or the strips' columns would be over a fifth idle:
// loss and adjoint 15 + 30 us with strips and 12 + 24 with tiles for three 512 x
// 512 planes, 16 + 25 and 12 + 14 for 300 of 32 x 32, 46 + 93 and 40 + 71 for 192
// of 128 x 128 (55 % used), but 31 + 64 and 39 + 69 for twelve of 512 x 512, 30 +
// 62 and 47 + 84 for thirty of 1024 x 100 (86 %).
bool ss_tiles(int planes, int W, int H) {
  const int64_t tiles = (int64_t)planes * div_up(W, kStTile) * div_up(H, kStTile);
  return tiles < 2048 || 5 * (int64_t)W < 4 * (int64_t)kSsOut * div_up(W, kSsOut);
}
void ss_args(int planes, int W, int H, int resident, SsArgs* a) {
  a->planes = planes;
  a->W = W;
  a->H = H;
  a->tile = ss_tiles(planes, W, H);
  a->tiles_x = div_up(W, kSsOut);
  const int64_t chip = (int64_t)resident * device_cus();
  int64_t best = INT64_MAX;
  for (int groups = 2; groups <= 12; ++groups) {
    const int strips = div_up(H, kSsTaps * (groups - 1) + 1);
    if (strips > 65535) continue;
    const int64_t cost = (((int64_t)planes * a->tiles_x * strips + chip - 1) / chip) * groups;
    if (cost >= best) continue;
    best = cost;
    a->tiles_y = strips;
    a->rows = div_up(H, strips);
    a->groups = div_up(a->rows + 2 * kSsHalo, kSsTaps);
  }
  if (a->tile) {
    a->tiles_x = div_up(W, kStTile);
    a->tiles_y = div_up(H, kStTile);
  }
  double g[11], s = 0.0;
  for (int j = 0; j < 11; ++j) {
    const double u = j - 5;
    g[j] = std::exp(-u * u / (2.0 * 1.5 * 1.5));
    s += g[j];
  }
  for (int j = 0; j < 11; ++j) a->w[j] = (float)(g[j] / s);
}

template <bool MAPS, bool SUM>
void launch_ssim(const SsArgs& a, const float* x, const float* y, float* maps, float* partial,
                 hipStream_t st) {
  const dim3 grid(a.tiles_x, a.tiles_y, a.planes);
  if (a.tile)
    hipLaunchKernelGGL((k_ssim_tile<MAPS, SUM>), grid, dim3(kStBlock), 0, st, x, y, a, maps, partial);
  else
    hipLaunchKernelGGL((k_ssim<MAPS, SUM>), grid, dim3(kSsBlock), 0, st, x, y, a, maps, partial);
}
template <bool ADD>
void launch_ssim_bwd(const SsArgs& a, const float* x, const float* y, const float* maps,
                     const float* d_loss, float* d_x, hipStream_t st) {
  const dim3 grid(a.tiles_x, a.tiles_y, a.planes);
  const float inv_n = (float)(1.0 / ((double)a.planes * a.W * a.H));
  if (a.tile)
    hipLaunchKernelGGL(k_ssim_bwd_tile<ADD>, grid, dim3(kStBlock), 0, st, x, y, a, maps, d_loss,
                       inv_n, d_x);
  else
    hipLaunchKernelGGL(k_ssim_bwd<ADD>, grid, dim3(kSsBlock), 0, st, x, y, a, maps, d_loss, inv_n,
                       d_x);
}

// -------------------------------------------------------------- regulariser
struct RegArgs {
  int n, nv, W, H;
  int view[VRS_MAX_CROPS], x0[VRS_MAX_CROPS], y0[VRS_MAX_CROPS], S[VRS_MAX_CROPS];
  long long fbase[VRS_MAX_CROPS], ebase[VRS_MAX_CROPS + 1];   // fovea offsets, element prefix
  const int4* place;
  bool wide;   // a crop of 2^32 elements or more
};

// WIDE: 64-bit divisions (as a branch in the one kernel they cost a whole
// objective of four 1024 x 1024 views 8 us).
template <bool WIDE>
__device__ inline void reg_locate(const RegArgs& a, long long e, int& k, int& c, int& yy,
                                  int& xx, int& x0, int& y0) {
  k = 0;
  while (k + 1 < a.n && a.ebase[k + 1] <= e) ++k;
  const long long r = e - a.ebase[k];
  const uint32_t S = (uint32_t)a.S[k];
  if (WIDE) {
    const long long plane = (long long)S * S;
    c = (int)(r / plane);
    const long long q = r - c * plane;
    yy = (int)(q / S);
    xx = (int)(q - (long long)yy * S);
  } else {   // 32-bit divisions
    c = (int)((uint32_t)r / (S * S));
    const uint32_t q = (uint32_t)r - (uint32_t)c * S * S;
    yy = (int)(q / S);
    xx = (int)(q - (uint32_t)yy * S);
  }
  if (a.place) {
    x0 = clamp_origin(a.place[k].x, a.W - a.S[k]);
    y0 = clamp_origin(a.place[k].y, a.H - a.S[k]);
  } else {
    x0 = a.x0[k];
    y0 = a.y0[k];
  }
}

constexpr int kRegBlock = 256, kRegBlocks = 1024;

template <bool WIDE>
__global__ __launch_bounds__(kRegBlock) void k_reg_sums(const float* __restrict__ fovea,
                                                        const float* __restrict__ rgb, RegArgs a,
                                                        double* __restrict__ partial) {
  __shared__ double s_f[kRegBlock / 64], s_p[kRegBlock / 64];
  const long long total = a.ebase[a.n];
  const int64_t plane = (int64_t)a.W * a.H;
  double sf = 0.0, sp = 0.0;
  for (long long e = blockIdx.x * (long long)kRegBlock + threadIdx.x; e < total;
       e += (long long)gridDim.x * kRegBlock) {
    int k, c, yy, xx, x0, y0;
    reg_locate<WIDE>(a, e, k, c, yy, xx, x0, y0);
    const int S = a.S[k];
    sf += (double)fovea[a.fbase[k] + ((long long)c * S + yy) * S + xx];
    sp += (double)rgb[((int64_t)a.view[k] * 3 + c) * plane + (int64_t)(y0 + yy) * a.W + x0 + xx];
  }
#pragma unroll
  for (int sh = 32; sh > 0; sh >>= 1) {
    sf += __shfl_xor(sf, sh, 64);
    sp += __shfl_xor(sp, sh, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    s_f[threadIdx.x >> 6] = sf;
    s_p[threadIdx.x >> 6] = sp;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double f = 0.0, p = 0.0;
    for (int w = 0; w < kRegBlock / 64; ++w) {
      f += s_f[w];
      p += s_p[w];
    }
    partial[2 * blockIdx.x] = f;
    partial[2 * blockIdx.x + 1] = p;
  }
}

__global__ __launch_bounds__(256) void k_reg_finish(const double* __restrict__ partial, int nb,
                                                    double inv_cnt, float* __restrict__ out) {
  __shared__ double s[2][256];
  double f = 0.0, p = 0.0;
  for (int b = threadIdx.x; b < nb; b += 256) {
    f += partial[2 * b];
    p += partial[2 * b + 1];
  }
  s[0][threadIdx.x] = f;
  s[1][threadIdx.x] = p;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      s[0][threadIdx.x] += s[0][threadIdx.x + w];
      s[1][threadIdx.x] += s[1][threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double d = (s[0][0] - s[1][0]) * inv_cnt;
    out[0] = (float)fabs(d);
    out[1] = (float)d;
  }
}

// dF += g, dP -= g over the crops, g = d_r sign(diff) / count.
template <bool WIDE>
__global__ __launch_bounds__(kRegBlock) void k_reg_bwd(RegArgs a, const float* __restrict__ r,
                                                       const float* __restrict__ d_r,
                                                       float inv_cnt, float* __restrict__ d_fovea,
                                                       float* __restrict__ d_rgb) {
  const float diff = r[1];
  const float sg = diff > 0.0f ? 1.0f : (diff < 0.0f ? -1.0f : 0.0f);
  const float g = (d_r ? *d_r : 1.0f) * sg * inv_cnt;
  if (g == 0.0f) return;
  const long long total = a.ebase[a.n];
  const int64_t plane = (int64_t)a.W * a.H;
  for (long long e = blockIdx.x * (long long)kRegBlock + threadIdx.x; e < total;
       e += (long long)gridDim.x * kRegBlock) {
    int k, c, yy, xx, x0, y0;
    reg_locate<WIDE>(a, e, k, c, yy, xx, x0, y0);
    const int S = a.S[k];
    if (d_fovea) d_fovea[a.fbase[k] + ((long long)c * S + yy) * S + xx] += g;
    if (d_rgb)
      atomicAdd(&d_rgb[((int64_t)a.view[k] * 3 + c) * plane + (int64_t)(y0 + yy) * a.W + x0 + xx],
                -g);
  }
}

bool reg_args(int nv, int W, int H, const vrs_crop* crops, int n, const vrs_crop_place* place,
              RegArgs* a) {
  if (nv < 1 || nv > VRS_MAX_VIEWS || W < 1 || H < 1 || n < 1 || n > VRS_MAX_CROPS || !crops)
    return false;
  a->n = n;
  a->nv = nv;
  a->W = W;
  a->H = H;
  a->place = reinterpret_cast<const int4*>(place);
  a->wide = false;
  long long fb = 0;
  a->ebase[0] = 0;
  for (int k = 0; k < n; ++k) {
    const vrs_crop& c = crops[k];
    if (c.view < 0 || c.view >= nv || c.size < 1 || c.size > W || c.size > H) return false;
    if (!place && (c.x0 < 0 || c.y0 < 0 || c.x0 + c.size > W || c.y0 + c.size > H)) return false;
    a->view[k] = c.view;
    a->x0[k] = c.x0;
    a->y0[k] = c.y0;
    a->S[k] = c.size;
    a->fbase[k] = fb;
    if ((3LL * c.size * c.size) >> 32) a->wide = true;
    fb += 3LL * c.size * c.size;
    a->ebase[k + 1] = fb;
  }
  return true;
}

// --------------------------------------------------------------------- Adam
constexpr int kAdamBlock = 256;

__device__ inline void adam1(float& p, float g, float& m, float& v, float b1, float b2, float lr,
                             float ibc1, float ibc2, float eps) {
#pragma clang fp contract(off)
  m = b1 * m + (1.0f - b1) * g;
  v = b2 * v + (1.0f - b2) * (g * g);
  const float mh = m * ibc1, vh = v * ibc2;
  p = p - lr * mh / (sqrtf(vh) + eps);
}

__global__ __launch_bounds__(kAdamBlock) void k_adam(float* __restrict__ p,
                                                     const float* __restrict__ g,
                                                     float* __restrict__ m, float* __restrict__ v,
                                                     int64_t n, float b1, float b2, float lr,
                                                     float ibc1, float ibc2, float eps) {
  const int64_t n4 = n >> 2;
  float4* p4 = reinterpret_cast<float4*>(p);
  const float4* g4 = reinterpret_cast<const float4*>(g);
  float4* m4 = reinterpret_cast<float4*>(m);
  float4* v4 = reinterpret_cast<float4*>(v);
  const int64_t stride = (int64_t)gridDim.x * kAdamBlock;
  for (int64_t i = blockIdx.x * (int64_t)kAdamBlock + threadIdx.x; i < n4; i += stride) {
    float4 pp = p4[i], mm = m4[i], vv = v4[i];
    const float4 gg = g4[i];
    adam1(pp.x, gg.x, mm.x, vv.x, b1, b2, lr, ibc1, ibc2, eps);
    adam1(pp.y, gg.y, mm.y, vv.y, b1, b2, lr, ibc1, ibc2, eps);
    adam1(pp.z, gg.z, mm.z, vv.z, b1, b2, lr, ibc1, ibc2, eps);
    adam1(pp.w, gg.w, mm.w, vv.w, b1, b2, lr, ibc1, ibc2, eps);
    p4[i] = pp;
    m4[i] = mm;
    v4[i] = vv;
  }
  for (int64_t i = 4 * n4 + blockIdx.x * (int64_t)kAdamBlock + threadIdx.x; i < n; i += stride) {
    float pp = p[i], mm = m[i], vv = v[i];
    adam1(pp, g[i], mm, vv, b1, b2, lr, ibc1, ibc2, eps);
    p[i] = pp;
    m[i] = mm;
    v[i] = vv;
  }
}

bool aligned16(const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; }

}  // namespace
}  // namespace vrs

using namespace vrs;

// ------------------------------------------------------------ entry points
extern "C" size_t vrs_tonemap_workspace_size(const vrs_view* views, int n_views, int n_resp) {
  TmArgs a;
  if (!tm_args(views, n_views, n_resp, &a)) return 0;
  return (size_t)n_views * tm_bwd_blocks(a) * (kTmFixed + n_resp) * sizeof(float);
}

extern "C" vrs_status vrs_tonemap(const float* in, const vrs_view* views, int n_views,
                                  const float* params, int n_resp, float* out, void* stream) {
  TmArgs a;
  if (!tm_args(views, n_views, n_resp, &a) || !in || !params || !out) return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(k_tonemap, dim3(tm_blocks(a), n_views), dim3(kTmBlock), 0, st, in, params,
                     a, out);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_tonemap_backward(const float* in, const vrs_view* views, int n_views,
                                           const float* params, int n_resp, const float* d_out,
                                           float* d_in, float* d_params, void* ws,
                                           size_t ws_bytes, void* stream) {
  TmArgs a;
  if (!tm_args(views, n_views, n_resp, &a) || !in || !params || !d_out) return VRS_EINVAL;
  if (d_params && (!ws || ws_bytes < vrs_tonemap_workspace_size(views, n_views, n_resp)))
    return VRS_EINVAL;
  if (!d_in && !d_params) return VRS_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int nb = tm_bwd_blocks(a);
  float* partial = d_params ? static_cast<float*>(ws) : nullptr;
  auto bwd = tm_lanes(n_resp) ? k_tonemap_bwd<true> : k_tonemap_bwd<false>;
  hipLaunchKernelGGL(bwd, dim3(nb, n_views), dim3(kTmBlock), tm_lds(n_resp), st, in, params, a,
                     d_out, d_in, partial);
  VRS_LAUNCH_CHECK();
  if (d_params) {
    hipLaunchKernelGGL(k_reduce_partials, dim3(kTmFixed + n_resp, n_views), dim3(256), 0, st,
                       partial, nb, kTmFixed + n_resp, d_params);
    VRS_LAUNCH_CHECK();
  }
  return VRS_OK;
}

extern "C" size_t vrs_dssim_workspace_size(int planes, int width, int height) {
  if (!ss_ok(planes, width, height)) return 0;
  // the three derivative maps of the adjoint (the forward's block partials
  // are fewer than one map's elements)
  return 3 * (size_t)planes * width * height * sizeof(float);
}

extern "C" vrs_status vrs_dssim(const float* x, const float* y, int planes, int width,
                                int height, float* loss, void* ws, size_t ws_bytes,
                                void* stream) {
  if (!ss_ok(planes, width, height) || !x || !y || !loss || !ws ||
      ws_bytes < vrs_dssim_workspace_size(planes, width, height))
    return VRS_EINVAL;
  SsArgs a;
  ss_args(planes, width, height, kSsResident, &a);
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* partial = static_cast<float*>(ws);
  launch_ssim<false, true>(a, x, y, nullptr, partial, st);
  VRS_LAUNCH_CHECK();
  const int64_t nb = (int64_t)planes * a.tiles_x * a.tiles_y;
  hipLaunchKernelGGL(k_dssim_finish, dim3(1), dim3(256), 0, st, partial, nb,
                     1.0 / ((double)planes * width * height), loss);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_dssim_backward(const float* x, const float* y, int planes, int width,
                                         int height, const float* d_loss, float* d_x, void* ws,
                                         size_t ws_bytes, void* stream) {
  if (!ss_ok(planes, width, height) || !x || !y || !d_x || !ws ||
      ws_bytes < vrs_dssim_workspace_size(planes, width, height))
    return VRS_EINVAL;
  SsArgs a, b;
  ss_args(planes, width, height, kSsResident, &a);
  ss_args(planes, width, height, kSsResidentBwd, &b);
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* maps = static_cast<float*>(ws);
  launch_ssim<true, false>(a, x, y, maps, nullptr, st);
  VRS_LAUNCH_CHECK();
  launch_ssim_bwd<true>(b, x, y, maps, d_loss, d_x, st);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" size_t vrs_dssim_maps_size(int planes, int width, int height) {
  if (!ss_ok(planes, width, height)) return 0;
  SsArgs a;
  ss_args(planes, width, height, kSsResident, &a);
  return vrs_dssim_workspace_size(planes, width, height) +
         (size_t)planes * a.tiles_x * a.tiles_y * sizeof(float);
}

extern "C" vrs_status vrs_dssim_forward_maps(const float* x, const float* y, int planes, int width,
                                             int height, float* loss, void* maps,
                                             size_t maps_bytes, void* stream) {
  if (!ss_ok(planes, width, height) || !x || !y || !loss || !maps ||
      maps_bytes < vrs_dssim_maps_size(planes, width, height))
    return VRS_EINVAL;
  SsArgs a;
  ss_args(planes, width, height, kSsResident, &a);
  hipStream_t st = static_cast<hipStream_t>(stream);
  float* m = static_cast<float*>(maps);
  float* partial = m + 3 * (int64_t)planes * width * height;
  launch_ssim<true, true>(a, x, y, m, partial, st);
  VRS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_dssim_finish, dim3(1), dim3(256), 0, st, partial,
                     (int64_t)planes * a.tiles_x * a.tiles_y,
                     1.0 / ((double)planes * width * height), loss);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_dssim_backward_maps(const float* x, const float* y, int planes, int width,
                                              int height, const void* maps, size_t maps_bytes,
                                              const float* d_loss, float* d_x, void* stream) {
  if (!ss_ok(planes, width, height) || !x || !y || !d_x || !maps ||
      maps_bytes < vrs_dssim_maps_size(planes, width, height))
    return VRS_EINVAL;
  SsArgs b;
  ss_args(planes, width, height, kSsResidentBwd, &b);
  launch_ssim_bwd<false>(b, x, y, static_cast<const float*>(maps), d_loss, d_x,
                         static_cast<hipStream_t>(stream));
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" size_t vrs_regulariser_workspace_size(void) {
  return 2 * sizeof(double) * kRegBlocks;
}

extern "C" vrs_status vrs_regulariser(const float* fovea_rgb, const float* rgb, int n_views,
                                      int width, int height, const vrs_crop* crops, int n_crops,
                                      const vrs_crop_place* place, float* r, void* ws,
                                      size_t ws_bytes, void* stream) {
  RegArgs a;
  if (!reg_args(n_views, width, height, crops, n_crops, place, &a) || !fovea_rgb || !rgb || !r ||
      !ws || ws_bytes < vrs_regulariser_workspace_size())
    return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int nb = std::max(1, std::min(kRegBlocks, div_up(a.ebase[n_crops], kRegBlock)));
  double* partial = static_cast<double*>(ws);
  hipLaunchKernelGGL((a.wide ? k_reg_sums<true> : k_reg_sums<false>), dim3(nb), dim3(kRegBlock), 0,
                     st, fovea_rgb, rgb, a, partial);
  VRS_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_reg_finish, dim3(1), dim3(256), 0, st, partial, nb,
                     1.0 / (double)a.ebase[n_crops], r);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_regulariser_backward(int n_views, int width, int height,
                                               const vrs_crop* crops, int n_crops,
                                               const vrs_crop_place* place, const float* r,
                                               const float* d_r, float* d_fovea, float* d_rgb,
                                               void* stream) {
  RegArgs a;
  if (!reg_args(n_views, width, height, crops, n_crops, place, &a) || !r) return VRS_EINVAL;
  if (!d_fovea && !d_rgb) return VRS_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const int nb = std::max(1, std::min(kRegBlocks, div_up(a.ebase[n_crops], kRegBlock)));
  hipLaunchKernelGGL((a.wide ? k_reg_bwd<true> : k_reg_bwd<false>), dim3(nb), dim3(kRegBlock), 0,
                     st, a, r, d_r,
                     (float)(1.0 / (double)a.ebase[n_crops]), d_fovea, d_rgb);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}

extern "C" vrs_status vrs_adam_step(float* param, const float* grad, float* m, float* v,
                                    int64_t n, int step, float lr, float beta1, float beta2,
                                    float eps, void* stream) {
  if (n < 0 || step < 1 || (n > 0 && (!param || !grad || !m || !v))) return VRS_EINVAL;
  if (!(beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps >= 0.0f))
    return VRS_EINVAL;
  if (!aligned16(param) || !aligned16(grad) || !aligned16(m) || !aligned16(v)) return VRS_EINVAL;
  if (n == 0) return VRS_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const double bc1 = 1.0 - std::pow((double)beta1, step), bc2 = 1.0 - std::pow((double)beta2, step);
  const int blocks = std::max(1, std::min(8192, div_up(std::max<int64_t>(n >> 2, 1), kAdamBlock)));
  hipLaunchKernelGGL(k_adam, dim3(blocks), dim3(kAdamBlock), 0, st, param, grad, m, v, n, beta1,
                     beta2, lr, (float)(1.0 / bc1), (float)(1.0 / bc2), eps);
  VRS_LAUNCH_CHECK();
  return VRS_OK;
}
