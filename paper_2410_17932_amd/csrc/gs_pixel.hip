// Periphery in per-pixel order (Sec. 3.2: Gaussian contributions sorted per
// pixel instead of per primitive, the sorting of Radl and Steiner et al. that
// removes popping).  The depth of Gaussian g at pixel p is the camera depth
// z* of the maximum of g's 3D density along the ray through p's centre:
// with the camera-space mean mu, camera-space precision M and the ray
// direction d = (u, v, 1), z* = (d^T M mu) / (d^T M d).  Each pixel blends its
// Gaussians in (z*, index) order, and Eq. 1 accumulates z*.
//
// The exact per-pixel order without per-pixel lists:
//   k_gs_pixdepth   per (view, Gaussian): the key's coefficients in single
//                   precision (the order decision, in a documented operation
//                   order) and a lower bound of the key over the Gaussian's
//                   rectangle, which replaces the depth-sort key (only an
//                   initial order: the tile lists are sorted again)
//   k_gs_tile_zsort per tile: bound words for the list positions (see
//                   zs_word), the first kZsPrefix records sorted by z_t, a
//                   rigorous lower bound of the single-precision key over
//                   the tile's pixels
//   k_gs_blend_px   one lane per pixel keeps a sorted window of its pending
//                   contributions (key and list position).  A pending entry
//                   whose key is below every later record's least key over
//                   the 8x8 sub-tile precedes all of them and is blended.  At
//                   tile 8 that bound is the current position's bound word;
//                   with several sub-tiles, per staged batch, a suffix minimum
//                   of exact sub-tile minima (one wave minimum per record),
//                   closed by the bound word of the next batch's first
//                   position.  A pixel whose window has no room for the next
//                   contributions has its order unresolved: it is queued
//   k_gs_blend_px_fix  one wave per queued pixel redoes it exactly, in
//                   rounds of streaming selection of the least keys above
//                   the last blended one (scans cut off by the bound words)
// The adjoint is not provided for this order.
#include <type_traits>

#include "gs_layout.h"

namespace vrs {

constexpr int kPxWindow = 32;   // pending contributions per pixel
constexpr int kPxNew = 16;      // contributions taken in at a time

__device__ inline void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// order-preserving unsigned image of a float, and back
__device__ inline uint32_t f2ord(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float ord2f(uint32_t u) {
  return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

__device__ inline float dot3f(float a0, float a1, float a2, float b0, float b1, float b2) {
#pragma clang fp contract(off)
  float s = a0 * b0;
  s = s + a1 * b1;
  return s + a2 * b2;
}

// Key coefficients (m00, 2 m01, 2 m02, m11, 2 m12, m22, b0, b1, b2), b = M mu,
// in single precision: Sigma^-1 by cofactors over ((s00 c00 + s01 c01) +
// s02 c02), Q = R Sigma^-1, M_ij = Q_i . R_j, b_i = M_i . mu.  A non-positive
// or non-finite determinant gives the mean depth at every pixel.
__device__ inline void pix_coef32(const KView& cv, const float t[3], const float* s, float* k) {
#pragma clang fp contract(off)
  const float c00 = s[3] * s[5] - s[4] * s[4], c01 = s[2] * s[4] - s[1] * s[5];
  const float c02 = s[1] * s[4] - s[2] * s[3], c11 = s[0] * s[5] - s[2] * s[2];
  const float c12 = s[1] * s[2] - s[0] * s[4], c22 = s[0] * s[3] - s[1] * s[1];
  float det = s[0] * c00;
  det = det + s[1] * c01;
  det = det + s[2] * c02;
  if (!(det > 0.0f) || !isfinite(det)) {
    for (int q = 0; q < 9; ++q) k[q] = 0.0f;
    k[5] = 1.0f;
    k[8] = t[2];
    return;
  }
  const float id = 1.0f / det;
  const float P[3][3] = {{c00 * id, c01 * id, c02 * id},
                         {c01 * id, c11 * id, c12 * id},
                         {c02 * id, c12 * id, c22 * id}};
  float Q[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int q = 0; q < 3; ++q)
      Q[a][q] = dot3f(cv.R[3 * a], cv.R[3 * a + 1], cv.R[3 * a + 2], P[0][q], P[1][q], P[2][q]);
  float M[3][3];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b)
      M[a][b] = dot3f(Q[a][0], Q[a][1], Q[a][2], cv.R[3 * b], cv.R[3 * b + 1], cv.R[3 * b + 2]);
  k[0] = M[0][0];
  k[1] = 2.0f * M[0][1];
  k[2] = 2.0f * M[0][2];
  k[3] = M[1][1];
  k[4] = 2.0f * M[1][2];
  k[5] = M[2][2];
  k[6] = dot3f(M[0][0], M[0][1], M[0][2], t[0], t[1], t[2]);
  k[7] = dot3f(M[0][1], M[1][1], M[1][2], t[0], t[1], t[2]);
  k[8] = dot3f(M[0][2], M[1][2], M[2][2], t[0], t[1], t[2]);
}

// Ray coordinates of a pixel-centre coordinate: ((x + 0.5) - c) / f.
__device__ inline float pix_ray(int x, float c, float f) {
#pragma clang fp contract(off)
  return (((float)x + 0.5f) - c) / f;
}

// Numerator and denominator of the key at ray coordinates (u, v), with the
// coefficients staged as q0 = (m00, 2m01, 2m02, m11), q1 = (2m12, m22, b0,
// b1), q2 = (b2, z_lo, -, -) with z_lo the bound below over the Gaussian's
// whole rectangle.
__device__ inline void pix_numden(const float4& q0, const float4& q1, const float4& q2, float u,
                                  float v, float& num, float& den) {
#pragma clang fp contract(off)
  num = q1.z * u;
  num = num + q1.w * v;
  num = num + q2.x;
  float a = q0.x * u;
  a = a + q0.y * v;
  a = a + q0.z;
  float b = q0.w * v;
  b = b + q1.x;
  den = a * u;
  den = den + b * v;
  den = den + q1.y;
}

__device__ inline uint32_t pix_key_bits(const float4& q0, const float4& q1, const float4& q2,
                                        float u, float v) {
  float num, den;
  pix_numden(q0, q1, q2, u, v, num, den);
  return f2ord(num / den);
}

// A lower bound of the single-precision key over every pixel centre of the
// box [x0, x1] x [y0, y1] (-inf where none is proven).
//   The exact numerator N is linear in the ray coordinates (u, v) and the
//   exact denominator D a quadratic, convex when its 2x2 part is positive
//   definite (checked with a margin).  The evaluation order of the key
//   rounds N by at most An = 8 eps sum|terms| and D by at most Bd = 16 eps
//   sum|terms| (eps = 2^-24; three and six roundings deep), the sums taken
//   at the largest |u| and |v| of the box, so wherever N - An > 0 and
//   D - Bd > 0 the key is at least f = (N - An) / (D + Bd) (1 - eps).  For
//   c > 0, (N - An) - c (D + Bd) is concave, so its least value over the box
//   is at a corner: f is least at a corner, and the corners are pixel
//   centres.  Positivity: N's least value is at a corner; D is at least its
//   tangent plane at the (u0, v0) corner, least at one of the box's ends.  Corner values are computed with
//   2 An and 2 Bd to cover their own rounding, and the result is lowered by
//   2^-20 of itself, which covers the last few roundings (the hardware
//   reciprocal's among them: together under 4 units of 2^-24).  Ray coordinates
//   round monotonically, so every pixel's (u, v) lies in the corners' box.
// (No rounding here is part of a decision, so the terms are grouped per
// corner coordinate and fused: at most as many roundings as above, each of a
// sum of the same terms.)
__device__ inline float pix_box_bound_uv(const float4& q0, const float4& q1, const float4& q2,
                                         float u0, float u1, float v0, float v1) {
  const float m00 = q0.x, t01 = q0.y, t02 = q0.z, m11 = q0.w, t12 = q1.x, m22 = q1.y;
  const float pd = m00 * m11, od = 0.25f * t01 * t01;
  bool ok = m00 > 0.0f && m11 > 0.0f && pd > od * (1.0f + 0x1p-20f) && pd < INFINITY;
  const float U = fmaxf(fabsf(u0), fabsf(u1)), V = fmaxf(fabsf(v0), fabsf(v1));
  const float nabs = fmaf(fabsf(q1.z), U, fmaf(fabsf(q1.w), V, fabsf(q2.x)));
  const float au = fmaf(fabsf(t01), V, fabsf(t02)), av = fmaf(fabsf(m11), V, fabsf(t12));
  const float dabs = fmaf(fmaf(m00, U, au), U, fmaf(av, V, fabsf(m22)));
  const float An2 = 0x1p-20f * nabs, Bd2 = 0x1p-19f * dabs;   // 2 An, 2 Bd
  // corners
  const float nu0 = q1.z * u0, nu1 = q1.z * u1;
  const float nv0 = fmaf(q1.w, v0, q2.x) - An2, nv1 = fmaf(q1.w, v1, q2.x) - An2;
  const float du0 = fmaf(m00, u0, t02) * u0, du1 = fmaf(m00, u1, t02) * u1;
  const float dv0 = fmaf(fmaf(m11, v0, t12), v0, m22), dv1 = fmaf(fmaf(m11, v1, t12), v1, m22);
  const float x0 = t01 * u0, x1 = t01 * u1;
  const float d00 = fmaf(x0, v0, du0 + dv0);
  const float n00 = nu0 + nv0, n01 = nu0 + nv1, n10 = nu1 + nv0, n11 = nu1 + nv1;
  ok = ok && fminf(fminf(n00, n01), fminf(n10, n11)) > 0.0f;
  // tangent plane of D at (u0, v0) over the box
  const float du = (u1 - u0) * (1.0f + 0x1p-20f), dv = (v1 - v0) * (1.0f + 0x1p-20f);
  const float gu = fmaf(2.0f * m00, u0, fmaf(t01, v0, t02));
  const float gv = fmaf(2.0f * m11, v0, fmaf(t01, u0, t12));
  const float dlb = d00 + fminf(gu * du, 0.0f) + fminf(gv * dv, 0.0f);
  const float dlb_abs = fmaf(fmaf(2.0f * m00, U, au), fabsf(du),
                             fmaf(fmaf(fabsf(t01), U, av + fabsf(m11) * V), fabsf(dv), dabs));
  ok = ok && fmaf(-0x1p-20f, dlb_abs, dlb) > Bd2 && dlb_abs < INFINITY;
  auto at = [&](float nn, float den) { return nn * __builtin_amdgcn_rcpf(den + Bd2); };
  const float z = fminf(fminf(at(n00, d00), at(n01, fmaf(x0, v1, du0 + dv1))),
                        fminf(at(n10, fmaf(x1, v0, du1 + dv0)), at(n11, fmaf(x1, v1, du1 + dv1))));
  return ok && z < INFINITY ? z - z * 0x1p-20f : -INFINITY;
}

__device__ inline float pix_box_bound(const float4& q0, const float4& q1, const float4& q2,
                                      const KView& cv, int x0, int x1, int y0, int y1) {
  return pix_box_bound_uv(q0, q1, q2, pix_ray(x0, cv.cx, cv.fx), pix_ray(x1, cv.cx, cv.fx),
                          pix_ray(y0, cv.cy, cv.fy), pix_ray(y1, cv.cy, cv.fy));
}

// Coefficients and the sort key of every (view, Gaussian) entry the
// preprocess kept (its depth key is replaced; culled entries keep theirs):
// z_lo, the bound above over the Gaussian's whole rectangle, so that every
// tile list comes out of the binning in z_lo order.  Thread 0 also clears
// the count of pixels queued for the exact pass.
__global__ __launch_bounds__(256) void k_gs_pixdepth(const float* __restrict__ mean,
                                                     const float* __restrict__ cov, int64_t n,
                                                     KViews views,
                                                     const float4* __restrict__ rec,
                                                     uint32_t* __restrict__ dkey,
                                                     float4* __restrict__ pcoef,
                                                     uint32_t* __restrict__ fix_count) {
  const int64_t vn = n * views.n;
  if (blockIdx.x == 0 && threadIdx.x == 0) *fix_count = 0u;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < vn;
       e += (int64_t)gridDim.x * blockDim.x) {
    if (dkey[e] == 0xffffffffu) {   // culled by the preprocess
      pcoef[kPcStride * e] = pcoef[kPcStride * e + 1] = pcoef[kPcStride * e + 2] = make_float4(0, 0, 0, 0);
      continue;
    }
    const int v = (int)(e / n);
    const int64_t i = e - (int64_t)v * n;
    const KView& cv = views.v[v];
    float t[3];
    {
#pragma clang fp contract(off)
      const float mx = mean[i], my = mean[n + i], mz = mean[2 * n + i];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        float p = cv.R[3 * a + 0] * mx;
        float q = cv.R[3 * a + 1] * my;
        float s = p + q;
        float r = cv.R[3 * a + 2] * mz;
        s = s + r;
        t[a] = s + cv.t[a];
      }
    }
    float s6[6], k[9];
#pragma unroll
    for (int q = 0; q < 6; ++q) s6[q] = cov[q * n + i];
    pix_coef32(cv, t, s6, k);
    const float4 q0 = make_float4(k[0], k[1], k[2], k[3]);
    const float4 q1 = make_float4(k[4], k[5], k[6], k[7]);
    const float4 r2 = rec[3 * e + 2];
    const uint32_t lo = __float_as_uint(r2.z), hi = __float_as_uint(r2.w);
    const float zlo = pix_box_bound(q0, q1, make_float4(k[8], 0.0f, 0.0f, 0.0f), cv,
                                    (int)(lo & 0xffffu), (int)(hi & 0xffffu), (int)(lo >> 16),
                                    (int)(hi >> 16));
    pcoef[kPcStride * e] = q0;
    pcoef[kPcStride * e + 1] = q1;
    pcoef[kPcStride * e + 2] = make_float4(k[8], zlo, 0.0f, 0.0f);
    dkey[e] = f2ord(zlo);
  }
}

// ---------------------------------------------------------------- tile sort
// Bound words.  Every list position j gets w(j) = beta(j) << 32 | index with
// beta non-decreasing along the list and every key of every record at
// positions >= j, at every pixel of the tile in its rectangle, at least
// beta(j) (order-preserving bits throughout).  The first kZsPrefix records
// (or all) are sorted by z_t, the bound over the tile's pixel box: beta =
// min(z_t, z_lo of the first record after the prefix).  After the prefix the list
// keeps its z_lo order and beta = z_lo.  Blending stops long before most
// lists end, so only the prefix is sorted; a pixel that reads past it still
// gets valid, if looser, bounds.
constexpr int kZsBlock = 256, kZsPrefix = 4096, kZsSlotBits = 12;
constexpr int kZsPer = kZsPrefix / kZsBlock, kZsBuckets = 1024, kZsSmall = 128, kZsRank = 512;
static_assert(kZsPrefix == 1 << kZsSlotBits, "one slot per prefix position");

__device__ inline uint64_t zs_word(const uint64_t* __restrict__ tkey,
                                   const uint32_t* __restrict__ ids,
                                   const float4* __restrict__ pcoef, int64_t vbase, uint32_t begin,
                                   uint32_t j) {
  if (j - begin < (uint32_t)kZsPrefix) return tkey[j];
  const uint32_t id = ids[j];
  return ((uint64_t)f2ord(pcoef[kPcStride * (vbase + id) + 2].y) << 32) | id;
}

// One workgroup per tile: bounds, then a bucket sort in LDS (counts, scan,
// placing, ranks inside the buckets); short lists are ranked by comparison.
// Bound by the gather of the coefficients (48 B a record): stereo 2016 x 2240,
// 500k Gaussians, tile 8, 137M prefix records, 3.38 ms with three loads per
// record and lane and a bitonic sort, 1.93 now.
__global__ __launch_bounds__(kZsBlock) void k_gs_tile_zsort(
    const uint32_t* __restrict__ ids, const float4* __restrict__ pcoef, int64_t n, KViews views,
    int tile, int64_t tiles_x, int64_t tiles_per_view, const uint2* __restrict__ ranges,
    uint64_t* __restrict__ out) {
  __shared__ uint32_t s_key[kZsPrefix];   // z_t bits rounded down to 20 | prefix slot
  __shared__ uint32_t s_cnt[kZsBuckets];
  __shared__ float4 s_stage[kZsBlock / 64][64 * 3];
  __shared__ uint32_t s_lo[kZsBlock / 64], s_hi[kZsBlock / 64];
  const int64_t tglob = blockIdx.x;
  const uint2 rg = ranges[tglob];
  const uint32_t begin = rg.x;
  const int len = (int)(rg.y - rg.x);
  if (len <= 0) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int v = (int)(tglob / tiles_per_view);
  const int64_t tl = tglob - (int64_t)v * tiles_per_view;
  const int ty = (int)(tl / tiles_x), tx = (int)(tl - (int64_t)ty * tiles_x);
  const KView& cv = views.v[v];
  const int X0 = tx * tile, Y0 = ty * tile;
  const int X1 = min(X0 + tile, cv.W) - 1, Y1 = min(Y0 + tile, cv.H) - 1;
  const float u0 = pix_ray(X0, cv.cx, cv.fx), u1 = pix_ray(X1, cv.cx, cv.fx);
  const float v0 = pix_ray(Y0, cv.cy, cv.fy), v1 = pix_ray(Y1, cv.cy, cv.fy);
  const int64_t vbase = (int64_t)v * n;
  const int m = min(len, kZsPrefix);
  uint32_t cap = 0xffffffffu;   // z_lo of the first record after the prefix
  if (len > m) cap = f2ord(pcoef[kPcStride * (vbase + ids[begin + m]) + 2].y);
  const bool small = m <= kZsSmall;
  if (!small)
    for (int b = tid; b < kZsBuckets; b += kZsBlock) s_cnt[b] = 0u;
  // every record's word, kZsPer per thread; the range of the finite bounds.
  // Four lanes fetch a record's line (one request, where a lane's three
  // 16-byte loads were three), 16 records per instruction, and hand it over
  // through LDS.
  constexpr uint32_t kSlot = (1u << kZsSlotBits) - 1u;
  const uint32_t none = f2ord(-INFINITY) & ~kSlot;
  uint32_t w[kZsPer];
  uint32_t lo = 0xffffffffu, hi = 0u;
  float4* st = s_stage[wave];
#pragma unroll
  for (int r = 0; r < kZsPer; ++r) {
    if (r * kZsBlock >= m) break;   // uniform
    const int i = tid + r * kZsBlock;
    const int id = (int)ids[begin + min(i, m - 1)];
    float4 part[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int from = __shfl(id, q * 16 + (lane >> 2), 64);
      part[q] = pcoef[kPcStride * (vbase + from) + (lane & 3)];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((lane & 3) < 3) st[(q * 16 + (lane >> 2)) * 3 + (lane & 3)] = part[q];
    wave_sync_lds();
    const float4 c0 = st[lane * 3], c1 = st[lane * 3 + 1], c2 = st[lane * 3 + 2];
    wave_sync_lds();
    const uint32_t z = f2ord(pix_box_bound_uv(c0, c1, c2, u0, u1, v0, v1)) & ~kSlot;
    w[r] = z | (uint32_t)i;
    if (i < m && z != none) {
      lo = min(lo, z);
      hi = max(hi, z);
    }
  }
  if (small) {
    if (tid < m) s_key[tid] = w[0];
    __syncthreads();
    if (tid < m) {
      int rank = 0;
      for (int j = 0; j < m; ++j) rank += s_key[j] < w[0] ? 1 : 0;
      out[begin + rank] = ((uint64_t)min(w[0] & ~kSlot, cap) << 32) | ids[begin + tid];
    }
    return;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
  }
  if (lane == 0) {
    s_lo[wave] = lo;
    s_hi[wave] = hi;
  }
  __syncthreads();
  lo = min(min(s_lo[0], s_lo[1]), min(s_lo[2], s_lo[3]));
  hi = max(max(s_hi[0], s_hi[1]), max(s_hi[2], s_hi[3]));
  // bucket of a bound, monotone: 0 for no bound, the others by value
  const float zlo = ord2f(lo), zhi = ord2f(hi);
  const float scale = hi > lo ? (float)(kZsBuckets - 2) / (zhi - zlo) : 0.0f;
  auto bucket = [&](uint32_t word) {
    const uint32_t z = word & ~kSlot;
    return z == none ? 0 : 1 + min((int)((ord2f(z) - zlo) * scale), kZsBuckets - 2);
  };
#pragma unroll
  for (int r = 0; r < kZsPer; ++r)
    if (tid + r * kZsBlock < m) atomicAdd(&s_cnt[bucket(w[r])], 1u);
  __syncthreads();
  // exclusive scan of the counts, consecutive buckets per thread
  {
    constexpr int PER = kZsBuckets / kZsBlock;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      c[q] = s_cnt[tid * PER + q];
      sum += c[q];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = (uint32_t)__shfl_up((int)inc, o, 64);
      if (lane >= o) inc += t;
    }
    if (lane == 63) s_lo[wave] = inc;
    __syncthreads();
    uint32_t base = inc - sum;
    for (int q = 0; q < wave; ++q) base += s_lo[q];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      s_cnt[tid * PER + q] = base;
      base += c[q];
    }
  }
  __syncthreads();
  // into bucket order (the cursors end at the buckets' ends), then each record
  // to its rank in its bucket
#pragma unroll
  for (int r = 0; r < kZsPer; ++r)
    if (tid + r * kZsBlock < m) s_key[atomicAdd(&s_cnt[bucket(w[r])], 1u)] = w[r];
  __syncthreads();
  for (int p = tid; p < m; p += kZsBlock) {
    const uint32_t word = s_key[p];
    const int b = bucket(word);
    const int first = b ? (int)s_cnt[b - 1] : 0, last = (int)s_cnt[b];
    // (records without a bound, and buckets of very many, stay as they are:
    // such a bucket's records share its least bound)
    int at = p;
    uint32_t beta = word & ~kSlot;
    if (b > 0 && last - first <= kZsRank) {
      at = first;
      for (int q = first; q < last; ++q) at += s_key[q] < word ? 1 : 0;
    } else if (b > 0) {
      for (int q = first; q < last; ++q) beta = min(beta, s_key[q] & ~kSlot);
    }
    out[begin + at] = ((uint64_t)min(beta, cap) << 32) | ids[begin + (word & kSlot)];
  }
}

// A lane's pending contributions in registers: 64-bit words (key bits << 32 |
// list position), ascending, empty slots at the end.  Only finite keys other
// than zero enter, so a word read as a double is finite and orders by its key
// (a float's high bits order as the float does in a double too, of either
// sign; equal keys stand side by side), and a comparator is one v_min_f64 and
// one v_max_f64; empty slots hold +infinity (above every such word).
constexpr uint32_t kPxEmptyHi = 0x7ff00000u;
__device__ inline double px_word(uint32_t hi, uint32_t lo) {
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline uint32_t px_hi(double d) { return (uint32_t)(__builtin_bit_cast(uint64_t, d) >> 32); }
__device__ inline uint32_t px_lo(double d) { return (uint32_t)__builtin_bit_cast(uint64_t, d); }
__device__ inline void px_comp(double& a, double& b) {
  double lo, hi;
  asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(a), "v"(b));
  asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(a), "v"(b));
  a = lo;
  b = hi;
}
// N words (a power of two) into ascending order: odd-even merge sort
template <int N>
__device__ __attribute__((always_inline)) inline void px_sort(double* k) {
#pragma unroll
  for (int p = 1; p < N; p <<= 1)
#pragma unroll
    for (int d = p; d >= 1; d >>= 1)
#pragma unroll
      for (int j = d % p; j + d < N; j += 2 * d)
#pragma unroll
        for (int i = 0; i < d; ++i)
          if (i + j + d < N && (i + j) / (2 * p) == (i + j + d) / (2 * p))
            px_comp(k[i + j], k[i + j + d]);
}
// bitonic sequence of N words into ascending order
template <int N>
__device__ __attribute__((always_inline)) inline void px_merge(double* k) {
#pragma unroll
  for (int d = N / 2; d > 0; d >>= 1)
#pragma unroll
    for (int i = 0; i < N; ++i)
      if (!(i & d)) px_comp(k[i], k[i + d]);
}

// f(0), f(1), ... f(N - 1) with compile-time indices while f returns true (a
// loop with an exit is not unrolled, and a run-time index would put the
// window in scratch memory).
template <int I, int N, class F>
__device__ __attribute__((always_inline)) inline void static_while(F&& f) {
  if constexpr (I < N)
    if (f(std::integral_constant<int, I>{})) static_while<I + 1, N>(f);
}

template <int TILE>
struct PxCfg {
  static constexpr int NQ = TILE / 8;     // 8x8 sub-tiles per side, one wave each
  static constexpr int NW = NQ * NQ;
  static constexpr int BLOCK = 64 * NW;
  // records kept in LDS by list position, for the contributions' release: a
  // pixel whose oldest pending one would be overwritten is redone exactly
  // (at 256 and tile 8 some 400 of 9M pixels, 9 KB; at tile 16 a batch is
  // 256 records and lists are walked further: 1024)
  static constexpr int RING = TILE == 8 ? 256 : 1024;
};

// One workgroup per tile in the longest-first schedule, one wave per 8x8
// sub-tile, one pixel per lane.  Records are staged in batches with a ballot
// per sub-tile of those whose contributing ellipse may reach it.  A pixel's
// contributions are collected in LDS, unsorted; when one lane has kPxNew or no
// room for more (and at each batch's end) every lane sorts its own, merges them into its window
// (both networks of comparators on registers, every lane busy), blends the
// entries below the current bound in order and closes the gap with one more
// merge.  Alpha and colour are evaluated again from the record at release, so
// a window entry is one 64-bit word.  Inserting each contribution on its own
// moved the whole window (four words an entry) once per record in which any
// lane had one, and again for each release: 8.6 ms at 500k Gaussians, stereo
// 2016 x 2240, tile 8, against 3.0 here.
template <int TILE>
__global__ __launch_bounds__(PxCfg<TILE>::BLOCK) void k_gs_blend_px(
    const uint32_t* __restrict__ order, const uint64_t* __restrict__ tkey,
    const uint32_t* __restrict__ ids, const float4* __restrict__ rec, const float4* __restrict__ pcoef, int64_t n, KViews views,
    GsOpt o, int64_t tiles_x, int64_t tiles_per_view, const uint2* __restrict__ ranges,
    float* __restrict__ out_rgb, float* __restrict__ out_depth, float* __restrict__ out_t,
    int32_t* __restrict__ out_n, uint32_t* __restrict__ fix_list,
    uint32_t* __restrict__ fix_count) {
  using Cfg = PxCfg<TILE>;
  constexpr int BLOCK = Cfg::BLOCK, NW = Cfg::NW, NQ = Cfg::NQ, RING = Cfg::RING;
  constexpr int K = kPxWindow, B = kPxNew;
  static_assert(RING % BLOCK == 0 && BLOCK <= 256, "batches fill whole ring slots");
  // the ring: (px, py, A', B'), (C', opacity, r, g), b by position mod RING
  __shared__ float4 s_a[RING], s_b[RING];
  __shared__ float s_c[RING];
  // the batch: rectangles and key coefficients
  __shared__ uint2 s_rect[BLOCK];
  __shared__ float4 s_q0[BLOCK], s_q1[BLOCK];
  __shared__ float s_q2[BLOCK];
  __shared__ uint64_t s_mask[NW][NW];
  __shared__ uint32_t s_beta[BLOCK];         // per record: its position's bound word
  __shared__ uint32_t s_bound[NW > 1 ? NW : 1][NW > 1 ? BLOCK : 1];   // per sub-tile and record: release bound
  // per lane: its new contributions' keys and places in the batch
  __shared__ float s_newz[NW][B][64];
  __shared__ uint8_t s_newk[NW][B][64];
  const int64_t tglob = order[blockIdx.x];
  const int v = (int)(tglob / tiles_per_view);
  const int64_t tl = tglob - (int64_t)v * tiles_per_view;
  const int ty = (int)(tl / tiles_x), tx = (int)(tl - (int64_t)ty * tiles_x);
  const KView& cv = views.v[v];
  const int W = cv.W, H = cv.H;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int px = tx * TILE + (wave % NQ) * 8 + (lane & 7);
  const int py = ty * TILE + (wave / NQ) * 8 + (lane >> 3);
  const float xc = (float)px + 0.5f, yc = (float)py + 0.5f;
  const float ur = pix_ray(px, cv.cx, cv.fx), vr = pix_ray(py, cv.cy, cv.fy);
  const float aclamp = o.aclamp, amin = o.amin, tmin = o.tmin, inv_amin = 1.0f / amin;
  bool alive = px < W && py < H;
  bool inexact = false;
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, D = 0.0f;
  int cnt = 0;
  const double empty = px_word(kPxEmptyHi, 0u);
  double win[K];
#pragma unroll
  for (int q = 0; q < K; ++q) win[q] = empty;
  int nwin = 0, nnew = 0;   // the lane's entries in the window and in s_new
  const uint2 rg = ranges[tglob];
  const uint32_t begin = rg.x, end = rg.y;
  // Gaussian index at a list position
  auto tkey_id = [&](uint32_t pos) {
    return (uint32_t)zs_word(tkey, ids, pcoef, (int64_t)v * n, begin, begin + pos);
  };
  for (uint32_t b0 = begin; b0 < end; b0 += BLOCK) {
    // this batch's records overwrite the ring slots of positions b0 - RING
    // onwards: a pixel still holding one of those cannot be finished here
    if (b0 - begin + BLOCK > (uint32_t)RING) {
      uint32_t oldest = ~0u;
#pragma unroll
      for (int q = 0; q < K; ++q)
        oldest = px_hi(win[q]) != kPxEmptyHi ? min(oldest, px_lo(win[q])) : oldest;
      if (alive && nwin > 0 && oldest + RING < (b0 - begin) + BLOCK) {
        inexact = true;
        alive = false;
      }
    }
    if (__syncthreads_count(alive) == 0) break;
    const uint32_t jr = b0 + tid;
    const bool has = jr < end;
    int x0 = 1, x1 = 0, y0 = 1, y1 = 0;
    float cx = 0.0f, cy = 0.0f, ga = 1.0f, gb = 0.0f, gc = 1.0f, thr = -1.0f;
    if (has) {
      const uint64_t wd = zs_word(tkey, ids, pcoef, (int64_t)v * n, begin, jr);
      const uint32_t id = (uint32_t)wd;
      s_beta[tid] = (uint32_t)(wd >> 32);
      const int64_t e = (int64_t)v * n + (id < (uint64_t)n ? id : 0);
      float4 a, b, c;
      gs_stage(rec, e, a, b, c);
      const uint32_t slot = (jr - begin) & (RING - 1);
      s_a[slot] = a;
      s_b[slot] = make_float4(b.x, b.y, c.x, c.y);
      s_c[slot] = c.z;
      const uint32_t lo = __float_as_uint(b.z), hi = __float_as_uint(b.w);
      s_rect[tid] = make_uint2(lo, hi);
      s_q0[tid] = pcoef[kPcStride * e];
      s_q1[tid] = pcoef[kPcStride * e + 1];
      s_q2[tid] = pcoef[kPcStride * e + 2].x;
      x0 = (int)(lo & 0xffffu); y0 = (int)(lo >> 16);
      x1 = (int)(hi & 0xffffu); y1 = (int)(hi >> 16);
      cx = a.x; cy = a.y;
      ga = -a.z; gb = -a.w; gc = -b.x;
      thr = b.y >= amin ? __builtin_amdgcn_logf(b.y * inv_amin) * 1.001f + 1.0e-3f : -1.0f;
      if (!(ga > 0.0f && gc > 0.0f)) thr = 3.0e38f;
    }
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int qx0 = tx * TILE + (w % NQ) * 8, qy0 = ty * TILE + (w / NQ) * 8;
      const int xlo = max(x0, qx0), xhi = min(x1, qx0 + 7);
      const int ylo = max(y0, qy0), yhi = min(y1, qy0 + 7);
      bool hit = has && xlo <= xhi && ylo <= yhi;
      if (hit) {
        // as in the per-primitive blend: out of reach only where every
        // pixel's own test would fail
        const float g = box_min_quadratic(
            ga, gb, gc, 0.5f * __builtin_amdgcn_rcpf(ga), 0.5f * __builtin_amdgcn_rcpf(gc),
            cx - ((float)xhi + 0.5f), cx - ((float)xlo + 0.5f), cy - ((float)yhi + 0.5f),
            cy - ((float)ylo + 0.5f));
        hit = !(g > thr);
      }
      const uint64_t m = __ballot(hit);
      if (lane == 0) s_mask[w][wave] = m;
    }
    __syncthreads();
    if (!__ballot(alive)) continue;
    const uint32_t slot0 = (b0 - begin) & (RING - 1);
    // Release bounds.  One sub-tile: the bound word of record k's position.
    // Several: walking this batch's records backwards, before record k every
    // later key at any pixel of the sub-tile is at least the least key of
    // records k.. of the batch over the sub-tile's pixels (a wave minimum of
    // exact keys), and at least the bound word of the next batch's first
    // position.
    if constexpr (NW > 1) {
      uint32_t bound =
          b0 + BLOCK < end
              ? (uint32_t)(zs_word(tkey, ids, pcoef, (int64_t)v * n, begin, b0 + BLOCK) >> 32)
              : 0xffffffffu;
      for (int g = NW - 1; g >= 0; --g) {
        uint64_t m = s_mask[wave][g];
        while (m) {
          const int bit = 63 - __builtin_clzll(m);
          m &= ~(1ull << bit);
          const int k = g * 64 + bit;
          const uint2 r = s_rect[k];
          const bool inr = px < W && py < H && px >= (int)(r.x & 0xffffu) &&
                           px <= (int)(r.y & 0xffffu) && py >= (int)(r.x >> 16) &&
                           py <= (int)(r.y >> 16);
          uint32_t kb = inr ? pix_key_bits(s_q0[k], s_q1[k], make_float4(s_q2[k], 0, 0, 0), ur, vr)
                            : 0xffffffffu;
#pragma unroll
          for (int sh = 32; sh > 0; sh >>= 1) kb = min(kb, (uint32_t)__shfl_xor((int)kb, sh, 64));
          bound = min(bound, kb);
          if (lane == 0) s_bound[wave][k] = bound;
        }
      }
      // lane 0's bounds are read by the whole wave below
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    int g = 0;
    uint64_t m = s_mask[wave][0];
    uint32_t bound = 0;   // every key from the current position on is at least this
    while (true) {
      while (m == 0 && g + 1 < NW) m = s_mask[wave][++g];
      const bool more = m != 0;
      if (more) {
        const int k = g * 64 + __builtin_ctzll(m);
        m &= m - 1;
        bound = NW > 1 ? s_bound[wave][k] : s_beta[k];
        const float4 a = s_a[slot0 + k], b = s_b[slot0 + k];
        const uint2 r = s_rect[k];
        const int rx0 = (int)(r.x & 0xffffu), ry0 = (int)(r.x >> 16);
        const bool inr = alive && (uint32_t)(px - rx0) <= (uint32_t)((int)(r.y & 0xffffu) - rx0) &&
                         (uint32_t)(py - ry0) <= (uint32_t)((int)(r.y >> 16) - ry0);
        const float dx = a.x - xc, dy = a.y - yc;
        const float P = (a.z * dx) * dx, R = a.w * dx;
        const float qq = fmaf(dy, fmaf(b.x, dy, R), P);
        const float al = fminf(b.y * __builtin_amdgcn_exp2f(qq), aclamp);
        if (inr && al >= amin) {
          float num, den;
          pix_numden(s_q0[k], s_q1[k], make_float4(s_q2[k], 0, 0, 0), ur, vr, num, den);
          const float z = num / den;
          if (z != 0.0f && fabsf(z) < INFINITY) {
            s_newz[wave][nnew][lane] = z;
            s_newk[wave][nnew][lane] = (uint8_t)k;
            ++nnew;
          } else {   // not a word of the window's order: the pixel is redone exactly
            inexact = true;
            alive = false;
          }
        }
        if (!__ballot(alive && (nnew == B || nwin + nnew == K))) continue;
      } else if (b0 + BLOCK >= end) {
        bound = 0xffffffffu;   // the end of the list: everything goes
      }
      // ---- the new contributions into the window
      {
        double nw[B];
#pragma unroll
        for (int q = 0; q < B; ++q) {
          const double w = px_word(__float_as_uint(s_newz[wave][q][lane]),
                                   b0 - begin + (uint32_t)s_newk[wave][q][lane]);
          nw[q] = q < nnew ? w : empty;
        }
        px_sort<B>(nw);
        // descending into the last slots, empty where the lane has new ones
#pragma unroll
        for (int q = 0; q < B; ++q)
          asm("v_min_f64 %0, %0, %1" : "+v"(win[K - 1 - q]) : "v"(nw[q]));
        px_merge<K>(win);
        nwin += nnew;
        nnew = 0;
      }
      // ---- blend the entries below the bound, in order
      // (no bound, an image below the infinities', is a NaN: nothing goes; past
      // the list, or next to nothing but NaN keys, everything but the empty
      // slots, whose keys read as NaN)
      const float lim = bound >= 0xff800000u ? INFINITY : ord2f(bound);
      bool released = false;
      static_while<0, K>([&](auto index) __attribute__((always_inline)) {
        constexpr int i = decltype(index)::value;
        const uint32_t zb = px_hi(win[i]);
        const bool go = alive && __uint_as_float(zb) < lim;
        if (!__ballot(go)) return false;
        released = true;
        if (go) {
          // equal keys: the smaller index first (three alike: the exact pass)
          constexpr int i1 = i + 1 < K ? i + 1 : i, i2 = i + 2 < K ? i + 2 : i;
          if (i1 > i && px_hi(win[i1]) == zb) {
            if (i2 > i && px_hi(win[i2]) == zb) {
              inexact = true;
              alive = false;
            } else if (tkey_id(px_lo(win[i1])) < tkey_id(px_lo(win[i]))) {
              const double t = win[i];
              win[i] = win[i1];
              win[i1] = t;
            }
          }
          if (alive) {
            const uint32_t slot = px_lo(win[i]) & (RING - 1);
            const float4 a = s_a[slot], b = s_b[slot];
            const float dx = a.x - xc, dy = a.y - yc;
            const float P = (a.z * dx) * dx, R = a.w * dx;
            const float qq = fmaf(dy, fmaf(b.x, dy, R), P);
            const float al = fminf(b.y * __builtin_amdgcn_exp2f(qq), aclamp);
            const float Tn = fmaf(-al, T, T);
            if (Tn < tmin) {
              alive = false;   // stops before this contribution; the rest is moot
            } else {
              const float w0 = al * T;
              C0 = fmaf(b.z, w0, C0);
              C1 = fmaf(b.w, w0, C1);
              C2 = fmaf(s_c[slot], w0, C2);
              D = fmaf(__uint_as_float(zb), w0, D);
              T = Tn;
              ++cnt;
            }
          }
          win[i] = empty;
          --nwin;
        }
        return true;
      });
      // ---- close the gap at the front (empty words, then ascending)
      if (released) px_merge<K>(win);
      if (alive && nwin == K) {
        inexact = true;   // full, and none may go: the pixel is redone exactly
        alive = false;
      }
      if (!more || !__ballot(alive)) break;
    }
  }
  if (px < W && py < H) {
    const int64_t plane = (int64_t)W * H;
    const int64_t off = (int64_t)py * W + px;
    float* rgb = out_rgb + (int64_t)v * 3 * plane + off;
    rgb[0] = C0 + T * o.bg[0];
    rgb[plane] = C1 + T * o.bg[1];
    rgb[2 * plane] = C2 + T * o.bg[2];
    out_depth[(int64_t)v * plane + off] = D;
    out_t[(int64_t)v * plane + off] = T;
    out_n[(int64_t)v * plane + off] = cnt;
    if (inexact) fix_list[atomicAdd(fix_count, 1u)] = (uint32_t)((int64_t)v * plane + off);
  }
}

// Exact per-pixel order for the queued pixels, one wave per pixel, in
// rounds.  A round streams the pixel's tile list 64 records at a time and
// keeps, in LDS, the kFixCap least (key, index) above the last blended one:
// candidates go into a buffer of twice that size; when it overflows it is
// sorted and cut back, and its kFixCap-th key becomes a threshold below
// which a candidate must lie.  The scan stops at the first position whose
// bound word exceeds the threshold (every later key is at least that word),
// so the kept entries are exactly the least ones of the whole list.  They
// are blended in order; a round that keeps fewer than kFixCap entries has
// exhausted the list.
constexpr int kFixCap = 256, kFixWaves = 4;

struct FixAcc {
  float T, C0, C1, C2, D;
  int cnt;
  bool stop;
};

// Blend one contribution (wave-uniform values); false once the pixel stops.
__device__ __attribute__((always_inline)) inline bool fix_blend(FixAcc& s, float al, float r0,
                                                                float r1, float r2, float z,
                                                                float tmin) {
  const float w0 = al * s.T;
  const float Tn = fmaf(-al, s.T, s.T);   // as the windowed blend
  if (Tn < tmin) {
    s.stop = true;
    return false;
  }
  s.C0 = fmaf(r0, w0, s.C0);
  s.C1 = fmaf(r1, w0, s.C1);
  s.C2 = fmaf(r2, w0, s.C2);
  s.D = fmaf(z, w0, s.D);
  s.T = Tn;
  ++s.cnt;
  return true;
}

// Ascending bitonic sort of one wave's (key, alpha) pairs in LDS, P a power
// of two (pads hold ~0).
__device__ inline void wave_sort(uint64_t* ck, float* ca, int P, int lane) {
  for (int k = 2; k <= P; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = lane; i < (P >> 1); i += 64) {
        const int a = ((i & ~(j - 1)) << 1) | (i & (j - 1)), b = a + j;
        const uint64_t x = ck[a], y = ck[b];
        if ((x > y) == ((a & k) == 0)) {
          ck[a] = y;
          ck[b] = x;
          const float t = ca[a];
          ca[a] = ca[b];
          ca[b] = t;
        }
      }
      wave_sync_lds();
    }
}

__global__ __launch_bounds__(64 * kFixWaves) void k_gs_blend_px_fix(
    const uint32_t* __restrict__ fix_list, const uint32_t* __restrict__ fix_count,
    const uint64_t* __restrict__ tkey, const uint32_t* __restrict__ ids,
    const float4* __restrict__ rec, const float4* __restrict__ pcoef, int64_t n, KViews views,
    GsOpt o, int tile, int64_t tiles_x, int64_t tiles_per_view, const uint2* __restrict__ ranges,
    float* __restrict__ out_rgb, float* __restrict__ out_depth, float* __restrict__ out_t,
    int32_t* __restrict__ out_n) {
  constexpr int CAP2 = 2 * kFixCap;
  __shared__ uint64_t s_ck[kFixWaves][CAP2];
  __shared__ float s_ca[kFixWaves][CAP2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint64_t* ck = s_ck[wave];
  float* ca = s_ca[wave];
  const uint64_t below = (1ull << lane) - 1ull;
  const uint32_t nfix = *fix_count;
  for (uint32_t f = blockIdx.x * kFixWaves + wave; f < nfix; f += gridDim.x * kFixWaves) {
    const int64_t pix = fix_list[f];
    const KView& cv0 = views.v[0];
    const int64_t plane = (int64_t)cv0.W * cv0.H;
    const int v = (int)(pix / plane);
    const int64_t off = pix - (int64_t)v * plane;
    const KView& cv = views.v[v];
    const int py = (int)(off / cv.W), px = (int)(off - (int64_t)py * cv.W);
    const float xc = (float)px + 0.5f, yc = (float)py + 0.5f;
    const float ur = pix_ray(px, cv.cx, cv.fx), vr = pix_ray(py, cv.cy, cv.fy);
    const uint2 rg =
        ranges[(int64_t)v * tiles_per_view + (int64_t)(py / tile) * tiles_x + px / tile];
    const int64_t vbase = (int64_t)v * n;
    FixAcc acc{1.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0, false};
    uint64_t last = 0;   // the last blended (key, index), valid unless `first`
    bool first = true;
    while (!acc.stop) {
      int nc = 0;
      uint64_t thr = ~0ull;   // candidates must lie below
      for (uint32_t c0 = rg.x; c0 < rg.y; c0 += 64) {
        if (thr != ~0ull &&
            (uint32_t)(zs_word(tkey, ids, pcoef, vbase, rg.x, c0) >> 32) > (uint32_t)(thr >> 32))
          break;   // every key from here on is above the threshold
        const uint32_t j = c0 + lane;
        uint64_t key = ~0ull;
        float al = 0.0f;
        bool ok = false;
        if (j < rg.y) {
          const uint32_t id = (uint32_t)zs_word(tkey, ids, pcoef, vbase, rg.x, j);
          const int64_t e = vbase + id;
          float4 a, b, c;
          gs_stage(rec, e, a, b, c);
          const uint32_t lo = __float_as_uint(b.z), hi = __float_as_uint(b.w);
          if (px >= (int)(lo & 0xffffu) && px <= (int)(hi & 0xffffu) && py >= (int)(lo >> 16) &&
              py <= (int)(hi >> 16)) {
            const float dx = a.x - xc, dy = a.y - yc;
            const float P = (a.z * dx) * dx, R = a.w * dx;
            const float qq = fmaf(dy, fmaf(b.x, dy, R), P);
            al = fminf(b.y * __builtin_amdgcn_exp2f(qq), o.aclamp);
            if (al >= o.amin) {
              key = ((uint64_t)pix_key_bits(pcoef[kPcStride * e], pcoef[kPcStride * e + 1], pcoef[kPcStride * e + 2], ur,
                                            vr) << 32) | id;
              ok = (first || key > last) && key < thr;
            }
          }
        }
        const uint64_t m = __ballot(ok);
        if (ok) {
          const int q = nc + __builtin_popcountll(m & below);
          ck[q] = key;
          ca[q] = al;
        }
        nc += __builtin_popcountll(m);
        wave_sync_lds();
        if (nc > kFixCap + (CAP2 - kFixCap - 64)) {
          // buffer nearly full: keep the kFixCap least, tighten the threshold
          for (int i = nc + lane; i < CAP2; i += 64) ck[i] = ~0ull;
          wave_sync_lds();
          wave_sort(ck, ca, CAP2, lane);
          nc = kFixCap;
          thr = ck[kFixCap - 1];
        }
      }
      // the round's least entries, in order
      int P = 64;
      while (P < nc) P <<= 1;
      for (int i = nc + lane; i < P; i += 64) ck[i] = ~0ull;
      wave_sync_lds();
      wave_sort(ck, ca, P, lane);
      const int m = min(nc, kFixCap);
      for (int b0 = 0; b0 < m && !acc.stop; b0 += 64) {
        const int i = b0 + lane;
        const uint64_t k = i < m ? ck[i] : ~0ull;
        const float al = i < m ? ca[i] : 0.0f;
        float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
        if (i < m) {
          const int64_t e = vbase + (uint32_t)k;
          const float4 r1 = rec[3 * e + 1], r2 = rec[3 * e + 2];
          c0 = r1.z;
          c1 = r1.w;
          c2 = r2.x;
        }
        const int cnt = min(64, m - b0);
        for (int q = 0; q < cnt; ++q) {
          const uint64_t kq = __shfl(k, q, 64);
          if (!fix_blend(acc, __shfl(al, q, 64), __shfl(c0, q, 64), __shfl(c1, q, 64),
                         __shfl(c2, q, 64), ord2f((uint32_t)(kq >> 32)), o.tmin))
            break;
          last = kq;
          first = false;
        }
      }
      wave_sync_lds();
      if (nc < kFixCap) break;   // the list is exhausted
    }
    if (lane == 0) {
      float* rgb = out_rgb + (int64_t)v * 3 * plane + off;
      rgb[0] = acc.C0 + acc.T * o.bg[0];
      rgb[plane] = acc.C1 + acc.T * o.bg[1];
      rgb[2 * plane] = acc.C2 + acc.T * o.bg[2];
      out_depth[(int64_t)v * plane + off] = acc.D;
      out_t[(int64_t)v * plane + off] = acc.T;
      out_n[(int64_t)v * plane + off] = acc.cnt;
    }
  }
}

void launch_gs_pixdepth(const RenderWs& L, void* ws, const float* mean, const float* cov,
                        int64_t n, const KViews& kv, hipStream_t st) {
  const int64_t vn = L.vn;
  hipLaunchKernelGGL(k_gs_pixdepth, dim3((unsigned)std::min<int64_t>(8192, std::max<int64_t>(1, div_up(vn, 256)))),
                     dim3(256), 0, st, mean, cov, n, kv, at<float4>(ws, L.rec),
                     at<uint32_t>(ws, L.dkey0), at<float4>(ws, L.pcoef),
                     at<uint32_t>(ws, L.fix_count));
}

void launch_gs_tile_zsort(const RenderWs& L, void* ws, int64_t n, const KViews& kv, int tile,
                         hipStream_t st) {
  if (L.tiles_total == 0) return;
  hipLaunchKernelGGL(k_gs_tile_zsort, dim3((unsigned)L.tiles_total), dim3(kZsBlock), 0, st,
                     at<uint32_t>(ws, L.ids), at<float4>(ws, L.pcoef), n, kv, tile, L.tiles_x,
                     L.tiles_x * L.tiles_y, at<uint2>(ws, L.ranges), at<uint64_t>(ws, L.tkey));
}

void launch_gs_blend_px(const RenderWs& L, void* ws, int64_t n, const uint32_t* order,
                        const KViews& kv, const GsOpt& o, float* rgb, float* depth, float* tf,
                        int32_t* nc, hipStream_t st) {
  const uint64_t* tk = at<uint64_t>(ws, L.tkey);
  const uint32_t* ids = at<uint32_t>(ws, L.ids);
  const float4* rec = at<float4>(ws, L.rec);
  const float4* pc = at<float4>(ws, L.pcoef);
  const uint2* ranges = at<uint2>(ws, L.ranges);
  uint32_t* fl = at<uint32_t>(ws, L.fix_list);
  uint32_t* fc = at<uint32_t>(ws, L.fix_count);
  const int64_t tpv = L.tiles_x * L.tiles_y;
  switch (o.tile) {
    case 8:
      hipLaunchKernelGGL(k_gs_blend_px<8>, dim3((unsigned)L.tiles_total), dim3(PxCfg<8>::BLOCK),
                         0, st, order, tk, ids, rec, pc, n, kv, o, L.tiles_x, tpv, ranges, rgb,
                         depth, tf, nc, fl, fc);
      break;
    default:  // 16 (the entry point rejects larger tiles in this order)
      hipLaunchKernelGGL(k_gs_blend_px<16>, dim3((unsigned)L.tiles_total), dim3(PxCfg<16>::BLOCK),
                         0, st, order, tk, ids, rec, pc, n, kv, o, L.tiles_x, tpv, ranges, rgb,
                         depth, tf, nc, fl, fc);
      break;
  }
  hipLaunchKernelGGL(k_gs_blend_px_fix, dim3(1024), dim3(64 * kFixWaves), 0, st, fl, fc, tk, ids,
                     rec, pc, n, kv, o, o.tile, L.tiles_x, tpv, ranges, rgb, depth, tf, nc);
}

}  // namespace vrs
