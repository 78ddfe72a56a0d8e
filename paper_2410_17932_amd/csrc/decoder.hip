// Foveal decoder, forward: the small gated CNN that resolves each crop's
// neural-point pyramid into the foveal image F, with the periphery crop
// injected at the finest level (Sec. 3.3).
//
// Each level is one implicit-GEMM 3x3 convolution on the matrix cores:
//   M = output pixels (a tile of TH rows x 16 columns per workgroup, one
//       16-pixel row segment per MFMA row block),
//   N = 2 * Kp pre-activations, ordered so N-tile 2t holds the feature half
//       and N-tile 2t+1 the gate half of channels [16t, 16t+16): the gated
//       epilogue ELU(f) * sigmoid(g) pairs values held by the same lane,
//   K = 9 taps x Cin8 input channels (Cin padded to 8), padded to the MFMA
//       depth.
// The loader builds the zero-padded (TH+2) x 18 halo tile of the level's
// input in LDS directly from its sources -- pyramid layer, bilinear x2
// upsample of the coarser level's output, periphery crop -- so the
// concatenated input never exists in HBM.  One launch per level covers all
// crops (crops of uneven size are packed back to back in the grid).
// Arithmetic: float operands with v_mfma_f32_16x16x4_f32 (VRS_F32), or
// bfloat16 operands with v_mfma_f32_16x16x32_bf16 and float accumulation
// (VRS_BF16); biases, activations and the RGB head in float.
#include <type_traits>

#include "vrs_common.h"

namespace vrs {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kDecMaxNT = 8;  // widths up to 64 channels

struct DecLevel {
  int C, cin, cin8, kpad, kp, nout, kn, kpn, has_p, n_crops, W, H, width;
  int tile_base[VRS_MAX_CROPS + 1];
  int tiles_x[VRS_MAX_CROPS];
  int S[VRS_MAX_CROPS];
  int view[VRS_MAX_CROPS], x0[VRS_MAX_CROPS], y0[VRS_MAX_CROPS];
  int mx0[VRS_MAX_CROPS], my0[VRS_MAX_CROPS];   // largest origin inside the view
  const int4* place;                 // device crop placement (x0, y0, gaze), or null
  long long pyr_off[VRS_MAX_CROPS];  // float offset of this layer in the pyramid
  long long h_off[VRS_MAX_CROPS];    // element offset of h_l
  long long hn_off[VRS_MAX_CROPS];   // element offset of h_{l+1}
  long long pre_off[VRS_MAX_CROPS];  // float offset of the pre-activations
};

template <typename T>
struct DecTraits;
template <>
struct DecTraits<float> {
  static constexpr int KSTEP = 4;
  static constexpr int TH = 8;
};
template <>
struct DecTraits<__bf16> {
  static constexpr int KSTEP = 32;
  static constexpr int TH = 16;
};

// Origin of crop k in its view: the host value, or the device placement
// table's clamped into the view.
__device__ inline int dec_x0(const DecLevel& d, int k) {
  return d.place ? clamp_origin(d.place[k].x, d.mx0[k]) : d.x0[k];
}
__device__ inline int dec_y0(const DecLevel& d, int k) {
  return d.place ? clamp_origin(d.place[k].y, d.my0[k]) : d.y0[k];
}

__device__ inline float to_f(float x) { return x; }
__device__ inline float to_f(__bf16 x) { return (float)x; }

// Activations of the gated convolution, on the hardware exp2 and reciprocal
// (a few ulp; the reference and the gradients use the library functions).
__device__ inline float elu_f(float x) {
  return x > 0.0f ? x : __builtin_amdgcn_exp2f(x * 1.4426950408889634f) - 1.0f;
}
__device__ inline float sigmoid_f(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-x * 1.4426950408889634f));
}

// value of input channel c of level l at pixel (y, x) of crop k (inside the
// S x S layer)
template <typename T>
__device__ inline float dec_input(const DecLevel& d, int k, int S, int y, int x, int c,
                                  const float* __restrict__ pyr, const float* __restrict__ periph,
                                  const T* __restrict__ hnext) {
  if (c < d.C) return pyr[d.pyr_off[k] + ((long long)y * S + x) * d.C + c];
  c -= d.C;
  if (c < d.kn) {
    const int Sn = S >> 1;
    const float sx = 0.5f * (float)x - 0.25f, sy = 0.5f * (float)y - 0.25f;
    const float fx0 = floorf(sx), fy0 = floorf(sy);
    const float fx = sx - fx0, fy = sy - fy0;
    int xa = (int)fx0, ya = (int)fy0, xb = xa + 1, yb = ya + 1;
    xa = xa < 0 ? 0 : (xa > Sn - 1 ? Sn - 1 : xa);
    xb = xb < 0 ? 0 : (xb > Sn - 1 ? Sn - 1 : xb);
    ya = ya < 0 ? 0 : (ya > Sn - 1 ? Sn - 1 : ya);
    yb = yb < 0 ? 0 : (yb > Sn - 1 ? Sn - 1 : yb);
    const T* h = hnext + d.hn_off[k];
    const float v00 = to_f(h[((long long)ya * Sn + xa) * d.kpn + c]);
    const float v01 = to_f(h[((long long)ya * Sn + xb) * d.kpn + c]);
    const float v10 = to_f(h[((long long)yb * Sn + xa) * d.kpn + c]);
    const float v11 = to_f(h[((long long)yb * Sn + xb) * d.kpn + c]);
    return (1.0f - fy) * ((1.0f - fx) * v00 + fx * v01) + fy * ((1.0f - fx) * v10 + fx * v11);
  }
  c -= d.kn;
  if (d.has_p && c < 3) {
    const long long plane = (long long)d.W * d.H;
    return periph[(long long)d.view[k] * 3 * plane + c * plane +
                  (long long)(dec_y0(d, k) + y) * d.W + (dec_x0(d, k) + x)];
  }
  return 0.0f;
}

// Channel order of the halo tile in LDS (and of the packed weights' K
// dimension): [upsampled coarser output (kn) | pyramid layer (C) | periphery
// crop (3, finest level only) | zero padding], so the upsampled channels form
// aligned 8-channel groups.  Returns the original input channel, or -1 for
// padding.
__device__ __host__ inline int lds_to_orig(int c, int C, int kn, int has_p) {
  if (c < kn) return C + c;
  c -= kn;
  if (c < C) return c;
  c -= C;
  if (has_p && c < 3) return C + kn + c;
  return -1;
}

template <typename T>
__device__ inline void load8(const T* p, float* v);
template <>
__device__ inline void load8<__bf16>(const __bf16* p, float* v) {
  const v8bf a = *reinterpret_cast<const v8bf*>(p);
#pragma unroll
  for (int j = 0; j < 8; ++j) v[j] = (float)a[j];
}
template <>
__device__ inline void load8<float>(const float* p, float* v) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <typename T>
__device__ inline void store8(T* p, const float* v);
template <>
__device__ inline void store8<__bf16>(__bf16* p, const float* v) {
  // one vector conversion: four packed two-value conversions
  typedef float v8f __attribute__((ext_vector_type(8)));
  const v8f f = {v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]};
  *reinterpret_cast<v8bf*>(p) = __builtin_convertvector(f, v8bf);
}
template <>
__device__ inline void store8<float>(float* p, const float* v) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
// eight elements moved as they are
template <typename T>
__device__ inline void copy8(T* dst, const T* src) {
  static_assert(sizeof(T) == 2 || sizeof(T) == 4, "BF16 or float");
  *reinterpret_cast<uint4*>(dst) = *reinterpret_cast<const uint4*>(src);
  if constexpr (sizeof(T) == 4)
    *reinterpret_cast<uint4*>(dst + 4) = *reinterpret_cast<const uint4*>(src + 4);
}

// head: optional fused RGB head at the finest level (fovea != null):
// F = W_o h_0 + b_o written straight to the packed foveal image; h_0 is
// then only written when pre-activations are requested (backward).
struct HeadFuse {
  const float* wo;
  const float* bo;
  float* fovea;
  long long out_base[VRS_MAX_CROPS];
};

// Geometry of one workgroup's LDS: halo tile, the coarser level's footprint
// and the weights.  ONE: the whole weight operand (up to 24 KB) is loaded
// once, at the start, overlapping the halo fill; otherwise two chunks of CHS
// k-steps are double-buffered: 8 KB, or 4 KB for two N-tiles, whose level
// (the finest) is bound by the halo fill's latency, so four workgroups per
// CU (40 KB each) beat whole weights at three.
template <typename T, int NT, bool ONE>
struct ConvCfg {
  // 8-row tiles where the accumulators would leave one wave per SIMD
  static constexpr int TH = sizeof(T) == 2 && NT >= 8 ? 8 : DecTraits<T>::TH;
  static constexpr int KSTEP = DecTraits<T>::KSTEP;
  static constexpr int NPIX = (TH + 2) * 18;
  // halo pixel stride: cin8 channels, plus 8 (16 bytes) in the BF16 levels:
  // their strides of an odd number of 16-byte units (80 and 144 bytes) meet
  // more LDS bank conflicts in the fill's 16-byte stores and the A-operand
  // reads than 96 and 160 bytes.  The coarse footprint is then kept in BF16,
  // so the finest level still fits four workgroups per CU (together: LDS
  // conflict cycles -57 %, -49 % and -16 % for 2, 4 and 8 N-tiles).
  static constexpr int CPAD = sizeof(T) == 2 ? 8 : 0;
  static constexpr int CR = TH / 2 + 2, CC = 10;       // coarse rows / columns staged
  static constexpr int NOUT = NT * 16;
  static constexpr int NBUF = ONE ? 1 : 2;
  static constexpr int CBYTES = ONE ? 24576 : (NT <= 2 ? 4096 : 8192);
  static constexpr int CHS = CBYTES / (NOUT * KSTEP * (int)sizeof(T)) > 0
                                 ? CBYTES / (NOUT * KSTEP * (int)sizeof(T)) : 1;
  static constexpr int CK = CHS * KSTEP;                // k per chunk
  static constexpr int BROW = CK + 16 / (int)sizeof(T); // padded LDS row (elements)
  static constexpr int PPR = CK * (int)sizeof(T) / 16;  // 16-byte pieces per row
  static constexpr int PIECES = NOUT * PPR;
  static constexpr int PPT = (PIECES + 255) / 256;
};

// The weight chunks reuse the coarse footprint's LDS (the coarser level's
// output as stored, T) once the halo tile is filled; the per-k-step A
// offsets (int [k-steps][4]) follow.
template <typename T, int NT, bool ONE>
__host__ __device__ inline int conv_region_bytes(int kn) {
  using Cfg = ConvCfg<T, NT, ONE>;
  const int kn8 = (kn + 7) & ~7;
  const int coarse = Cfg::CR * Cfg::CC * kn8 * (int)sizeof(T);
  const int wchunks = Cfg::NBUF * Cfg::NOUT * Cfg::BROW * (int)sizeof(T);
  return coarse > wchunks ? coarse : wchunks;
}
template <typename T, int NT, bool ONE>
__host__ __device__ inline size_t conv_smem_bytes(int cin8, int kn, int kpad) {
  using Cfg = ConvCfg<T, NT, ONE>;
  return (size_t)Cfg::NPIX * (cin8 + Cfg::CPAD) * sizeof(T) + conv_region_bytes<T, NT, ONE>(kn) +
         (size_t)(kpad / Cfg::KSTEP) * 4 * sizeof(int);
}

// One 16-channel slice of the RGB head on the matrix cores: acc += A B with
// A = the head weights (lane (col, kq): W_o[col][4 kq + i]) and B = the
// gated values (lane (col, kq): channels 4 kq + i of pixel col).  BF16
// operands with float accumulation (one 16x16x16 step), or float operands
// (four 16x16x4 steps, the slice's k = 4 kq + i taken as k-index kq of
// step i).
template <typename T>
__device__ inline v4f head_mfma(const float* wa, const float* hv, v4f acc) {
  if constexpr (sizeof(T) == 2) {
    typedef short v4s __attribute__((ext_vector_type(4)));
    v4s a, b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      a[i] = __builtin_bit_cast(short, (__bf16)wa[i]);
      b[i] = __builtin_bit_cast(short, (__bf16)hv[i]);
    }
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc, 0, 0, 0);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[i], hv[i], acc, 0, 0, 0);
    return acc;
  }
}

// Register budget per N-tile count: the occupancy the accumulators allow
// (4, 3, 2, 2 waves per SIMD for 2, 4, 6, 8 N-tiles; 8 N-tiles use 8-row
// tiles).
template <int NT>
constexpr int conv_waves() { return NT <= 2 ? 4 : (NT <= 4 ? 3 : 2); }
template <typename T, int NT, bool ONE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(conv_waves<NT>())))
void k_dec_conv(DecLevel d, const float* __restrict__ pyr,
                                                  const float* __restrict__ periph,
                                                  const T* __restrict__ hnext,
                                                  const T* __restrict__ wp,
                                                  const float* __restrict__ bp,
                                                  T* __restrict__ hout, float* __restrict__ pre,
                                                  HeadFuse hf) {
  using Cfg = ConvCfg<T, NT, ONE>;
  constexpr int TH = Cfg::TH, RPW = TH / 4, KSTEP = Cfg::KSTEP, NPIX = Cfg::NPIX;
  constexpr int CR = Cfg::CR, CC = Cfg::CC, NOUT = Cfg::NOUT, CHS = Cfg::CHS, CK = Cfg::CK;
  constexpr int BROW = Cfg::BROW;
  extern __shared__ __align__(16) char smem[];
  const int cin8 = d.cin8, kn8 = (d.kn + 7) & ~7;
  const int cs = cin8 + Cfg::CPAD;   // halo pixel stride (elements)
  T* tile = reinterpret_cast<T*>(smem);
  char* region = smem + (size_t)NPIX * cs * sizeof(T);
  T* ctile = reinterpret_cast<T*>(region);
  T* sB = reinterpret_cast<T*>(region);   // after the fill
  int* s_aoff = reinterpret_cast<int*>(region + conv_region_bytes<T, NT, ONE>(d.kn));
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int k = 0;
  while (k + 1 < d.n_crops && (int)blockIdx.x >= d.tile_base[k + 1]) ++k;
  const int tl = blockIdx.x - d.tile_base[k];
  const int S = d.S[k];
  const int oy = (tl / d.tiles_x[k]) * TH, ox = (tl % d.tiles_x[k]) * 16;
  const int nsteps = d.kpad / KSTEP;
  const int nchunks = (nsteps + CHS - 1) / CHS;
  // ---- weight chunks: global -> registers -> LDS, one chunk ahead
  uint4 breg[Cfg::PPT];
  auto load_chunk = [&](int c) {
#pragma unroll
    for (int q = 0; q < Cfg::PPT; ++q) {
      const int pc = tid + q * 256;
      breg[q] = make_uint4(0, 0, 0, 0);
      if (pc < Cfg::PIECES) {
        const int n = pc / Cfg::PPR, kk = (pc - n * Cfg::PPR) * (16 / (int)sizeof(T));
        const int gk = c * CK + kk;
        if (gk < d.kpad) breg[q] = *reinterpret_cast<const uint4*>(wp + (long long)n * d.kpad + gk);
      }
    }
  };
  auto store_chunk = [&](int buf) {
#pragma unroll
    for (int q = 0; q < Cfg::PPT; ++q) {
      const int pc = tid + q * 256;
      if (pc < Cfg::PIECES) {
        const int n = pc / Cfg::PPR, kk = (pc - n * Cfg::PPR) * (16 / (int)sizeof(T));
        *reinterpret_cast<uint4*>(&sB[(buf * NOUT + n) * BROW + kk]) = breg[q];
      }
    }
  };
  load_chunk(0);
  // ---- the coarser level's output under this tile, clamped at the layer
  // edge, staged once (each coarse pixel feeds up to 16 fine pixels)
  const int Sn = S >> 1;
  const int cy0 = (oy >> 1) - 1, cx0 = (ox >> 1) - 1;
  if (d.kn > 0) {
    // copied as stored (8 channels = one 16-byte piece in BF16)
    const int kg = kn8 >> 3;
    const int nco = CR * CC * kg;
    auto csrc = [&](int e) {
      const int cp = e / kg, g = e - cp * kg;
      const int cyi = cp / CC, cxi = cp - cyi * CC;
      int yy = cy0 + cyi, xx = cx0 + cxi;
      yy = yy < 0 ? 0 : (yy > Sn - 1 ? Sn - 1 : yy);
      xx = xx < 0 ? 0 : (xx > Sn - 1 ? Sn - 1 : xx);
      return hnext + d.hn_off[k] + ((long long)yy * Sn + xx) * d.kpn + g * 8;
    };
    // two items per thread and round, both loads in flight before the stores
    for (int e0 = tid; e0 < nco; e0 += 512) {
      const int e1 = e0 + 256;
      uint4 r0[sizeof(T) / 2], r1[sizeof(T) / 2];
      const T* p0 = csrc(e0);
#pragma unroll
      for (int h = 0; h < (int)sizeof(T) / 2; ++h) r0[h] = reinterpret_cast<const uint4*>(p0)[h];
      if (e1 < nco) {
        const T* p1 = csrc(e1);
#pragma unroll
        for (int h = 0; h < (int)sizeof(T) / 2; ++h) r1[h] = reinterpret_cast<const uint4*>(p1)[h];
      }
#pragma unroll
      for (int h = 0; h < (int)sizeof(T) / 2; ++h) reinterpret_cast<uint4*>(&ctile[e0 * 8])[h] = r0[h];
      if (e1 < nco)
#pragma unroll
        for (int h = 0; h < (int)sizeof(T) / 2; ++h) reinterpret_cast<uint4*>(&ctile[e1 * 8])[h] = r1[h];
    }
    __syncthreads();
  }
  // A-operand offset of each k-step and lane group kq: k = 32 s + 8 kq (BF16,
  // one 8-channel unit) or 4 s + kq (FP32, one channel) is tap * cin8 +
  // channel.  Steps past the 9 taps read tap 8 (their weights are zero).
  {
    const int units = sizeof(T) == 2 ? (cin8 >> 3) : cin8;
    for (int i = tid; i < nsteps * 4; i += 256) {
      const int u = i;   // unit index along K: 4 per k-step
      int tap = u / units, cu = u - tap * units;
      if (tap > 8) {
        tap = 8;
        cu = 0;
      }
      const int ty = tap / 3, tx = tap - 3 * ty;
      s_aoff[i] = (ty * 18 + tx) * cs + cu * (sizeof(T) == 2 ? 8 : 1);
    }
  }
  // ---- halo tile fill.  Upsampled channels: one work item per 2x2 block of
  // fine pixels and 8-channel group -- fine rows 2m+1, 2m+2 (and columns
  // likewise) interpolate the same two coarse rows with weights 3/4, 1/4 and
  // 1/4, 3/4, so four coarse reads serve four pixels.  Other channels
  // (pyramid layer, periphery crop, padding): one item per pixel and group.
  // Pixels outside the layer are zero.
  const int G = cin8 >> 3;
  const int kgf = d.kn >> 3;   // full 8-channel groups of upsampled channels
  constexpr int NB = (TH + 2) / 2 * 9;   // 2x2 blocks of the halo tile
  const bool fast_py = d.C == 4 && (d.kn & 7) == 0 && (reinterpret_cast<uintptr_t>(pyr) & 15) == 0;
  const long long plane = (long long)d.W * d.H;
  const int n_up = NB * kgf, n_items = n_up + NPIX * (G - kgf);
  // this crop's pyramid layer and periphery window (the origin read once)
  const float* pyr_base = pyr + d.pyr_off[k];
  const float* per_base = d.has_p ? periph + (long long)d.view[k] * 3 * plane +
                                        (long long)dec_y0(d, k) * d.W + dec_x0(d, k)
                                  : periph;
  // every halo pixel inside the layer: no zero selects
  const bool interior = oy >= 1 && ox >= 1 && oy + TH + 1 <= S && ox + 17 <= S;
  // upsampled item e = block * kgf + group (groups fastest, so that a wave's
  // coarse reads and tile writes are runs of consecutive 32- and 16-byte
  // pieces), advanced by 256 items per round without divisions
  const int kgf_s = kgf > 0 ? kgf : 1;
  const int up_sb = 256 / kgf_s, up_sg = 256 - up_sb * kgf_s;
  int up_blk = tid / kgf_s, up_g = tid - up_blk * kgf_s;
  for (int e = tid; e < n_items; e += 256) {
    const int blk = up_blk, g = up_g;
    up_blk += up_sb;
    up_g += up_sg;
    if (up_g >= kgf_s) {
      up_g -= kgf_s;
      ++up_blk;
    }
    if (e < n_up) {
      const int bi = blk / 9, bj = blk - bi * 9;
      const T* c00 = &ctile[(bi * CC + bj) * kn8 + g * 8];
      float a00[8], a01[8], a10[8], a11[8];
      load8<T>(c00, a00);
      load8<T>(c00 + kn8, a01);
      load8<T>(c00 + CC * kn8, a10);
      load8<T>(c00 + (CC + 1) * kn8, a11);
      // horizontal: left fine column (3/4 a_0 + 1/4 a_1), right (1/4, 3/4),
      // each pair from the difference: a_0 + d/4 and a_1 - d/4
      float tl[8], tr[8], bl[8], br[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float dt = a01[j] - a00[j], db = a11[j] - a10[j];
        tl[j] = fmaf(0.25f, dt, a00[j]);
        tr[j] = fmaf(-0.25f, dt, a01[j]);
        bl[j] = fmaf(0.25f, db, a10[j]);
        br[j] = fmaf(-0.25f, db, a11[j]);
      }
      auto put = [&](auto inside_tag) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int dy = q >> 1, dx = q & 1;
          const int hy = 2 * bi + dy, hx = 2 * bj + dx;
          const int y = oy + hy - 1, x = ox + hx - 1;
          const bool in = decltype(inside_tag)::value || (y >= 0 && y < S && x >= 0 && x < S);
          float v[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            // vertical likewise: top + e/4 (upper fine row), bot - e/4
            const float top = dx ? tr[j] : tl[j], bot = dx ? br[j] : bl[j];
            const float e = bot - top;
            const float val = dy ? fmaf(-0.25f, e, bot) : fmaf(0.25f, e, top);
            v[j] = in ? val : 0.0f;
          }
          store8<T>(&tile[(hy * 18 + hx) * cs + g * 8], v);
        }
      };
      if (interior)
        put(std::true_type{});
      else
        put(std::false_type{});
    } else {
      const int e2 = e - n_up;
      const int g = kgf + e2 / NPIX, pix = e2 - (g - kgf) * NPIX;
      const int hy = pix / 18, hx = pix - hy * 18;
      const int y = oy + hy - 1, x = ox + hx - 1;
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = 0.0f;
      if (y >= 0 && y < S && x >= 0 && x < S) {
        const int c0 = g * 8;
        if (fast_py && c0 == d.kn) {
          // pyramid layer (4 channels, one 16-byte load) and periphery crop
          const float4 pv = *reinterpret_cast<const float4*>(pyr_base + ((long long)y * S + x) * 4);
          v[0] = pv.x; v[1] = pv.y; v[2] = pv.z; v[3] = pv.w;
          if (d.has_p) {
            const float* pp = per_base + (long long)y * d.W + x;
            v[4] = pp[0];
            v[5] = pp[plane];
            v[6] = pp[2 * plane];
          }
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int oc = lds_to_orig(c0 + j, d.C, d.kn, d.has_p);
            if (oc >= 0) v[j] = dec_input<T>(d, k, S, y, x, oc, pyr, periph, hnext);
          }
        }
      }
      store8<T>(&tile[pix * cs + g * 8], v);
    }
  }
  __syncthreads();   // the coarse footprint is dead from here
  store_chunk(0);
  __syncthreads();
  // ---- MFMA main loop over weight chunks
  // the accumulators start from the biases (lane (col, kq) holds channels
  // 4 kq + i of each N-tile), so the epilogue adds nothing
  const int r0 = wave * RPW;
  const int col = lane & 15, kq = lane >> 4;
  v4f acc[RPW][NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const float4 bj = *reinterpret_cast<const float4*>(&bp[j * 16 + 4 * kq]);
#pragma unroll
    for (int r = 0; r < RPW; ++r) acc[r][j] = v4f{bj.x, bj.y, bj.z, bj.w};
  }
  const int rowbase = (r0 * 18 + col) * cs;
  for (int c = 0; c < nchunks; ++c) {
    if (!ONE && c + 1 < nchunks) load_chunk(c + 1);
    const T* B = sB + (ONE ? 0 : (c & 1)) * NOUT * BROW;
#pragma unroll
    for (int s = 0; s < CHS; ++s) {
      const int ks = c * CHS + s;
      if (ks >= nsteps) break;
      const int abase = rowbase + s_aoff[ks * 4 + kq];
      if constexpr (sizeof(T) == 2) {
        v8bf a[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r)
          a[r] = *reinterpret_cast<const v8bf*>(&tile[abase + r * 18 * cs]);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const v8bf b = *reinterpret_cast<const v8bf*>(&B[(j * 16 + col) * BROW + s * KSTEP + kq * 8]);
#pragma unroll
          for (int r = 0; r < RPW; ++r)
            acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b, a[r], acc[r][j], 0, 0, 0);
        }
      } else {
        float a[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r) a[r] = to_f(tile[abase + r * 18 * cs]);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const float b = to_f(B[(j * 16 + col) * BROW + s * KSTEP + kq]);
#pragma unroll
          for (int r = 0; r < RPW; ++r)
            acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b, a[r], acc[r][j], 0, 0, 0);
        }
      }
    }
    if (!ONE) {
      if (c + 1 < nchunks) store_chunk((c + 1) & 1);
      __syncthreads();
    }
  }
  // ---- gated epilogue.  The weights are the MFMA's A operand, so lane
  // (col, kq) holds channels 4 kq + i (i < 4) of N-tile j for the pixel in
  // column col: feature and gate of a channel sit in the same lane, and the
  // lane's four channels are contiguous in h and in the pre-activations.
  const bool write_h = hf.fovea == nullptr || pre != nullptr;
  const int x = ox + col;
  // The fused RGB head F = W_o h + b_o is one small matrix product per row
  // on the matrix cores: the gated values already sit in the layout of the
  // B operand (lane (col, kq): channels 4 kq + i of pixel col), W_o (rows:
  // colour channels, padded to 16) is the A operand, and the result's lanes
  // kq = 0 hold the three colours of pixel col.  Channel pairs outer, rows
  // inner: the head's A operand is built once per pair.
  v4f head[RPW];
  if (hf.fovea) {
    const v4f hb0 = kq == 0 ? v4f{hf.bo[0], hf.bo[1], hf.bo[2], 0.0f} : v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < RPW; ++r) head[r] = hb0;
  }
#pragma unroll
  for (int t = 0; t < NT / 2; ++t) {
    float wa[4];   // A operand: W_o[col][t 16 + 4 kq + i] (zero beyond 3 colours or the width)
    if (hf.fovea) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ch = t * 16 + 4 * kq + i;
        wa[i] = col < 3 && ch < d.width ? hf.wo[col * d.width + ch] : 0.0f;
      }
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int y = oy + r0 + r;
      if (y >= S) continue;   // uniform over the wave
      const long long p = (long long)y * S + x;
      const float f[4] = {acc[r][2 * t][0], acc[r][2 * t][1], acc[r][2 * t][2],
                          acc[r][2 * t][3]};
      const float g[4] = {acc[r][2 * t + 1][0], acc[r][2 * t + 1][1], acc[r][2 * t + 1][2],
                          acc[r][2 * t + 1][3]};
      float hv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) hv[i] = elu_f(f[i]) * sigmoid_f(g[i]);
      if (hf.fovea) head[r] = head_mfma<T>(wa, hv, head[r]);
      if (x < S) {
        if (write_h) {
          T* hp = hout + d.h_off[k] + p * d.kp + t * 16 + 4 * kq;
          if constexpr (sizeof(T) == 2) {
            typedef __bf16 v4bf __attribute__((ext_vector_type(4)));
            *reinterpret_cast<v4bf*>(hp) = v4bf{(__bf16)hv[0], (__bf16)hv[1], (__bf16)hv[2], (__bf16)hv[3]};
          } else {
            *reinterpret_cast<float4*>(hp) = make_float4(hv[0], hv[1], hv[2], hv[3]);
          }
        }
        if (pre) {
          float* pp = pre + d.pre_off[k] + p * d.nout;
          *reinterpret_cast<float4*>(pp + 2 * t * 16 + 4 * kq) = make_float4(f[0], f[1], f[2], f[3]);
          *reinterpret_cast<float4*>(pp + (2 * t + 1) * 16 + 4 * kq) = make_float4(g[0], g[1], g[2], g[3]);
        }
      }
    }
  }
  if (hf.fovea && kq == 0 && x < S) {
    const long long opl = (long long)S * S;
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
      const int y = oy + r0 + r;
      if (y >= S) continue;
      const long long p = (long long)y * S + x;
      hf.fovea[hf.out_base[k] + p] = head[r][0];
      hf.fovea[hf.out_base[k] + opl + p] = head[r][1];
      hf.fovea[hf.out_base[k] + 2 * opl + p] = head[r][2];
    }
  }
}

// Re-order every level's float weights [2K][3][3][Cin] into its GEMM
// operand [nout][kpad] (N-tile pairs of feature/gate halves, k = tap*Cin8 + c
// with c in the LDS channel order, zero padding) and its bias, all levels in
// one launch.
template <typename T>
struct PackArgs {
  int n;
  int K[VRS_MAX_LEVELS], cin[VRS_MAX_LEVELS], cin8[VRS_MAX_LEVELS], kp[VRS_MAX_LEVELS],
      kpad[VRS_MAX_LEVELS], kn[VRS_MAX_LEVELS];
  long long start[VRS_MAX_LEVELS + 1];   // first element of each level
  const float* w[VRS_MAX_LEVELS];
  const float* b[VRS_MAX_LEVELS];
  T* wp[VRS_MAX_LEVELS];
  float* bp[VRS_MAX_LEVELS];
  int C;
};

template <typename T>
__global__ void k_dec_pack(PackArgs<T> a) {
  const long long total = a.start[a.n];
  for (long long e0 = blockIdx.x * (long long)blockDim.x + threadIdx.x; e0 < total;
       e0 += (long long)gridDim.x * blockDim.x) {
    int l = 0;
    while (l + 1 < a.n && e0 >= a.start[l + 1]) ++l;
    const long long e = e0 - a.start[l];
    const int kpad = a.kpad[l], cin8 = a.cin8[l], K = a.K[l];
    const int n = (int)(e / kpad), kk = (int)(e - (long long)n * kpad);
    const int t = n / 32, half = (n % 32) / 16, ch = t * 16 + (n % 16);
    const int tap = kk / cin8, c = kk - tap * cin8;
    const int oc = lds_to_orig(c, a.C, a.kn[l], l == 0 ? 1 : 0);
    float v = 0.0f;
    if (ch < K && tap < 9 && oc >= 0 && oc < a.cin[l]) {
      const int row = half ? K + ch : ch;
      v = a.w[l][((long long)row * 9 + tap) * a.cin[l] + oc];
    }
    a.wp[l][e] = (T)v;
    if (kk == 0) a.bp[l][n] = ch < K ? a.b[l][half ? K + ch : ch] : 0.0f;
  }
}

// ------------------------------------------------------------ host side
struct DecPlan {
  int nd, C, dtype;
  int K[VRS_MAX_LEVELS], kp[VRS_MAX_LEVELS], cin[VRS_MAX_LEVELS], cin8[VRS_MAX_LEVELS],
      kpad[VRS_MAX_LEVELS];
  size_t w_off[VRS_MAX_LEVELS], b_off[VRS_MAX_LEVELS];   // offsets into the float weights
  size_t head_w, head_b;
  // workspace (bytes)
  size_t wp[VRS_MAX_LEVELS], bp[VRS_MAX_LEVELS], h[VRS_MAX_LEVELS];
  // the adjoint's weights, pre-activations and input gradient (one level at a time)
  size_t wb[VRS_MAX_LEVELS], pre, dx, total;
  long long h_elems[VRS_MAX_LEVELS];
  int n_crops;
  // level l's weights in the adjoint's padded channel order
  long long wb_elems(int l) const {
    return (long long)2 * kp[l] * 9 * ((l + 1 < nd ? kp[l + 1] : 0) + 16);
  }
};

static int round_up(int a, int b) { return (a + b - 1) / b * b; }

static bool dec_plan(const vrs_decoder_desc* dd, const vrs_crop* crops, int n_crops, DecPlan* P) {
  if (!dd || dd->n_levels < 1 || dd->n_levels > VRS_MAX_LEVELS || dd->in_ch < 1) return false;
  if (dd->dtype != VRS_F32 && dd->dtype != VRS_BF16) return false;
  if (n_crops < 1 || n_crops > VRS_MAX_CROPS || !crops) return false;
  P->nd = dd->n_levels;
  P->C = dd->in_ch;
  P->dtype = dd->dtype;
  P->n_crops = n_crops;
  const int kstep = dd->dtype == VRS_BF16 ? 32 : 4;
  const size_t esz = dd->dtype == VRS_BF16 ? 2 : 4;
  size_t wo = 0;
  for (int l = 0; l < P->nd; ++l) {
    const int K = dd->width[l];
    if (K < 1 || K > 16 * kDecMaxNT / 2) return false;
    P->K[l] = K;
    P->kp[l] = round_up(K, 16);
  }
  for (int l = 0; l < P->nd; ++l) {
    P->cin[l] = P->C + (l + 1 < P->nd ? P->K[l + 1] : 0) + (l == 0 ? 3 : 0);
    P->cin8[l] = round_up(P->cin[l], 8);
    P->kpad[l] = round_up(9 * P->cin8[l], kstep);
    P->w_off[l] = wo;
    wo += (size_t)2 * P->K[l] * 9 * P->cin[l];
    P->b_off[l] = wo;
    wo += 2 * P->K[l];
  }
  P->head_w = wo;
  P->head_b = wo + 3 * P->K[0];
  const int unit = 1 << (P->nd - 1);
  Carver c;
  long long pre = 0, dx = 0;
  for (int l = 0; l < P->nd; ++l) {
    long long he = 0;
    for (int k = 0; k < n_crops; ++k) {
      if (crops[k].size < unit || crops[k].size % unit) return false;
      const long long s = crops[k].size >> l;
      he += s * s;
    }
    P->h_elems[l] = he * P->kp[l];
    P->wp[l] = c.take((size_t)2 * P->kp[l] * P->kpad[l] * esz);
    P->bp[l] = c.take((size_t)2 * P->kp[l] * 4);
    P->h[l] = c.take((size_t)P->h_elems[l] * esz);
    P->wb[l] = c.take((size_t)P->wb_elems(l) * 4);
    pre = std::max(pre, he * 2 * P->kp[l]);
    if (l + 1 < P->nd) dx = std::max(dx, he * P->kp[l + 1]);
  }
  P->pre = c.take((size_t)pre * 4);
  P->dx = c.take((size_t)dx * 4);
  P->total = c.off;
  return true;
}

static void level_args(const DecPlan& P, int l, const vrs_crop* crops, int n_crops,
                       const KViews& kv, int levels, const vrs_crop_place* place, DecLevel* d,
                       int* blocks) {
  d->place = reinterpret_cast<const int4*>(place);
  const int NT = 2 * P.kp[l] / 16;
  const int TH = P.dtype == VRS_BF16 && NT < 8 ? 16 : 8;   // as ConvCfg
  d->C = P.C;
  d->cin = P.cin[l];
  d->cin8 = P.cin8[l];
  d->kpad = P.kpad[l];
  d->kp = P.kp[l];
  d->nout = 2 * P.kp[l];
  d->kn = l + 1 < P.nd ? P.K[l + 1] : 0;
  d->kpn = l + 1 < P.nd ? P.kp[l + 1] : 0;
  d->has_p = l == 0;
  d->n_crops = n_crops;
  d->W = kv.v[0].W;
  d->H = kv.v[0].H;
  d->width = P.K[l];
  long long pyr = 0, h = 0, hn = 0, pre = 0;
  int tb = 0;
  for (int k = 0; k < n_crops; ++k) {
    const int S = crops[k].size >> l;
    const int tx = (S + 15) / 16, ty = (S + TH - 1) / TH;
    d->tile_base[k] = tb;
    d->tiles_x[k] = tx;
    tb += tx * ty;
    d->S[k] = S;
    d->view[k] = crops[k].view;
    d->x0[k] = crops[k].x0;
    d->y0[k] = crops[k].y0;
    d->mx0[k] = kv.v[crops[k].view].W - crops[k].size;
    d->my0[k] = kv.v[crops[k].view].H - crops[k].size;
    long long lay = pyr;
    for (int q = 0; q < l; ++q) lay += (long long)(crops[k].size >> q) * (crops[k].size >> q);
    d->pyr_off[k] = lay * P.C;
    for (int q = 0; q < levels; ++q) pyr += (long long)(crops[k].size >> q) * (crops[k].size >> q);
    d->h_off[k] = h;
    h += (long long)S * S * P.kp[l];
    d->pre_off[k] = pre;
    pre += (long long)S * S * 2 * P.kp[l];
    if (l + 1 < P.nd) {
      d->hn_off[k] = hn;
      hn += (long long)(S / 2) * (S / 2) * P.kp[l + 1];
    } else {
      d->hn_off[k] = 0;
    }
  }
  d->tile_base[n_crops] = tb;
  *blocks = tb;
}

// LDS a workgroup may allocate on the current device (queried once).
static size_t max_lds_bytes() {
  static size_t cached = 0;
  if (!cached) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess)
      cached = (size_t)v;
    else
      cached = 64 * 1024;
  }
  return cached;
}

template <typename T, int NT>
static hipError_t launch_nt(const DecLevel& d, int blocks, const float* pyr, const float* periph,
                            const T* hn, const T* wp, const float* bp, T* h, float* pre,
                            const HeadFuse& hf, hipStream_t st) {
  // the whole weight operand in one LDS chunk when it fits (not with two
  // N-tiles: see ConvCfg)
  using One = ConvCfg<T, NT, true>;
  const bool one = NT > 2 && d.kpad <= One::CK;
  const size_t need = one ? conv_smem_bytes<T, NT, true>(d.cin8, d.kn, d.kpad)
                          : conv_smem_bytes<T, NT, false>(d.cin8, d.kn, d.kpad);
  if (need > max_lds_bytes()) return hipErrorInvalidValue;
  if (one)
    hipLaunchKernelGGL((k_dec_conv<T, NT, true>), dim3(blocks), dim3(256), need, st, d, pyr,
                       periph, hn, wp, bp, h, pre, hf);
  else
    hipLaunchKernelGGL((k_dec_conv<T, NT, false>), dim3(blocks), dim3(256), need, st, d, pyr,
                       periph, hn, wp, bp, h, pre, hf);
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_conv(const DecLevel& d, int NT, int blocks, const float* pyr,
                              const float* periph, const T* hn, const T* wp, const float* bp, T* h,
                              float* pre, const HeadFuse& hf, hipStream_t st) {
  switch (NT) {
    case 2: return launch_nt<T, 2>(d, blocks, pyr, periph, hn, wp, bp, h, pre, hf, st);
    case 4: return launch_nt<T, 4>(d, blocks, pyr, periph, hn, wp, bp, h, pre, hf, st);
    case 6: return launch_nt<T, 6>(d, blocks, pyr, periph, hn, wp, bp, h, pre, hf, st);
    default: return launch_nt<T, 8>(d, blocks, pyr, periph, hn, wp, bp, h, pre, hf, st);
  }
}

template <typename T>
static vrs_status decode_impl(const DecPlan& P, const float* pyramid, int levels,
                              const float* periph, const KViews& kv, const vrs_crop* crops,
                              int n_crops, const vrs_crop_place* place, const float* weights,
                              float* out, void* ws, hipStream_t st) {
  {
    PackArgs<T> pa;
    pa.n = P.nd;
    pa.C = P.C;
    long long s = 0;
    for (int l = 0; l < P.nd; ++l) {
      pa.K[l] = P.K[l];
      pa.cin[l] = P.cin[l];
      pa.cin8[l] = P.cin8[l];
      pa.kp[l] = P.kp[l];
      pa.kpad[l] = P.kpad[l];
      pa.kn[l] = l + 1 < P.nd ? P.K[l + 1] : 0;
      pa.w[l] = weights + P.w_off[l];
      pa.b[l] = weights + P.b_off[l];
      pa.wp[l] = at<T>(ws, P.wp[l]);
      pa.bp[l] = at<float>(ws, P.bp[l]);
      pa.start[l] = s;
      s += (long long)2 * P.kp[l] * P.kpad[l];
    }
    pa.start[P.nd] = s;
    const int blocks = (int)std::min<long long>(1024, (s + 255) / 256);
    hipLaunchKernelGGL(k_dec_pack<T>, dim3(blocks), dim3(256), 0, st, pa);
    VRS_LAUNCH_CHECK();
  }
  DecLevel d;
  for (int l = P.nd - 1; l >= 0; --l) {
    int blocks = 0;
    level_args(P, l, crops, n_crops, kv, levels, place, &d, &blocks);
    const T* hn = l + 1 < P.nd ? at<T>(ws, P.h[l + 1]) : nullptr;
    HeadFuse hf{};
    if (l == 0) {
      // the RGB head runs in the finest level's epilogue
      hf.wo = weights + P.head_w;
      hf.bo = weights + P.head_b;
      hf.fovea = out;
      long long o = 0;
      for (int k = 0; k < n_crops; ++k) {
        hf.out_base[k] = o;
        o += 3LL * crops[k].size * crops[k].size;
      }
    }
    VRS_HIP_CHECK(launch_conv<T>(d, 2 * P.kp[l] / 16, blocks, pyramid, periph, hn,
                                 at<T>(ws, P.wp[l]), at<float>(ws, P.bp[l]), at<T>(ws, P.h[l]),
                                 nullptr, hf, st));
  }
  return VRS_OK;
}

bool dec_plan_public(const vrs_decoder_desc* dd, const vrs_crop* crops, int n_crops, size_t* total) {
  DecPlan P;
  if (!dec_plan(dd, crops, n_crops, &P)) return false;
  *total = P.total;
  return true;
}

}  // namespace vrs

using namespace vrs;

extern "C" size_t vrs_decoder_workspace_size(const vrs_decoder_desc* dd, const vrs_crop* crops,
                                             int n_crops) {
  DecPlan P;
  if (!dec_plan(dd, crops, n_crops, &P)) return 0;
  return P.total;
}

// crops inside their (equally sized) views, sizes multiples of the coarsest
// layer; the origins only when no device placement table overrides them
static bool dec_crops_ok(const vrs_view* views, int n_views, const vrs_crop* crops, int n_crops,
                         int levels, const vrs_crop_place* place) {
  for (int i = 1; i < n_views; ++i)
    if (views[i].width != views[0].width || views[i].height != views[0].height) return false;
  for (int k = 0; k < n_crops; ++k) {
    const vrs_crop& c = crops[k];
    if (c.view < 0 || c.view >= n_views || c.size < 1 || c.size > views[c.view].width ||
        c.size > views[c.view].height || c.size % (1 << (levels - 1)))
      return false;
    if (!place && (c.x0 < 0 || c.y0 < 0 || c.x0 + c.size > views[c.view].width ||
                   c.y0 + c.size > views[c.view].height))
      return false;
  }
  return true;
}

namespace vrs {
vrs_status decode_impl_entry(const float* pyramid, int levels, const float* rgb_periphery,
                             const vrs_view* views, int n_views, const vrs_crop* crops,
                             int n_crops, const vrs_crop_place* place, const float* weights,
                             const vrs_decoder_desc* dd, float* fovea_rgb, void* ws,
                             size_t ws_bytes, void* stream, const Trace* tr) {
  DecPlan P;
  KViews kv;
  if (!make_views(views, n_views, &kv) || !dec_plan(dd, crops, n_crops, &P)) return VRS_EINVAL;
  if (levels < P.nd || levels > VRS_MAX_LEVELS) return VRS_EINVAL;
  if (!pyramid || !rgb_periphery || !weights || !fovea_rgb || !ws || ws_bytes < P.total)
    return VRS_EINVAL;
  if (dd->in_ch != 4) return VRS_EUNSUPPORTED;
  if (!dec_crops_ok(views, n_views, crops, n_crops, levels, place)) return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  trace_begin(tr, VRS_TRACE_DECODER, st);
  vrs_status r;
  if (P.dtype == VRS_BF16)
    r = decode_impl<__bf16>(P, pyramid, levels, rgb_periphery, kv, crops, n_crops, place,
                            weights, fovea_rgb, ws, st);
  else
    r = decode_impl<float>(P, pyramid, levels, rgb_periphery, kv, crops, n_crops, place,
                           weights, fovea_rgb, ws, st);
  trace_end(tr, VRS_TRACE_DECODER, st);
  return r;
}
}  // namespace vrs

extern "C" vrs_status vrs_decode_fovea(const float* pyramid, int levels,
                                       const float* rgb_periphery, const vrs_view* views,
                                       int n_views, const vrs_crop* crops, int n_crops,
                                       const vrs_crop_place* place, const float* weights,
                                       const vrs_decoder_desc* dd, float* fovea_rgb, void* ws,
                                       size_t ws_bytes, void* stream) {
  return decode_impl_entry(pyramid, levels, rgb_periphery, views, n_views, crops, n_crops, place,
                           weights, dd, fovea_rgb, ws, ws_bytes, stream, nullptr);
}

// ------------------------------------------------------------- backward
// Per level, finest first: the pre-activations are recomputed, the gate's
// adjoint turns them into their gradients, and the weight gradient and the
// input gradient are matrix products on the FP32 matrix cores (operands and
// sums stay in float32, as the pre-activations' gradients and the weights
// are).  Four 512 crops, 16/32/64/64: 109 GFLOP, 0.73 ms at the 150 TFLOP/s a
// large float32 product reaches; the products take 1.6 ms (0.65 input, 0.95
// weights) where per-element loops took 15.9 (11.9 and 4.0), the whole adjoint
// with the forward 2.07 ms instead of 16.7.
//
// Both products take the input channels in one padded order of 16-channel
// tiles, [pyramid 4 | upsampled kpn | periphery 3 | 1 spare | zeros], so that
// every group of four lanes' values has one destination.
namespace vrs {

// Input channel (of the weights) of padded channel n, or -1.
__device__ inline int pad_to_orig(int n, int kn, int kpn, int has_p) {
  if (n < 4) return n;
  n -= 4;
  if (n < kpn) return n < kn ? 4 + n : -1;
  n -= kpn;
  return has_p && n < 3 ? 4 + kn + n : -1;
}

// Weights as the input gradient's A operand, all levels in one launch:
// [nout / 32][tap][2 groups of 16 k][N-tile][lane][4], lane (col, kq) holding
// channel 16 j + col against pre-activations 16 g + 4 kq + s (s < 4): one
// 16-byte load per lane feeds four matrix steps.
struct PackBwdArgs {
  int n;
  int K[VRS_MAX_LEVELS], kn[VRS_MAX_LEVELS], kpn[VRS_MAX_LEVELS], cin[VRS_MAX_LEVELS];
  long long start[VRS_MAX_LEVELS + 1];
  const float* w[VRS_MAX_LEVELS];
  float* wb[VRS_MAX_LEVELS];
};

__global__ void k_dec_pack_bwd(PackBwdArgs a) {
  for (long long e0 = blockIdx.x * (long long)blockDim.x + threadIdx.x; e0 < a.start[a.n];
       e0 += (long long)gridDim.x * blockDim.x) {
    int l = 0;
    while (l + 1 < a.n && e0 >= a.start[l + 1]) ++l;
    const int e = (int)(e0 - a.start[l]);
    const int nt = a.kpn[l] / 16 + 1;
    const int s = e & 3, lane = (e >> 2) & 63;
    int q = e >> 8;
    const int j = q % nt;
    q /= nt;
    const int g = q & 1, tap = (q >> 1) % 9, c = (q >> 1) / 9;
    const int ch = c * 16 + 4 * (lane >> 4) + s;      // feature (g = 0) or gate (g = 1) half
    const int oc = pad_to_orig(j * 16 + (lane & 15), a.kn[l], a.kpn[l], l == 0);
    float v = 0.0f;
    if (ch < a.K[l] && oc >= 0)
      v = a.w[l][((long long)(g ? a.K[l] + ch : ch) * 9 + tap) * a.cin[l] + oc];
    a.wb[l][e] = v;
  }
}

// Gate: h = ELU(f) sigmoid(g); the pre-activations are overwritten by their
// gradients.  dh comes from the RGB head (HEAD, finest level: W_o^T dF, with
// the head's weight gradients summed on the way) or is gathered from the
// finer level's input gradient dx [pixel][kp]: the bilinear upsample's
// adjoint, rows and columns 2m-1 .. 2m+2 with weights 1/4, 3/4, 3/4, 1/4 (1
// for the pixel whose outer neighbour the clamp folds back).  A gather reads
// each value four times from cache, where the scatter it replaces took four
// device atomics per value.  HBM-bound: 16 B per pre-activation pair read
// and written.  One thread per pixel and four channels; a thread keeps its
// channels over its pixels.
struct GateArgs {
  int n_crops, kp, K;
  int S[VRS_MAX_CROPS];
  long long pix_base[VRS_MAX_CROPS + 1];
  long long out_base[VRS_MAX_CROPS];
};

template <typename T, bool HEAD>
__global__ __launch_bounds__(256) void k_dec_gate_bwd(GateArgs a, float* __restrict__ pre,
                                                      const float* __restrict__ dx,
                                                      const T* __restrict__ h0,
                                                      const float* __restrict__ wo,
                                                      const float* __restrict__ dF,
                                                      float* __restrict__ dwo,
                                                      float* __restrict__ dbo) {
  __shared__ float s_acc[3 * 64 + 3];
  const int G = a.kp >> 2, per = 256 / G;      // channel groups; pixels per workgroup and round
  const int g = threadIdx.x % G, slot = threadIdx.x / G, c0 = g * 4;
  float w[3][4], aw[3][4], ab[3] = {0, 0, 0};
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[r][i] = HEAD && c0 + i < a.K ? wo[r * a.K + c0 + i] : 0.0f;
      aw[r][i] = 0.0f;
    }
  if (HEAD) {
    for (int e = threadIdx.x; e < 3 * a.K + 3; e += 256) s_acc[e] = 0.0f;
    __syncthreads();
  }
  const long long npix = a.pix_base[a.n_crops];
  for (long long p = blockIdx.x * (long long)per + slot; slot < per && p < npix;
       p += (long long)gridDim.x * per) {
    int k = 0;
    while (k + 1 < a.n_crops && p >= a.pix_base[k + 1]) ++k;
    const int S = a.S[k];
    const int q = (int)(p - a.pix_base[k]);
    float dh[4] = {0, 0, 0, 0};
    if (HEAD) {
      const long long plane = (long long)S * S;
      float gr[3];
#pragma unroll
      for (int r = 0; r < 3; ++r) gr[r] = dF[a.out_base[k] + r * plane + q];
      float hv[4] = {0, 0, 0, 0};
      if (dwo)
#pragma unroll
        for (int i = 0; i < 4; ++i) hv[i] = to_f(h0[p * a.kp + c0 + i]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dh[i] = w[0][i] * gr[0] + w[1][i] * gr[1] + w[2][i] * gr[2];
#pragma unroll
        for (int r = 0; r < 3; ++r) aw[r][i] += gr[r] * hv[i];
      }
#pragma unroll
      for (int r = 0; r < 3; ++r) ab[r] += gr[r];
    } else {
      const int y = q / S, x = q - y * S, Sf = 2 * S;
      const float* src = dx + 4 * a.pix_base[k] * a.kp + c0;   // the finer layer has four times the pixels
#pragma unroll
      for (int iy = 0; iy < 4; ++iy) {
        const int fy = 2 * y - 1 + iy;
        if (fy < 0 || fy >= Sf) continue;
        const float wy = fy == 0 || fy == Sf - 1 ? 1.0f : (iy == 0 || iy == 3 ? 0.25f : 0.75f);
        float row[4] = {0, 0, 0, 0};
#pragma unroll
        for (int ix = 0; ix < 4; ++ix) {
          const int fx = 2 * x - 1 + ix;
          if (fx < 0 || fx >= Sf) continue;
          const float wx = fx == 0 || fx == Sf - 1 ? 1.0f : (ix == 0 || ix == 3 ? 0.25f : 0.75f);
          const float4 v =
              *reinterpret_cast<const float4*>(src + ((long long)fy * Sf + fx) * a.kp);
          row[0] = fmaf(wx, v.x, row[0]);
          row[1] = fmaf(wx, v.y, row[1]);
          row[2] = fmaf(wx, v.z, row[2]);
          row[3] = fmaf(wx, v.w, row[3]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) dh[i] = fmaf(wy, row[i], dh[i]);
      }
    }
    float* pf = pre + p * 2 * a.kp + (c0 >> 4) * 32 + (c0 & 15);
    const float4 f4 = *reinterpret_cast<const float4*>(pf);
    const float4 g4 = *reinterpret_cast<const float4*>(pf + 16);
    const float fv[4] = {f4.x, f4.y, f4.z, f4.w}, gv[4] = {g4.x, g4.y, g4.z, g4.w};
    float of[4], og[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float sg = 1.0f / (1.0f + expf(-gv[i]));
      const float el = fv[i] > 0.0f ? fv[i] : expm1f(fv[i]);
      const float del = fv[i] > 0.0f ? 1.0f : el + 1.0f;
      const bool in = c0 + i < a.K;
      of[i] = in ? dh[i] * sg * del : 0.0f;
      og[i] = in ? dh[i] * el * sg * (1.0f - sg) : 0.0f;
    }
    *reinterpret_cast<float4*>(pf) = make_float4(of[0], of[1], of[2], of[3]);
    *reinterpret_cast<float4*>(pf + 16) = make_float4(og[0], og[1], og[2], og[3]);
  }
  if (!HEAD || !dwo) return;
#pragma unroll
  for (int r = 0; r < 3; ++r) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (slot < per && c0 + i < a.K) atomicAdd(&s_acc[r * a.K + c0 + i], aw[r][i]);
    if (slot < per && g == 0) atomicAdd(&s_acc[3 * a.K + r], ab[r]);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 3 * a.K + 3; e += 256)
    atomicAdd(e < 3 * a.K ? &dwo[e] : &dbo[e - 3 * a.K], s_acc[e]);
}

// Input gradient: a 3x3 convolution of the pre-activations' gradients with
// the flipped weights.  One workgroup per tile of 4 RPW rows x 16 columns,
// RPW rows per wave; the halo of 32 pre-activations at a time in LDS, weights
// from L2 in operand order, one step ahead of their use.  Bound by the FP32
// matrix rate (4 RPW NT steps of 32 cycles for RPW 16-byte LDS reads and NT
// 16-byte global loads per lane).  The pixel stride of 36 floats spreads the
// 16 columns of a read over all LDS banks.
template <int NT, int RPW>
__global__ __launch_bounds__(256) void k_dec_dgrad(DecLevel d, const float* __restrict__ dpre,
                                                   const float* __restrict__ wb,
                                                   float* __restrict__ dpyr,
                                                   float* __restrict__ dx,
                                                   float* __restrict__ dper) {
  constexpr int TH = 4 * RPW, NPIX = (TH + 2) * 18, PS = 36;
  __shared__ __align__(16) float s_g[NPIX * PS];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int k = 0;
  while (k + 1 < d.n_crops && (int)blockIdx.x >= d.tile_base[k + 1]) ++k;
  const int tl = blockIdx.x - d.tile_base[k], S = d.S[k];
  const int oy = (tl / d.tiles_x[k]) * TH, ox = (tl % d.tiles_x[k]) * 16;
  const int r0 = wave * RPW, col = lane & 15, kq = lane >> 4;
  const float* src = dpre + d.pre_off[k];
  v4f acc[RPW][NT];
#pragma unroll
  for (int r = 0; r < RPW; ++r)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[r][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  const int chunks = d.nout >> 5;
  const v4f* wp = reinterpret_cast<const v4f*>(wb) + lane;
  v4f b[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) b[j] = wp[j * 64];
  for (int c = 0; c < chunks; ++c) {
    if (c) __syncthreads();
    for (int i = tid; i < NPIX * 8; i += 256) {
      const int pix = i >> 3, q = i & 7;
      const int y = oy + pix / 18 - 1, x = ox + pix % 18 - 1;
      float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (y >= 0 && y < S && x >= 0 && x < S)
        v = *reinterpret_cast<const float4*>(src + ((long long)y * S + x) * d.nout + c * 32 + q * 4);
      *reinterpret_cast<float4*>(&s_g[pix * PS + q * 4]) = v;
    }
    __syncthreads();
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
      for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          wp += NT * 64;
          // the next step's weights (past the end: this step's again)
          const bool end = c == chunks - 1 && ky == 2 && kx == 2 && g == 1;
          v4f bn[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) bn[j] = wp[(end ? -NT * 64 : 0) + j * 64];
          v4f av[RPW];
#pragma unroll
          for (int r = 0; r < RPW; ++r)
            av[r] = *reinterpret_cast<const v4f*>(
                &s_g[((r0 + r + 2 - ky) * 18 + col + 2 - kx) * PS + g * 16 + kq * 4]);
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int j = 0; j < NT; ++j)
#pragma unroll
              for (int r = 0; r < RPW; ++r)
                acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][s], av[r][s], acc[r][j], 0, 0, 0);
#pragma unroll
          for (int j = 0; j < NT; ++j) b[j] = bn[j];
        }
  }
  // lane (col, kq) holds padded channels 16 j + 4 kq + i (i < 4) of pixel col
  const int x = ox + col;
  if (x >= S) return;
  const long long pix0 = d.pre_off[k] / d.nout;
#pragma unroll
  for (int r = 0; r < RPW; ++r) {
    const int y = oy + r0 + r;
    if (y >= S) continue;
    const long long p = (long long)y * S + x;
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int n0 = j * 16 + kq * 4 - 4;     // after the pyramid's four
      if (n0 < 0) {
        if (dpyr)
#pragma unroll
          for (int i = 0; i < 4; ++i) dpyr[d.pyr_off[k] + p * 4 + i] += acc[r][j][i];
      } else if (n0 < d.kpn) {
        *reinterpret_cast<v4f*>(dx + (pix0 + p) * d.kpn + n0) = acc[r][j];
      } else if (n0 == d.kpn && d.has_p && dper) {
        const long long plane = (long long)d.W * d.H;
        float* o = dper + (long long)d.view[k] * 3 * plane +
                   (long long)(dec_y0(d, k) + y) * d.W + (dec_x0(d, k) + x);
#pragma unroll
        for (int i = 0; i < 3; ++i) atomicAdd(o + i * plane, acc[r][j][i]);
      }
    }
  }
}

// Weight gradient dW[row][tap][c] = sum over pixels of dpre[p][row]
// x[p + tap][c], and db from a channel of ones (the spare one): a matrix
// product with the pixels as its depth.  A workgroup takes 32 rows (blockIdx.y)
// and keeps their 2 x 9 NT output tiles in registers, a quarter per wave, over
// its share of the 8 x 16 pixel tiles, so that each sum reaches memory once
// per workgroup.  Bound by the FP32 matrix rate: 2 + 9 NT / 4 LDS reads for
// 9 NT / 2 steps of 32 cycles.  The pixel strides put a read's four pixels in
// different banks.
template <int NT>
constexpr int wg_stride() { return NT % 2 ? 16 * NT : 16 * NT + 16; }
constexpr int kWgRows = 36;   // dpre pixel stride in LDS (32 rows)
template <int NT>
constexpr size_t wg_smem() { return (size_t)(180 * wg_stride<NT>() + 128 * kWgRows) * 4; }

template <typename T, int NT>
__global__ __launch_bounds__(256) void k_dec_wgrad(DecLevel d, const float* __restrict__ pyr,
                                                   const float* __restrict__ periph,
                                                   const T* __restrict__ hnext,
                                                   const float* __restrict__ dpre,
                                                   float* __restrict__ dw, float* __restrict__ db) {
  constexpr int NQ = (9 * NT + 3) / 4, CS = wg_stride<NT>();
  extern __shared__ __align__(16) char smem[];
  float* s_x = reinterpret_cast<float*>(smem);    // [10][18] pixels, padded channels
  float* s_g = s_x + 180 * CS;                    // [8][16] pixels, 32 rows
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4, rg = blockIdx.y;
  v4f acc[2][NQ];
  int off[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    acc[0][i] = acc[1][i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    const int q = wave + 4 * i < 9 * NT ? wave + 4 * i : 0;
    const int tap = q / NT;
    off[i] = ((tap / 3) * 18 + tap % 3) * CS + (q - tap * NT) * 16;
  }
  // the last channel tile's zeros, which no pixel tile overwrites
  for (int e = tid; e < 180 * 8; e += 256) s_x[(e >> 3) * CS + 16 * NT - 8 + (e & 7)] = 0.0f;
  const int tiles = d.tile_base[d.n_crops];
  const long long plane = (long long)d.W * d.H;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    int k = 0;
    while (k + 1 < d.n_crops && tile >= d.tile_base[k + 1]) ++k;
    const int S = d.S[k], tl = tile - d.tile_base[k];
    const int oy = (tl / d.tiles_x[k]) * 8, ox = (tl % d.tiles_x[k]) * 16;
    __syncthreads();
    // upsampled channels, four per item: loads without branches (clamped
    // places, the weights of pixels outside the layer zero), so that several
    // items' loads are in flight; 64-bit offsets (a 64-wide level of more than
    // 5792 pixels a side passes 2^31 elements)
    constexpr int KG = 4 * (NT - 1);
    if (KG > 0) {
      const int Sn = S >> 1;
      const T* h = hnext + d.hn_off[k];
#pragma unroll 3
      for (int e = tid; e < 180 * KG; e += 256) {
        const int pix = e / (KG > 0 ? KG : 1), n = (e - pix * KG) * 4;
        const int y = oy + pix / 18 - 1, x = ox + pix % 18 - 1;
        const bool in = y >= 0 && y < S && x >= 0 && x < S;
        const int ya = (y - 1) >> 1, xa = (x - 1) >> 1;    // floor((y - 1/2) / 2)
        const float fy = y & 1 ? 0.25f : 0.75f, fx = x & 1 ? 0.25f : 0.75f;
        const int y0 = min(max(ya, 0), Sn - 1), y1 = min(max(ya + 1, 0), Sn - 1);
        const int x0 = min(max(xa, 0), Sn - 1), x1 = min(max(xa + 1, 0), Sn - 1);
        typedef T v4t __attribute__((ext_vector_type(4)));
        const v4t a00 = *reinterpret_cast<const v4t*>(h + (long long)(y0 * Sn + x0) * (KG * 4) + n);
        const v4t a01 = *reinterpret_cast<const v4t*>(h + (long long)(y0 * Sn + x1) * (KG * 4) + n);
        const v4t a10 = *reinterpret_cast<const v4t*>(h + (long long)(y1 * Sn + x0) * (KG * 4) + n);
        const v4t a11 = *reinterpret_cast<const v4t*>(h + (long long)(y1 * Sn + x1) * (KG * 4) + n);
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[i] = (1.0f - fy) * ((1.0f - fx) * to_f(a00[i]) + fx * to_f(a01[i])) +
                 fy * ((1.0f - fx) * to_f(a10[i]) + fx * to_f(a11[i]));
          v[i] = in ? v[i] : 0.0f;
        }
        *reinterpret_cast<float4*>(&s_x[pix * CS + 4 + n]) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
    // pyramid layer, periphery crop and the channel of ones
    if (tid < 180) {
      const int y = oy + tid / 18 - 1, x = ox + tid % 18 - 1;
      float v[4] = {0.0f, 0.0f, 0.0f, 0.0f}, w[4] = {0.0f, 0.0f, 0.0f, 0.0f};
      if (y >= 0 && y < S && x >= 0 && x < S) {
        const float* p = pyr + d.pyr_off[k] + ((long long)y * S + x) * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = p[i];
        if (d.has_p) {
          const float* q = periph + (long long)d.view[k] * 3 * plane +
                           (long long)(dec_y0(d, k) + y) * d.W + (dec_x0(d, k) + x);
#pragma unroll
          for (int i = 0; i < 3; ++i) w[i] = q[i * plane];
        }
        w[3] = 1.0f;
      }
      *reinterpret_cast<float4*>(&s_x[tid * CS]) = make_float4(v[0], v[1], v[2], v[3]);
      *reinterpret_cast<float4*>(&s_x[tid * CS + 4 + KG * 4]) = make_float4(w[0], w[1], w[2], w[3]);
    }
#pragma unroll
    for (int e = tid; e < 128 * 8; e += 256) {
      const int pix = e >> 3, q = e & 7;
      const int y = oy + (pix >> 4), x = ox + (pix & 15);
      float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (y < S && x < S)
        v = *reinterpret_cast<const float4*>(dpre + d.pre_off[k] +
                                             ((long long)y * S + x) * d.nout + rg * 32 + q * 4);
      *reinterpret_cast<float4*>(&s_g[pix * kWgRows + q * 4]) = v;
    }
    __syncthreads();
#pragma unroll 2
    for (int ks = 0; ks < 32; ++ks) {
      const float a0 = s_g[(ks * 4 + kq) * kWgRows + col];
      const float a1 = s_g[(ks * 4 + kq) * kWgRows + 16 + col];
      const float* xb = &s_x[((ks >> 2) * 18 + (ks & 3) * 4 + kq) * CS + col];
      float bv[NQ];
#pragma unroll
      for (int i = 0; i < NQ; ++i) bv[i] = xb[off[i]];
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        acc[0][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, bv[i], acc[0][i], 0, 0, 0);
        acc[1][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, bv[i], acc[1][i], 0, 0, 0);
      }
    }
  }
  // lane (col, kq) holds rows 4 kq + r of padded channel 16 ct + col
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int q = wave + 4 * i;
    if (q >= 9 * NT) break;
    const int tap = q / NT, n = (q - tap * NT) * 16 + col;
    const int oc = pad_to_orig(n, d.kn, d.kpn, d.has_p);
    const bool ones = tap == 4 && n == 4 + d.kpn + 3;
    if (oc < 0 && !ones) continue;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ch = rg * 16 + 4 * kq + r;
        if (ch >= d.width) continue;
        const int row = m ? d.width + ch : ch;
        atomicAdd(ones ? &db[row] : &dw[((long long)row * 9 + tap) * d.cin + oc], acc[m][i][r]);
      }
  }
}

// The level's tiles of TH rows x 16 columns.
static int level_tiles(DecLevel* d, int TH) {
  int tb = 0;
  for (int k = 0; k < d->n_crops; ++k) {
    d->tile_base[k] = tb;
    d->tiles_x[k] = (d->S[k] + 15) / 16;
    tb += d->tiles_x[k] * ((d->S[k] + TH - 1) / TH);
  }
  d->tile_base[d->n_crops] = tb;
  return tb;
}

// 16-row tiles where they still give every compute unit four workgroups,
// 8-row tiles below (a level of 64 tiles would leave most of the chip idle).
template <int NT>
static hipError_t launch_dgrad(DecLevel d, const float* dpre, const float* wb, float* dpyr,
                               float* dx, float* dper, hipStream_t st) {
  int tiles = level_tiles(&d, 16);
  if (tiles >= 4 * device_cus()) {
    hipLaunchKernelGGL((k_dec_dgrad<NT, 4>), dim3(tiles), dim3(256), 0, st, d, dpre, wb, dpyr, dx,
                       dper);
  } else {
    tiles = level_tiles(&d, 8);
    hipLaunchKernelGGL((k_dec_dgrad<NT, 2>), dim3(tiles), dim3(256), 0, st, d, dpre, wb, dpyr, dx,
                       dper);
  }
  return hipGetLastError();
}

// As many workgroups per compute unit as the LDS holds (three up to three
// channel tiles, two above), so that one's loads run under another's matrix
// steps; fewer where there are not that many pixel tiles.
template <typename T, int NT>
static hipError_t launch_wgrad(DecLevel d, const float* pyr, const float* periph, const T* hn,
                               const float* dpre, float* dw, float* db, hipStream_t st) {
  const int tiles = level_tiles(&d, 8), groups = d.nout / 32;
  const int blocks = std::max(1, std::min(tiles, (NT <= 3 ? 3 : 2) * device_cus() / groups));
  hipLaunchKernelGGL((k_dec_wgrad<T, NT>), dim3(blocks, groups), dim3(256), wg_smem<NT>(), st, d,
                     pyr, periph, hn, dpre, dw, db);
  return hipGetLastError();
}

template <typename T>
static vrs_status decode_bwd_impl(const DecPlan& P, const float* pyramid, int levels,
                                  const float* periph, const KViews& kv, const vrs_crop* crops,
                                  int n_crops, const vrs_crop_place* place,
                                  const float* weights, const float* d_fovea,
                                  float* d_pyr, float* d_per, float* d_w, void* ws,
                                  hipStream_t st) {
  {
    PackBwdArgs pa;
    pa.n = P.nd;
    long long s = 0;
    for (int l = 0; l < P.nd; ++l) {
      pa.K[l] = P.K[l];
      pa.kn[l] = l + 1 < P.nd ? P.K[l + 1] : 0;
      pa.kpn[l] = l + 1 < P.nd ? P.kp[l + 1] : 0;
      pa.cin[l] = P.cin[l];
      pa.w[l] = weights + P.w_off[l];
      pa.wb[l] = at<float>(ws, P.wb[l]);
      pa.start[l] = s;
      s += P.wb_elems(l);
    }
    pa.start[P.nd] = s;
    hipLaunchKernelGGL(k_dec_pack_bwd, dim3((unsigned)std::min<long long>(1024, (s + 255) / 256)),
                       dim3(256), 0, st, pa);
    VRS_LAUNCH_CHECK();
  }
  float *dpre = at<float>(ws, P.pre), *dx = at<float>(ws, P.dx);
  for (int l = 0; l < P.nd; ++l) {
    DecLevel d;
    int blocks = 0;
    level_args(P, l, crops, n_crops, kv, levels, place, &d, &blocks);
    // the level's pre-activations again (the forward's h_l stay valid)
    const T* hn = l + 1 < P.nd ? at<T>(ws, P.h[l + 1]) : nullptr;
    VRS_HIP_CHECK(launch_conv<T>(d, 2 * P.kp[l] / 16, blocks, pyramid, periph, hn,
                                 at<T>(ws, P.wp[l]), at<float>(ws, P.bp[l]), at<T>(ws, P.h[l]),
                                 dpre, HeadFuse{}, st));
    GateArgs ga;
    ga.n_crops = n_crops;
    ga.kp = P.kp[l];
    ga.K = P.K[l];
    long long p = 0, o = 0;
    for (int k = 0; k < n_crops; ++k) {
      ga.S[k] = d.S[k];
      ga.pix_base[k] = p;
      ga.out_base[k] = o;
      p += (long long)d.S[k] * d.S[k];
      o += 3LL * d.S[k] * d.S[k];
    }
    ga.pix_base[n_crops] = p;
    const int per = 256 / (ga.kp / 4);
    if (l == 0) {
      // few workgroups: each ends with an atomic per head weight
      const int gb = (int)std::min<long long>(8 * device_cus(), (p + per - 1) / per);
      hipLaunchKernelGGL((k_dec_gate_bwd<T, true>), dim3(gb), dim3(256), 0, st, ga, dpre, nullptr,
                         at<T>(ws, P.h[0]), weights + P.head_w, d_fovea,
                         d_w ? d_w + P.head_w : nullptr, d_w ? d_w + P.head_b : nullptr);
    } else {
      const int gb = (int)std::min<long long>(16384, (p + per - 1) / per);
      hipLaunchKernelGGL((k_dec_gate_bwd<T, false>), dim3(gb), dim3(256), 0, st, ga, dpre, dx,
                         (const T*)nullptr, nullptr, nullptr, nullptr, nullptr);
    }
    VRS_LAUNCH_CHECK();
    const float* wb = at<float>(ws, P.wb[l]);
    float* dw = d_w ? d_w + P.w_off[l] : nullptr;
    float* db = d_w ? d_w + P.b_off[l] : nullptr;
    auto level = [&](auto nt) -> hipError_t {
      constexpr int NT = decltype(nt)::value;
      if (dw) {
        const hipError_t e = launch_wgrad<T, NT>(d, pyramid, periph, hn, dpre, dw, db, st);
        if (e != hipSuccess) return e;
      }
      return launch_dgrad<NT>(d, dpre, wb, d_pyr, dx, d_per, st);
    };
    switch (d.kpn / 16 + 1) {
      case 1: VRS_HIP_CHECK(level(std::integral_constant<int, 1>{})); break;
      case 2: VRS_HIP_CHECK(level(std::integral_constant<int, 2>{})); break;
      case 3: VRS_HIP_CHECK(level(std::integral_constant<int, 3>{})); break;
      case 4: VRS_HIP_CHECK(level(std::integral_constant<int, 4>{})); break;
      default: VRS_HIP_CHECK(level(std::integral_constant<int, 5>{})); break;
    }
  }
  return VRS_OK;
}

}  // namespace vrs

extern "C" vrs_status vrs_decode_fovea_backward(const float* pyramid, int levels,
                                                const float* rgb_periphery, const vrs_view* views,
                                                int n_views, const vrs_crop* crops, int n_crops,
                                                const vrs_crop_place* place,
                                                const float* weights, const vrs_decoder_desc* dd,
                                                const float* d_fovea, float* d_pyramid,
                                                float* d_rgb_periphery, float* d_weights,
                                                void* ws, size_t ws_bytes, void* stream) {
  DecPlan P;
  KViews kv;
  if (!make_views(views, n_views, &kv) || !dec_plan(dd, crops, n_crops, &P)) return VRS_EINVAL;
  if (levels < P.nd || levels > VRS_MAX_LEVELS || !pyramid || !rgb_periphery || !weights ||
      !d_fovea || !ws || ws_bytes < P.total)
    return VRS_EINVAL;
  if (dd->in_ch != 4) return VRS_EUNSUPPORTED;
  if (!dec_crops_ok(views, n_views, crops, n_crops, levels, place)) return VRS_EINVAL;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (P.dtype == VRS_BF16)
    return decode_bwd_impl<__bf16>(P, pyramid, levels, rgb_periphery, kv, crops, n_crops, place,
                                   weights, d_fovea, d_pyramid, d_rgb_periphery, d_weights, ws,
                                   st);
  return decode_bwd_impl<float>(P, pyramid, levels, rgb_periphery, kv, crops, n_crops, place,
                                weights, d_fovea, d_pyramid, d_rgb_periphery, d_weights, ws, st);
}
