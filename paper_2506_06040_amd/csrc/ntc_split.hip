// FP32 decode on the BF16 matrix cores with split operands (the method of
// G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", arXiv 1904.06376).
//
// gfx950 multiplies FP32 matrices at 157 TFLOP/s and BF16 ones at 16 times
// that. An FP32 number is the sum of three BF16 numbers (8 significant bits
// each), so a product of two is the sum of nine BF16 products, of which six
// matter: with a = a1 + a2 + a3 and b = b1 + b2 + b3 (each term at most 2^-8
// of the one before), a2 b3, a3 b2 and a3 b3 are below 2^-24 |a b|. The six
// are exact in the FP32 accumulators' inputs and are added there smallest
// first. Activations are cut (the parts are the number's own bits, so the
// three add up exactly in the normal range), weights are rounded (the dropped terms then have no
// common sign). Against 64-bit results the error is that of the FP32 chain or
// smaller: a layer of 64 inputs rounds 24 times, not 64.
//
// Matrix time falls to 6 / 16 of FP32 products and the splitting costs about
// 6 vector instructions per activation. The two bound it: matrix cores 62% and
// VALU 68% busy, LDS 25%. 1920x1080, 14-64-64-64-8: 206 us; 727 with a lane per
// pixel and scalar-cache weights.
//
// Workgroups of kSplitWaves wavefronts share the split weights in LDS (22 KB
// per part for 14-64-64-64-8: they do not fit the registers three times
// over); a wavefront walks spans of 64 kSplitTiles pixels. BC1 texels are
// staged as FP16 numerators, which FP16 holds exactly, and blended in FP32
// as everywhere in the FP32 path.
//
// Numbers that could leave FP32's range (or are infinite or NaN) must not be
// split: infinity minus its leading part is NaN. Nor may small numbers be whose
// lower parts, below BF16's normal range, matter: that range ends where FP32's
// does, so a part of at most 2^-126 may be lost, and where a layer's numbers are
// all that small, and the next layer's weights large, it is many units in the
// last place. Bounds from the largest weight and bias of every layer and |u|,
// |v| <= 2^20 decide per network (split_setup), the coordinates (and float
// latents) per pixel; what fails is decoded by a
// second walk with the FP32 matrix instructions (exact_pixels), pixel by
// pixel, so that a pixel's result does not depend on its neighbours. That walk
// takes the weights as they stand from LDS, where they replace their parts once
// the workgroup has finished the first walk: no weight is fetched per tile (a
// load per product from the image: 1172 in place of 279 us, and registers that
// the first walk spilled). It is bound by the FP32 products, 112 of 64 cycles per
// 32 pixels of 14-64-64-8; 1920x1080 pixels of networks that are all out of range:
// 14-64-64-8 279 us, 14-64-64-64-8 405 (plain FMAs, a lane per pixel: 424, 697).
#include <hip/hip_runtime.h>

#include "ntc_device.hpp"
#include "ntc_internal.hpp"
#include "ntc_mfma_tile.hpp"

namespace ntc {

constexpr int kSplitWaves = 12;    // wavefronts per workgroup, three per SIMD
constexpr int kSplitTiles = 2;    // 64-pixel sub-spans per span
constexpr int kSplitStage = 640;  // staged texels per wavefront (8 bytes each)

template <int HP, int NL>
struct SplitMap {
  static constexpr int MT = (HP + 31) / 32, KS = HP / 16;
  static constexpr int F = MT + (NL - 2) * MT * KS + KS;  // operand fragments (1 KB each) of one part
  __device__ static constexpr int frag(int l, int m, int c) {
    return l == 0 ? m : (l < NL - 1 ? MT + ((l - 1) * MT + m) * KS + c : MT + (NL - 2) * MT * KS + c);
  }
  // byte offsets
  static constexpr int oBias = 3 * F * 1024;             // hidden layers 1 .. NL - 2: [l][m][h][16] floats
  static constexpr int oOut = oBias + (NL - 2) * MT * 128;  // output biases [16]
  static constexpr int oMax = oOut + 64;                 // largest |weight|, |bias| per layer [2 kMaxLayers], second walk needed
  static constexpr int oTab = (oMax + 4 * (2 * kMaxLayers + 1) + 15) & ~15;
  static constexpr int oRec = oTab + LevelTab::kLevelEntries * 16;
  static constexpr int oStage = oRec + kSplitWaves * 2 * kMaxLevels * 16;
  static constexpr int total(bool bc1) { return oStage + (bc1 ? kSplitWaves * kSplitStage * 8 : 0); }
};

// Two numbers into the three parts, cut: dword p holds part p of both. (The
// remainder as a BF16 dot product, one instruction in place of two, is
// slower: 290 against 263 us at that stage of the case above.)
__device__ __forceinline__ void cut3(float a, float b, unsigned (&p)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
    p[i] = __builtin_amdgcn_perm(ub, ua, 0x07060302u);
    a -= __uint_as_float(ua & 0xffff0000u);
    b -= __uint_as_float(ub & 0xffff0000u);
  }
}

// Column of the FP32 image's layer-l matrix fed to element e of lane half h
// in K-step c (-1: padding; first layer: -2 the constant 1, see
// slot order in pixel_operands).
__device__ __forceinline__ int split_col(int n_levels, int l, int c, int h, int e) {
  if (l > 0) return 32 * (c >> 1) + 16 * (c & 1) + 8 * (e >> 2) + 4 * h + (e & 3);
  if ((e & 3) < 3) {
    const int lvl = 2 * h + (e >> 2);
    return lvl < n_levels ? 3 * lvl + (e & 3) : -1;
  }
  if (h == 0) return 3 * n_levels + (e >> 2);
  return e == 3 ? -2 : -1;
}

// Element of layer l's matrix (column -2: of its bias) in the FP32 image, zero
// outside it, without branches.
__device__ __forceinline__ float split_weight(const DecodeArgs &a, const uint8_t *packed, int l, int row, int col) {
  const PackLayout &L = a.lay;
  const int r = min(row, L.rows_pad[l] - 1), c = min(max(col, 0), L.cols_pad[l] - 1);
  const unsigned at = col == -2 ? L.b_off[l] + 4 * r : L.w_off[l] + 4 * (r * L.cols_pad[l] + c);
  const float w = gload(reinterpret_cast<const float *>(packed + at));
  return r == row && (col == -2 || c == col) ? w : 0.0f;
}

// *m to at least big; NaN counts as infinite.
__device__ __forceinline__ void note_max(unsigned *m, float big) {
  atomicMax(m, big == big ? __float_as_uint(big) : 0x7f800000u);
}

// Weights into LDS, a fragment (layer l, rows 32 m .., K-step c) per wavefront
// at a time: the three parts of each, [part][fragment][lane], or as they stand
// (EXACT), [fragment][half][lane]. The parts note the largest weight of each layer.
template <int HP, int NL, bool EXACT>
__device__ __forceinline__ void fill_weights(const DecodeArgs &a, uint8_t *lds, int tid) {
  using M = SplitMap<HP, NL>;
  constexpr int kHidden = M::MT * M::KS;
  const int lane = tid & 63, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  u32x4_t *w = reinterpret_cast<u32x4_t *>(lds);
#pragma unroll 1
  for (int f = wave; f < M::F; f += kSplitWaves) {
    const int l = f < M::MT ? 0 : (f < M::F - M::KS ? 1 + (f - M::MT) / kHidden : NL - 1);
    const int g = f < M::MT ? 0 : (f - M::MT) % kHidden;  // m KS + c of a hidden layer
    const int m = l == 0 ? f : (l == NL - 1 ? 0 : g / M::KS), c = l == NL - 1 ? f - (M::F - M::KS) : g % M::KS;
    const int row = 32 * m + (lane & 31);
    float v[8], big = 0.0f;
    if (l == 0) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = split_weight(a, a.packed, 0, row, split_col(a.lat.n_levels, 0, 0, h, e));
    } else {
      // columns 4 h .. 4 h + 3 and 8 further on, of rows and columns that exist
      const int col = 32 * (c >> 1) + 16 * (c & 1) + 4 * h;
      const int cols = a.lay.cols_pad[l];
      const float *p = reinterpret_cast<const float *>(a.packed + a.lay.w_off[l]) + min(row, a.lay.rows_pad[l] - 1) * cols;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const f32x4 q = gload(reinterpret_cast<const f32x4 *>(p + min(col + 8 * j, cols - 4)));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * j + e] = row < a.lay.rows_pad[l] && col + 8 * j < cols ? q[e] : 0.0f;
      }
    }
    if constexpr (EXACT) {
      f32x4 *q = reinterpret_cast<f32x4 *>(lds) + 2 * f * 64 + lane;
      q[0] = (f32x4){v[0], v[1], v[2], v[3]};
      q[64] = (f32x4){v[4], v[5], v[6], v[7]};
      continue;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) big = fmaxf(big, v[e] == v[e] ? fabsf(v[e]) : __builtin_inff());
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      bf16x8_t q;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        q[e] = (__bf16)v[e];
        v[e] -= (float)q[e];
      }
      w[(p * M::F + f) * 64 + lane] = __builtin_bit_cast(u32x4_t, q);
    }
    note_max(reinterpret_cast<unsigned *>(lds + M::oMax) + l, big);
  }
}

// Weights, biases and level table into LDS; returns whether the network's
// numbers stay in range: no sum of any layer passes 2^120, and the parts lost
// below the normal range (with products below it, at most 2^-122 per operand)
// change no output's pre-activation by more than 2^-30, a 64th of what FP32
// rounds an output by. (Latents are at most 1 in BC1 images, float latents are
// checked with the coordinates.) Rolled loops: a short batch pays for
// every instruction line fetched.
template <int HP, int NL>
__device__ __forceinline__ bool split_setup(const DecodeArgs &a, uint8_t *lds, int tid) {
  using M = SplitMap<HP, NL>;
  unsigned *mx = reinterpret_cast<unsigned *>(lds + M::oMax);
  if (tid <= 2 * kMaxLayers) mx[tid] = 0u;
  __syncthreads();
  if (tid < kMaxLevels) {  // LevelTab::fill, a lane per level
    const LevelArgs &L = a.lat.lv[tid];
    const unsigned long long p = (unsigned long long)L.bc1;
    f32x4 *tab = reinterpret_cast<f32x4 *>(lds + M::oTab) + 3 * tid;
    tab[0] = (f32x4){L.fw, L.sx - 0.5f, (float)(L.w - 2), __int_as_float(L.w)};
    tab[1] = (f32x4){L.fh, L.sy - 0.5f, (float)(L.h - 2), __int_as_float(L.h)};
    tab[2] = (f32x4){__uint_as_float((unsigned)p), __uint_as_float((unsigned)(p >> 32)), __int_as_float(L.bw), 0.0f};
  }
  fill_weights<HP, NL, false>(a, lds, tid);
  // biases (the first layer's is a weight of the constant 1)
#pragma unroll 1
  for (int i = tid; i < (NL - 2) * M::MT * 32 + 16; i += 64 * kSplitWaves) {
    const bool out = i >= (NL - 2) * M::MT * 32;
    const int g = i / 32, e = i % 32;
    const int l = out ? NL - 1 : g / M::MT + 1;
    const int row = out ? i - (NL - 2) * M::MT * 32 : 32 * (g % M::MT) + 8 * ((e & 15) >> 2) + 4 * (e >> 4) + (e & 3);
    const float b = split_weight(a, a.packed, l, row, -2);
    reinterpret_cast<float *>(lds + M::oBias)[i] = b;
    note_max(mx + kMaxLayers + l, fabsf(b));
  }
  __syncthreads();
  float b = 0x1p20f;  // no input of layer l passes it
  float lost = 0.0f;  // what the inputs' sums may be off by for parts that were lost
  bool in_range = true;
#pragma unroll 1
  for (int l = 0; l < NL; ++l) {
    const float w = __uint_as_float(mx[l]);
    lost = 64.0f * (w * (lost + 0x1p-122f) + (b + 1.0f) * 0x1p-122f);
    b = 64.0f * w * b + __uint_as_float(mx[kMaxLayers + l]);
    in_range = in_range && b < 0x1p120f;
  }
  return __builtin_amdgcn_readfirstlane(in_range && lost <= 0x1p-30f ? 1 : 0) != 0;
}

// max(z, 0), 0 for NaN (see relu() of the training kernels).
__device__ __forceinline__ float relu_f32(float z) {
  float inf;
  asm("s_mov_b32 %0, 0x7f800000" : "=s"(inf));
  return __builtin_amdgcn_fmed3f(z, 0.0f, inf);
}

// acc += W X over one K-step, the six products smallest first.
__device__ __forceinline__ f32x16 mma6(const u32x4_t *w, int stride, const bf16x8_t (&x)[3], f32x16 acc) {
  bf16x8_t p[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) p[i] = __builtin_bit_cast(bf16x8_t, w[i * stride]);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[2], x[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[1], x[1], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[0], x[2], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[1], x[0], acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[0], x[1], acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[0], x[0], acc, 0, 0, 0);
}

// Samples of all levels of one pixel as K-slots (see pixel_operands): xl for
// lane half 0, xh for lane half 1.
__device__ __forceinline__ void put_slots(float (&xl)[8], float (&xh)[8], const float3 (&c)[kMaxLevels], float u,
                                          float v) {
#pragma unroll
  for (int k = 0; k < kMaxLevels; ++k) put_level(xl, xh, k, c[k]);
  xl[3] = u;
  xl[7] = v;
  xh[3] = 1.0f;
  xh[7] = 0.0f;
}

__device__ __forceinline__ float3 numer_values(float3 c) {
  return make_float3(c.x * kInvDenRB, c.y * kInvDenG, c.z * kInvDenRB);
}

__device__ __forceinline__ float3 staged_level(const uint2 *t, int pitch, float fx, float fy) {
  const Tex16 t00 = tex16_from(t[0]), t10 = tex16_from(t[1]), t01 = tex16_from(t[pitch]), t11 = tex16_from(t[pitch + 1]);
  auto f3 = [](const Tex16 &q) { return make_float3((float)q.rg[0], (float)q.rg[1], (float)q.b1[0]); };
  return numer_values(blend4(f3(t00), f3(t10), f3(t01), f3(t11), fx, fy));
}

__device__ __forceinline__ float3 direct_level(const TabLevel &L, float u, float v, int mode) {
  int i0, i1, j0, j1;
  float fx, fy;
  direct_taps<kEitherMode>(L, u, v, mode, i0, i1, j0, j1, fx, fy);
  auto at = [&](int i, int j) {
    const uint2 b = gload2u(L.bc1 + (int64_t)(j >> 2) * L.bw + (i >> 2));
    const uint32_t p = bc1_numer(b.x, b.y, (uint32_t)(((j & 3) << 2) | (i & 3)));
    return make_float3(numer_r(p), numer_g(p), numer_b(p));
  };
  return numer_values(blend4(at(i0, j0), at(i1, j0), at(i0, j1), at(i1, j1), fx, fy));
}

// Float latents: the loads of all levels in flight together. Levels past
// n_levels (which mirror level 0) give zeros: their weights are zero, but a
// texel of theirs may not be finite.
__device__ __forceinline__ void grid_levels(const LatArgs &lat, float u, float v, float3 (&c)[kMaxLevels]) {
  float fx[kMaxLevels], fy[kMaxLevels];
  int i0[kMaxLevels], i1[kMaxLevels], j0[kMaxLevels], j1[kMaxLevels];
#pragma unroll
  for (int k = 0; k < kMaxLevels; ++k) {
    float x = fmaf(u, lat.lv[k].fw, -0.5f) + lat.lv[k].sx;
    float y = fmaf(v, lat.lv[k].fh, -0.5f) + lat.lv[k].sy;
    x = fminf(fmaxf(x, -16777216.0f), 16777216.0f);
    y = fminf(fmaxf(y, -16777216.0f), 16777216.0f);
    const float xf = floorf(x), yf = floorf(y);
    fx[k] = x - xf;
    fy[k] = y - yf;
    i0[k] = (int)xf;
    j0[k] = (int)yf;
  }
  if (lat.address == 1) {
#pragma unroll
    for (int k = 0; k < kMaxLevels; ++k) {
      const int w = lat.lv[k].w, h = lat.lv[k].h;
      i0[k] = wrap_near(i0[k], w, __builtin_amdgcn_rcpf((float)w));
      j0[k] = wrap_near(j0[k], h, __builtin_amdgcn_rcpf((float)h));
      i1[k] = i0[k] + 1 == w ? 0 : i0[k] + 1;
      j1[k] = j0[k] + 1 == h ? 0 : j0[k] + 1;
    }
  } else {
#pragma unroll
    for (int k = 0; k < kMaxLevels; ++k) {
      i1[k] = address_coord(i0[k] + 1, lat.lv[k].w, 0);
      j1[k] = address_coord(j0[k] + 1, lat.lv[k].h, 0);
      i0[k] = address_coord(i0[k], lat.lv[k].w, 0);
      j0[k] = address_coord(j0[k], lat.lv[k].h, 0);
    }
  }
  float t[kMaxLevels][4][3];
#pragma unroll
  for (int k = 0; k < kMaxLevels; ++k)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float *p =
          lat.lv[k].grid + ((int64_t)((q >> 1) ? j1[k] : j0[k]) * lat.lv[k].w + ((q & 1) ? i1[k] : i0[k])) * 3;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) t[k][q][ch] = p[ch];
    }
#pragma unroll
  for (int k = 0; k < kMaxLevels; ++k) {
    c[k] = blend4(make_float3(t[k][0][0], t[k][0][1], t[k][0][2]), make_float3(t[k][1][0], t[k][1][1], t[k][1][2]),
                  make_float3(t[k][2][0], t[k][2][1], t[k][2][2]), make_float3(t[k][3][0], t[k][3][1], t[k][3][2]),
                  fx[k], fy[k]);
    if (k >= lat.n_levels) c[k] = make_float3(0.0f, 0.0f, 0.0f);
  }
}

// Outputs of one 32-pixel tile: rows 8 j + 4 h + r of pixel px (keep: of the
// lanes whose pixel is to be written).
__device__ __forceinline__ void split_store(const DecodeArgs &a, const f32x16 &z, const float *ob, int64_t px, int h,
                                            bool keep) {
  if (px >= a.n || !keep) return;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j == 1 && a.n_out <= 8) break;
    const int row0 = 8 * j + 4 * h;
    float f[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) f[r] = 1.0f / (1.0f + expf(-(z[4 * j + r] + ob[row0 + r])));
    if (row0 >= a.n_out) continue;
    if (a.out_f16) {
      _Float16 *o = reinterpret_cast<_Float16 *>(a.out) + px * a.n_out + row0;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (row0 + r < a.n_out) o[r] = (_Float16)f[r];
    } else {
      float *o = reinterpret_cast<float *>(a.out) + px * a.n_out + row0;
      if ((a.n_out & 3) == 0) {
        __builtin_nontemporal_store((f32x4){f[0], f[1], f[2], f[3]}, reinterpret_cast<f32x4 *>(o));
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (row0 + r < a.n_out) o[r] = f[r];
      }
    }
  }
}

// Pre-activations of the outputs of one 32-pixel tile by FP32 matrix products
// (w: this lane's weights as they stand, bias: the hidden layers' biases).
// 32x32x2 products take K-element e of a fragment as the split ones do.
template <int HP, int NL>
__device__ __forceinline__ void exact_tile(const f32x4 *w, const float *bias, int h, const float (&x)[8], f32x16 &z) {
  using M = SplitMap<HP, NL>;
  constexpr int MT = M::MT, KS = M::KS;
  f32x16 in[MT], out[MT];
  const f32x16 zero = {};
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    out[m] = zero;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f32x4 q = w[(2 * M::frag(0, m, 0) + j) * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e) out[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(q[e], x[4 * j + e], out[m], 0, 0, 0);
    }
  }
#pragma unroll 1
  for (int l = 1; l < NL; ++l) {
    const f32x4 *wl = w + 2 * (MT + (l - 1) * MT * KS) * 64;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int i = 0; i < 16; ++i) in[m][i] = relu_f32(out[m][i]);
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      if (m > 0 && l == NL - 1) break;
      out[m] = zero;
      if (l < NL - 1) {
        const f32x4 *b = reinterpret_cast<const f32x4 *>(bias + ((l - 1) * MT + m) * 32 + 16 * h);
        const f32x4 b0 = b[0], b1 = b[1], b2 = b[2], b3 = b[3];
        out[m] = (f32x16){b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3],
                          b2[0], b2[1], b2[2], b2[3], b3[0], b3[1], b3[2], b3[3]};
      }
#pragma unroll
      for (int c = 0; c < KS; ++c)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const f32x4 q = wl[(2 * (m * KS + c) + j) * 64];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            out[m] = __builtin_amdgcn_mfma_f32_32x32x2f32(q[e], in[c >> 1][8 * (c & 1) + 4 * j + e], out[m], 0, 0, 0);
        }
    }
  }
  z = out[0];
}

// Whether a pixel's numbers may be split (see the head of this file).
template <bool BC1>
__device__ __forceinline__ bool may_split(const float (&xl)[8], const float (&xh)[8]) {
  bool ok = fabsf(xl[3]) <= 0x1p20f && fabsf(xl[7]) <= 0x1p20f;
  if constexpr (!BC1) {
#pragma unroll
    for (int e = 0; e < 8; ++e) ok = ok && fabsf(xl[e]) <= 0x1p20f && fabsf(xh[e]) <= 0x1p20f;
  }
  return ok;
}

// A second walk over the samples: pixels that may not be split (all: every
// pixel). Wavefront `it0` of `step` takes the 64-pixel tiles of its spans.
template <int HP, int NL, bool BC1>
__device__ __forceinline__ void exact_pixels(const DecodeArgs &a, const uint8_t *lds, const float *ob, int64_t it0,
                                             int64_t step, int spx, bool all) {
  using M = SplitMap<HP, NL>;
  const f32x4 *ltab = reinterpret_cast<const f32x4 *>(lds + M::oTab);
  const int lane = threadIdx.x & 63, h = lane >> 5, c32 = lane & 31;
  const int per = spx / 64;
  auto load_uv = [&](int64_t it) { return a.uv[min(it * 64 + lane, a.n - 1)]; };
  float2 uv_next = load_uv(it0 * per);
  int64_t next;
#pragma unroll 1
  for (int64_t it = it0 * per; it * 64 < a.n; it = next) {
    next = it + (it % per == per - 1 ? (step - 1) * per + 1 : 1);
    const float2 uv = uv_next;
    uv_next = load_uv(next);
    float xl[8], xh[8];
    float3 c[kMaxLevels];
    if constexpr (BC1) {
#pragma unroll
      for (int k = 0; k < kMaxLevels; ++k) {
        TabLevel L;
        L.read(ltab, k);
        c[k] = direct_level(L, uv.x, uv.y, a.lat.address);
      }
    } else {
      grid_levels(a.lat, uv.x, uv.y, c);
    }
    put_slots(xl, xh, c, uv.x, uv.y);
    const int bad = all || !may_split<BC1>(xl, xh);
    const unsigned long long any = __builtin_amdgcn_ballot_w64(bad != 0);
    if (any == 0) continue;
    float x0[8], x1[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(xl[e]), __float_as_uint(xh[e]), false, false);
      x0[e] = __uint_as_float(r[0]);
      x1[e] = __uint_as_float(r[1]);
    }
#pragma unroll 1
    for (int t = 0; t < 2; ++t) {
      f32x16 z;
      const int off = opaque_zero(2 * (int)it + t);  // nothing of LDS is held in registers across tiles
      exact_tile<HP, NL>(reinterpret_cast<const f32x4 *>(lds) + lane + off,
                         reinterpret_cast<const float *>(lds + M::oBias) + off, h, x0, z);
      split_store(a, z, ob, it * 64 + 32 * t + c32, h, (any >> (32 * t + c32)) & 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) x0[e] = x1[e];
    }
  }
}

template <int HP, int NL, bool BC1>
__global__ __launch_bounds__(64 * kSplitWaves) __attribute__((amdgpu_waves_per_eu(kSplitWaves / 4)))
void decode_split_kernel(DecodeArgs a) {
  using M = SplitMap<HP, NL>;
  constexpr int MT = M::MT, KS = M::KS, ST = kSplitTiles;
  extern __shared__ uint8_t split_lds[];
  uint8_t *lds = split_lds;
  const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c32 = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  f32x4 *ltab = reinterpret_cast<f32x4 *>(lds + M::oTab);
  f32x4 *srec = reinterpret_cast<f32x4 *>(lds + M::oRec) + wave * 2 * kMaxLevels;
  f32x4 *stage = reinterpret_cast<f32x4 *>(lds + M::oStage + (BC1 ? wave * kSplitStage * 8 : 0));

  // wavefront w of workgroup b takes spans b + w * groups, ...: a short batch
  // spreads over the compute units first, and over more wavefronts as spans of
  // 64 pixels (a.n_tiles: pixels per span)
  const int spx = (int)a.n_tiles;
  const int64_t n_spans = (a.n + spx - 1) / spx;
  auto span_end = [&](int64_t s) { return min((s + 1) * spx, a.n); };
  const int64_t step = (int64_t)gridDim.x * kSplitWaves;
  const int64_t it0 = (int64_t)wave * gridDim.x + blockIdx.x;
  const float *ob = reinterpret_cast<const float *>(lds + M::oOut);
  SpanUv<ST> uvs;
  const bool bounded = split_setup<HP, NL>(a, lds, tid);
  if (it0 < n_spans) uvs.load(a.uv, it0 * spx, span_end(it0));
  bool left = false;  // some pixel may not be split
  for (int64_t it = bounded ? it0 : n_spans; it < n_spans; it += step) {
    const int64_t first = it * spx;
    const int span = (int)(span_end(it) - first);
    float u[ST], v[ST];
#pragma unroll
    for (int q = 0; q < ST; ++q) {
      u[q] = uvs.u[q];
      v[q] = uvs.v[q];
    }
    int kbw[kMaxLevels], kbase[kMaxLevels];
    bool in_unit, interior, staged = false;
    if constexpr (BC1)
      staged = a.lat.address == 0
                   ? stage_span<ST, true, true, kClampOnly>(a, u, v, stage, ltab, srec, (int)first, kbw, kbase, in_unit,
                                                            interior)
                   : stage_span<ST, true, true, kWrapOnly>(a, u, v, stage, ltab, srec, (int)first, kbw, kbase, in_unit,
                                                           interior);
    if (it + step < n_spans) uvs.load(a.uv, (it + step) * spx, span_end(it + step));

#pragma unroll 1
    for (int q = 0; q < ST; ++q) {
      if (64 * q >= span) break;
      const float uq = u[0], vq = v[0];
#pragma unroll
      for (int i = 0; i + 1 < ST; ++i) {
        u[i] = u[i + 1];
        v[i] = v[i + 1];
      }
      // ---- features
      float xl[8], xh[8];
      {
        float3 c[kMaxLevels];
        if constexpr (BC1) {
          const f32x4 *tab = ltab + opaque_zero((int)first + q);
          if (staged) {
#pragma unroll
            for (int k = 0; k < kMaxLevels; ++k) {
              c[k] = make_float3(0.0f, 0.0f, 0.0f);
              if (k >= a.lat.n_levels) continue;
              TabLevel L;
              L.read(tab, k);
              int i0, j0;
              float fx, fy;
              if (a.lat.address != 0) {
                span_tap<kTapWrap>(uq, L.fw, L.cx, L.wm2, i0, fx);
                span_tap<kTapWrap>(vq, L.fh, L.cy, L.hm2, j0, fy);
              } else {
                span_tap<kTapClamp>(uq, L.fw, L.cx, L.wm2, i0, fx);
                span_tap<kTapClamp>(vq, L.fh, L.cy, L.hm2, j0, fy);
              }
              c[k] = staged_level(reinterpret_cast<const uint2 *>(stage) + kbase[k] + __mul24(j0, kbw[k]) + i0, kbw[k],
                                  fx, fy);
            }
          } else {
#pragma unroll
            for (int k = 0; k < kMaxLevels; ++k) {
              c[k] = make_float3(0.0f, 0.0f, 0.0f);
              if (k >= a.lat.n_levels) continue;
              TabLevel L;
              L.read(tab, k);
              c[k] = direct_level(L, uq, vq, a.lat.address);
            }
          }
        } else {
          grid_levels(a.lat, uq, vq, c);
        }
        put_slots(xl, xh, c, uq, vq);
      }
      const unsigned long long ok = __builtin_amdgcn_ballot_w64(may_split<BC1>(xl, xh));
      left = left || ok != ~0ull;
      const int64_t px = first + 64 * q + c32;
      // ---- operands of the two 32-pixel tiles
      bf16x8_t x[2][3];
      {
        u32x4_t lo[3], hi[3];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          unsigned p[3];
          cut3(xl[2 * e], xl[2 * e + 1], p);
#pragma unroll
          for (int i = 0; i < 3; ++i) lo[i][e] = p[i];
          cut3(xh[2 * e], xh[2 * e + 1], p);
#pragma unroll
          for (int i = 0; i < 3; ++i) hi[i][e] = p[i];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          x[0][i] = __builtin_bit_cast(bf16x8_t, lo[i]);
          x[1][i] = __builtin_bit_cast(bf16x8_t, hi[i]);
          swap_halves<PrecBF16>(x[0][i], x[1][i]);
        }
      }
      // ---- layers, one tile after the other
#pragma unroll 1
      for (int t = 0; t < 2; ++t) {
        const u32x4_t *w = reinterpret_cast<const u32x4_t *>(lds) + lane + opaque_zero((int)first + 2 * q + t);
        const float *bias = reinterpret_cast<const float *>(lds + M::oBias) + opaque_zero((int)first + 2 * q + t);
        f32x16 acc[MT];
        const f32x16 zero = {};
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m] = mma6(w + M::frag(0, m, 0) * 64, M::F * 64, x[0], zero);
#pragma unroll
        for (int i = 0; i < 3; ++i) x[0][i] = x[1][i];
        bf16x8_t hb[KS][3];
#pragma unroll
        for (int l = 1; l < NL; ++l) {
          // ReLU and the three parts of the next layer's input
#pragma unroll
          for (int c = 0; c < KS; ++c) {
            u32x4_t p4[3];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              unsigned p[3];
              const int o = 8 * (c & 1) + 2 * e;
              cut3(relu_f32(acc[c >> 1][o]), relu_f32(acc[c >> 1][o + 1]), p);
#pragma unroll
              for (int i = 0; i < 3; ++i) p4[i][e] = p[i];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) hb[c][i] = __builtin_bit_cast(bf16x8_t, p4[i]);
          }
          const int mts = l == NL - 1 ? 1 : MT;
#pragma unroll
          for (int m = 0; m < mts; ++m) {
            if (l < NL - 1) {
              const f32x4 *b = reinterpret_cast<const f32x4 *>(bias + ((l - 1) * MT + m) * 32 + 16 * h);
              const f32x4 b0 = b[0], b1 = b[1], b2 = b[2], b3 = b[3];
              acc[m] = (f32x16){b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3],
                                b2[0], b2[1], b2[2], b2[3], b3[0], b3[1], b3[2], b3[3]};
            } else {
              acc[m] = zero;
            }
#pragma unroll
            for (int c = 0; c < KS; ++c) acc[m] = mma6(w + M::frag(l, m, c) * 64, M::F * 64, hb[c], acc[m]);
          }
        }
        split_store(a, acc[0], ob + opaque_zero((int)first + 2 * q + t), px + 32 * t, h, (ok >> (32 * t + c32)) & 1);
      }
    }
  }
  // the second walk, with the weights as they stand in the place of their parts
  unsigned *again = reinterpret_cast<unsigned *>(lds + M::oMax) + 2 * kMaxLayers;
  if (left) *again = 1u;
  __syncthreads();
  if (bounded && *again == 0u) return;
  fill_weights<HP, NL, true>(a, lds, tid);
  __syncthreads();
  if (!bounded || left) exact_pixels<HP, NL, BC1>(a, lds, ob, it0, step, spx, !bounded);
}

template <int HP, bool BC1>
static hipError_t launch_split_hp(const DecodeArgs &a, int n_layers, int groups, hipStream_t st) {
  auto go = [&](auto kernel, int bytes) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(64 * kSplitWaves), bytes, st, a);
    return hipGetLastError();
  };
  switch (n_layers) {
    case 2: return go(decode_split_kernel<HP, 2, BC1>, SplitMap<HP, 2>::total(BC1));
    case 3: return go(decode_split_kernel<HP, 3, BC1>, SplitMap<HP, 3>::total(BC1));
    case 4: return go(decode_split_kernel<HP, 4, BC1>, SplitMap<HP, 4>::total(BC1));
    case 5: return go(decode_split_kernel<HP, 5, BC1>, SplitMap<HP, 5>::total(BC1));
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_decode_f32(DecodeArgs a, const MlpShape &s, int n_cus, hipStream_t st) {
  a.stage_cap = kSplitStage / 2;  // counted in 16-byte texels
  // Spans of 64 pixels where longer ones would leave wavefronts without work:
  // 65,536 pixels of 14-64-64-64-8 take 20 us against 29 with 128-pixel spans,
  // whose two sub-spans are one chain of 528 matrix instructions.
  const int64_t waves = (int64_t)n_cus * kSplitWaves;
  const int spx = a.n >= waves * 64 * kSplitTiles ? 64 * kSplitTiles : 64;
  a.n_tiles = spx;
  const int64_t spans = (a.n + spx - 1) / spx;
  const int groups = (int)(spans < n_cus ? spans : n_cus);
  if (a.lat.format == 0)
    return s.hid > 32   ? launch_split_hp<64, true>(a, s.n_layers, groups, st)
           : s.hid > 16 ? launch_split_hp<32, true>(a, s.n_layers, groups, st)
                        : launch_split_hp<16, true>(a, s.n_layers, groups, st);
  return s.hid > 32   ? launch_split_hp<64, false>(a, s.n_layers, groups, st)
         : s.hid > 16 ? launch_split_hp<32, false>(a, s.n_layers, groups, st)
                      : launch_split_hp<16, false>(a, s.n_layers, groups, st);
}

}  // namespace ntc
