// BC1 latents as trainable parameters (Sec. 3.2, Eqs. 1-3).
//
// During training the paper keeps every BC1 texture as floating-point
// tensors, endpoints and per-texel interpolation weights, and obtains the
// BC1 values by a sigmoid followed by quantisation to the field widths
// (5, 6, 5 bits for the endpoints, 2 bits for the weight), with the
// quantisation transparent to gradients. Here one level of W x H texels
// is a float array [H/4][W/4][22] of logits per block:
//   e0 (r, g, b), e1 (r, g, b), alpha[16] (texel (x, y) of the block at 4y + x).
// Codes: E = round(sigmoid(e) (2^b - 1)), w = round(sigmoid(alpha) 3), and
// the texel value per channel is ((3 - w) E0 + w E1) / (3 (2^b - 1)): the
// four-colour BC1 palette, so the same texels come out of real BC1 blocks
// (ntc_qat_export_bc1) through the ordinary decoder.
//
// A code is decided by comparing the logit with the FP32 logits of the
// rounding midpoints (k + 1/2) / (2^b - 1), computed on the host in double
// precision: sigmoid is monotonic, so this is the rounding of the sigmoid
// without evaluating it, and the decision depends only on the input and a
// correctly rounded constant.
#include <hip/hip_runtime.h>

#include <cmath>

#include "ntc_device.hpp"
#include "ntc_internal.hpp"

namespace ntc {

namespace {

constexpr int kQatParams = 22;

struct QatArgs {
  const float *params;  // [bh][bw][22]
  const float *grad;    // texel gradients [h][w][3] (backward)
  float *texels;        // [h][w][3] (forward) or parameter gradients [bh][bw][22] (backward)
  uint2 *blocks;        // [bh][bw] (export)
  int32_t w, h, bw, bh;
  QatTables t;
};

__device__ __forceinline__ float sigmoidf(float x) { return 1.0f / (1.0f + __expf(-x)); }

// Code of logit x on M + 1 levels: the number of midpoint logits mid[0..M-1]
// at or below x. From two below a candidate of the FP32 sigmoid (within one
// level of the answer: its error is far below 1 / (2M)) four exact
// comparisons, whose midpoints load together. NaN gives 0.
__device__ __forceinline__ int quant_code(float x, const float *mid, int M) {
  const float s = sigmoidf(x) * (float)M;
  const int c = s >= 0.0f ? (int)rintf(fminf(s, (float)M)) : 0;
  const int lo = min(max(c - 2, 0), M - 3);
  int code = lo + (x >= mid[lo]) + (x >= mid[lo + 1]) + (x >= mid[lo + 2]);
  if (lo + 3 < M) code += x >= mid[lo + 3];
  return x == x ? code : 0;
}

// The same for the 2-bit weights, whose three midpoints are all compared.
__device__ __forceinline__ int weight_code(float x, const QatTables &t) {
  return (x >= t.mid2[0]) + (x >= t.mid2[1]) + (x >= t.mid2[2]);
}

// The texels and gradients kernels take a block in 16 lanes (a DPP row), one
// texel each; lanes 0 to 5 also hold the endpoint logits. One thread per block
// left a level of 512 x 512 texels to 256 wavefronts, each a chain of 22 codes
// of dependent loads: 24 us at 512 x 512 and at 1024 x 1024 alike (four levels
// up to 1024 x 1024: gradients 98 -> 22 us, texels 36 -> 21 us).
struct BlockLane {
  int64_t block;
  int t;         // texel (t & 3, t >> 2)
  int64_t texel; // its index in the level
};

__device__ __forceinline__ bool block_lane(const QatArgs &a, BlockLane &b) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  b.block = id >> 4;
  b.t = (int)(id & 15);
  if (b.block >= (int64_t)a.bw * a.bh) return false;
  const int bx = (int)(b.block % a.bw), by = (int)(b.block / a.bw);
  b.texel = (int64_t)(4 * by + (b.t >> 2)) * a.w + 4 * bx + (b.t & 3);
  return true;
}

// Code of lane t's endpoint logit x (t < 6; other lanes: of the last one).
__device__ __forceinline__ int endpoint_code(float x, int t, const QatTables &q) {
  const bool green = t == 1 || t == 4;
  return quant_code(x, green ? q.mid6 : q.mid5, green ? 63 : 31);
}

// Sum over the 16 lanes of a row, in every lane.
__device__ __forceinline__ float row_sum(float v) {
#define NTC_ROW_ADD(N) \
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xF, 0xF, false))  // row_ror:N
  NTC_ROW_ADD(8);
  NTC_ROW_ADD(4);
  NTC_ROW_ADD(2);
  NTC_ROW_ADD(1);
#undef NTC_ROW_ADD
  return v;
}

__global__ __launch_bounds__(256) void qat_texels_kernel(QatArgs a) {
  BlockLane b;
  if (!block_lane(a, b)) return;
  const float *p = a.params + b.block * kQatParams;
  const float xe = p[min(b.t, 5)], xw = p[6 + b.t];
  const int ec = endpoint_code(xe, b.t, a.t);
  const int w = weight_code(xw, a.t);
  // numerators over 6 (2^b - 1), as the BC1 decoder forms them, and their
  // quotient rounded once
  float *o = a.texels + b.texel * 3;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int e0 = __shfl(ec, c, 16), e1 = __shfl(ec, 3 + c, 16);
    const int n = 2 * (3 - w) * e0 + 2 * w * e1;
    o[c] = __fdiv_rn((float)n, c == 1 ? 378.0f : 186.0f);
  }
}

// Gradients with the quantisation passed through,
//   dL/dE0_c = sum_t (1 - w_t/3) g_tc, dL/dE1_c = sum_t (w_t/3) g_tc,
//   dL/dw_t = sum_c (E1_c - E0_c) g_tc  (values E, w/3 in [0, 1]),
// each times the sigmoid's derivative at its logit.
__global__ __launch_bounds__(256) void qat_backward_kernel(QatArgs a) {
  BlockLane b;
  if (!block_lane(a, b)) return;
  const float *p = a.params + b.block * kQatParams;
  float *gp = a.texels + b.block * kQatParams;
  const float *g = a.grad + b.texel * 3;
  const float xe = p[min(b.t, 5)], xw = p[6 + b.t];
  const float gt[3] = {g[0], g[1], g[2]};
  const bool green = b.t == 1 || b.t == 4;
  const float ev = (float)endpoint_code(xe, b.t, a.t) * (green ? 1.0f / 63.0f : 1.0f / 31.0f);
  const float wv = (float)weight_code(xw, a.t) * (1.0f / 3.0f);
  float ga = 0.f, ge = 0.f;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const float d = __shfl(ev, 3 + c, 16) - __shfl(ev, c, 16);
    ga = fmaf(d, gt[c], ga);
    const float g0 = row_sum((1.0f - wv) * gt[c]), g1 = row_sum(wv * gt[c]);
    ge = b.t == c ? g0 : (b.t == 3 + c ? g1 : ge);
  }
  const float sw = sigmoidf(xw);
  gp[6 + b.t] = sw * (1.0f - sw) * ga;
  if (b.t < 6) {
    const float se = sigmoidf(xe);
    gp[b.t] = se * (1.0f - se) * ge;
  }
}

// One thread per block: BC1 words whose four-colour decode gives the
// quantised texels. The palette of (c0, c1) in four-colour mode (c0 > c1)
// is indexed 0: E0, 1: E1, 2: (2 E0 + E1) / 3, 3: (E0 + 2 E1) / 3, so weight
// w maps to index {0, 2, 3, 1}[w]; with c0 < c1 the endpoints swap and w
// becomes 3 - w; equal endpoints make every weight give E0 (index 0).
__global__ __launch_bounds__(256) void qat_export_kernel(QatArgs a) {
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (int64_t)a.bw * a.bh) return;
  const float *p = a.params + id * kQatParams;
  uint32_t c[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const uint32_t r = (uint32_t)quant_code(p[3 * e], a.t.mid5, 31);
    const uint32_t g = (uint32_t)quant_code(p[3 * e + 1], a.t.mid6, 63);
    const uint32_t b = (uint32_t)quant_code(p[3 * e + 2], a.t.mid5, 31);
    c[e] = (r << 11) | (g << 5) | b;
  }
  const bool swap = c[0] < c[1];
  uint32_t idx = 0;
  if (c[0] != c[1]) {
    for (int t = 0; t < 16; ++t) {
      uint32_t w = (uint32_t)weight_code(p[6 + t], a.t);
      if (swap) w = 3u - w;
      idx |= ((0x78u >> (2u * w)) & 3u) << (2u * t);  // {0, 2, 3, 1}[w]
    }
  }
  const uint32_t lo = swap ? (c[1] | (c[0] << 16)) : (c[0] | (c[1] << 16));
  a.blocks[id] = make_uint2(lo, idx);
}

QatArgs qat_args(const float *params, int w, int h) {
  QatArgs a{};
  a.params = params;
  a.w = w;
  a.h = h;
  a.bw = w / 4;
  a.bh = h / 4;
  a.t = qat_tables();
  return a;
}

}  // namespace

QatTables qat_tables() {
  static QatTables t = [] {
    QatTables q{};
    auto fill = [](float *mid, int M) {
      for (int k = 0; k < M; ++k) {
        const double p = (k + 0.5) / M;
        mid[k] = (float)std::log(p / (1.0 - p));
      }
    };
    fill(q.mid5, 31);
    fill(q.mid6, 63);
    fill(q.mid2, 3);
    return q;
  }();
  return t;
}

hipError_t launch_qat_texels(const float *params, int w, int h, float *texels, hipStream_t st) {
  QatArgs a = qat_args(params, w, h);
  a.texels = texels;
  const int64_t n = (int64_t)w * h;  // 16 lanes a block
  hipLaunchKernelGGL(qat_texels_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_qat_backward(const float *params, int w, int h, const float *grad_texels, float *grad_params,
                               hipStream_t st) {
  QatArgs a = qat_args(params, w, h);
  a.grad = grad_texels;
  a.texels = grad_params;
  const int64_t n = (int64_t)w * h;
  hipLaunchKernelGGL(qat_backward_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_qat_export(const float *params, int w, int h, uint64_t *blocks, hipStream_t st) {
  QatArgs a = qat_args(params, w, h);
  a.blocks = reinterpret_cast<uint2 *>(blocks);
  const int64_t n = (int64_t)a.bw * a.bh;
  hipLaunchKernelGGL(qat_export_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace ntc
