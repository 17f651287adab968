// Backward of the FP32 decode for continuous latents (Sec. 3.2: gradients
// flow through the MLP into every latent element).
//
// Pass 1 (backward_mfma_kernel): per chunk of 32 samples, the forward is
// recomputed on the matrix cores (FP32 operands and accumulation), the
// deltas D_l = (W_{l+1}^T D_{l+1}) * [A_l > 0] (ReLU derivative 0 at 0) are
// products on the matrix cores too, and so are the weight gradients
// D_l A_l^T over the chunk's samples, accumulated in registers per
// wavefront. dx = W_0^T D_0, the gradient of the sample's latent features, is
// written to the workspace with the sample's coordinates. Activations are never stored in global memory.
// At the end every wavefront writes its FP32 partial sums; a second kernel
// adds the partials of all wavefronts in FP64 and rounds once to FP32.
// Pass 2 (latent gradients): the samples are grouped by spatial bin (a square
// of level-0 texels) with a counting sort; a workgroup takes up to kBinRun
// samples of a bin, spreads dx onto the four bilinear taps of every level,
// adding into LDS copies of the texels the bin's samples can reach, and then
// adds those windows to the latent gradients with one atomic per texel and
// channel (taps outside a window go straight to a global atomic).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "ntc_device.hpp"
#include "ntc_internal.hpp"

namespace ntc {

// Number of MLP parameters, laid out per layer as W_l [rows][cols] then b_l.
static inline int n_params_of(const MlpShape &s) {
  int n = 0;
  int d[kMaxLayers + 1];
  d[0] = s.in_dim;
  for (int l = 1; l < s.n_layers; ++l) d[l] = s.hid;
  d[s.n_layers] = s.n_out;
  for (int l = 0; l < s.n_layers; ++l) n += d[l] * d[l + 1] + d[l + 1];
  return n;
}

// Matrix-core backward: workgroups of kBwdWaves wavefronts (one per SIMD),
// each wavefront taking kBwdChunk samples per step; one row of partial
// weight-gradient sums per wavefront.
constexpr int kBwdWaves = 4;
constexpr int kBwdChunk = 32;
constexpr int kBwdMaxGroups = 256;

static int backward_groups(int64_t n) {
  const int64_t chunks = (n + kBwdChunk - 1) / kBwdChunk;
  const int64_t g = (chunks + kBwdWaves - 1) / kBwdWaves;
  return (int)(g > kBwdMaxGroups ? kBwdMaxGroups : (g < 1 ? 1 : g));
}

static int backward_blocks(int64_t n) { return kBwdWaves * backward_groups(n); }

// Spatial bins of the latent-gradient scatter: squares of 2^kBinShift (or a
// larger power of two, keeping at most kMaxBins bins) level-0 texels.
constexpr int kBinShift = 5;
constexpr int kMaxBins = 4096;
constexpr int kBinSamplesPerBlock = 4096;  // samples per workgroup of the count / scatter passes
constexpr int kBinRun = 1120;              // samples of a bin taken by one workgroup of the accumulation
constexpr int kAccThreads = 512;           // threads of that workgroup
constexpr int kBinWindowFloats = 12288;    // largest LDS of a bin's texel window (48 KB)
constexpr int kBinWindowCells = 4096;      // largest number of cells of one window

// LDS of one bin: floats and cells of its largest texel window.
// A bin spans 2^shift cells of level 0 (one more at a clamped edge, which
// also has a cell before the first texel), and on the others at most its
// scaled size and four cells (the ends, the shift, the edge); a window has
// one texel more than cells along each axis.
static void bin_window(const LatArgs &lat, int shift, int &floats, int &cells) {
  int64_t most_f = 0, most_c = 0;
  for (int k = 0; k < lat.n_levels; ++k) {
    auto axis = [&](int n, int n0) {
      const int64_t c = k == 0 ? ((int64_t)1 << shift) + 1 : ((int64_t)n << shift) / n0 + 4;
      return std::min<int64_t>(c, n + 1);
    };
    const int64_t nc = axis(lat.lv[k].w, lat.lv[0].w), nr = axis(lat.lv[k].h, lat.lv[0].h);
    most_f = std::max(most_f, 3 * (nc + 1) * (nr + 1));
    most_c = std::max(most_c, nc * nr);
  }
  floats = (int)std::min<int64_t>(most_f, kBinWindowFloats);
  cells = (int)std::min<int64_t>(most_c, kBinWindowCells);
}

static size_t align256(size_t v) { return (v + 255) / 256 * 256; }

BwdLayout backward_layout(const MlpShape &s, const LatArgs &lat, int64_t n) {
  BwdLayout L{};
  L.n_blocks = backward_blocks(n);
  L.n_params = n_params_of(s);
  L.n_feat = 3 * lat.n_levels;
  L.dx_stride = (L.n_feat + 2 + 3) & ~3;
  if (n < ((int64_t)1 << 31)) {  // sample indices of the bins are int32
    int t = kBinShift;
    const int w = lat.lv[0].w, h = lat.lv[0].h;
    auto bins = [&](int len) { return (len + (1 << t) - 1) >> t; };
    while ((int64_t)bins(w) * bins(h) > kMaxBins) ++t;
    L.bin_shift = t;
    L.bins_x = bins(w);
    L.n_bins = bins(w) * bins(h);
    L.n_runs = L.n_bins + (int32_t)(n / kBinRun);
    bin_window(lat, t, L.bin_lds, L.bin_cells);
  }
  size_t off = 0;
  L.wpart_off = off;
  off = align256(off + (size_t)L.n_blocks * L.n_params * sizeof(float));
  L.dx_off = off;
  off = align256(off + (size_t)n * L.dx_stride * sizeof(float));
  L.count_off = off;
  off = align256(off + (size_t)L.n_bins * sizeof(int32_t));
  L.cursor_off = off;
  off = align256(off + (size_t)L.n_bins * sizeof(int32_t));
  L.perm_off = off;
  off = align256(off + (size_t)(L.n_bins ? n : 0) * sizeof(int32_t));
  L.runs_off = off;
  off = align256(off + (size_t)(L.n_bins ? 1 + L.n_runs : 0) * sizeof(int4));
  L.total = off + 256;
  return L;
}

struct ReduceArgs {
  const float *part;
  int n_blocks;
  int n_params;
  int n_layers;
  int dims[kMaxLayers + 1];
  float *W[kMaxLayers];
  float *b[kMaxLayers];
};

// grad[p] = sum over workgroups of part[b][p], added in FP64, rounded once.
// A workgroup owns 64 consecutive parameters (one per lane, coalesced
// loads); its kReduceWaves wavefronts each add every kReduceWaves-th
// workgroup's partials, and the wavefront sums are then added in wavefront
// order, so the result does not depend on timing.
constexpr int kReduceWaves = 16;
__global__ __launch_bounds__(64 * kReduceWaves) void reduce_f64_kernel(ReduceArgs r) {
  __shared__ double wsum[kReduceWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = blockIdx.x * 64 + lane;
  double s = 0.0;
  if (p < r.n_params) {
#pragma unroll 8
    for (int b = w; b < r.n_blocks; b += kReduceWaves) s += (double)r.part[(int64_t)b * r.n_params + p];
  }
  wsum[w][lane] = s;
  __syncthreads();
  if (w != 0 || p >= r.n_params) return;
  s = 0.0;
#pragma unroll
  for (int i = 0; i < kReduceWaves; ++i) s += wsum[i][lane];
  int off = p;
  for (int l = 0; l < r.n_layers; ++l) {
    const int nw = r.dims[l] * r.dims[l + 1];
    if (off < nw) {
      r.W[l][off] = (float)s;
      return;
    }
    off -= nw;
    if (off < r.dims[l + 1]) {
      r.b[l][off] = (float)s;
      return;
    }
    off -= r.dims[l + 1];
  }
}

// ---------------------------------------------------------------------------
// Pass 1 on the matrix cores (FP32 operands, v_mfma_f32_32x32x2f32)
//
// A wavefront takes 32 samples per step (the 32 columns of the matrix
// tiles). Every product is a 32 x 32 tile of units x samples: the weights
// are the A operand (row = output unit, one float per lane), the layer input
// the B operand. In the accumulator a lane holds rows 8 j + 4 h + r (j, r < 4,
// h = lane / 32) of sample lane % 32; K-step t of a product whose input is
// such a tile takes element t of it (lane half h supplying unit
// 8 (t / 4) + 4 h + t % 4 of the tile), so layers chain in registers in both
// directions and the ReLU mask of a delta is the activation at the same
// register. The first layer's K-slots hold per lane half two levels'
// features: slot 2 s + h is channel s % 3 of level 2 h + s / 3 (s < 6), u
// or v (s = 6), the constant 1 that carries the bias (s = 7, h = 0) or
// padding. Weight gradients contract over the samples: each step writes the
// deltas and the layer inputs transposed to LDS ([unit][sample], even
// samples first) and accumulates D A^T over 16 K-steps of two samples;
// bias gradients are row sums of the staged deltas.
// ---------------------------------------------------------------------------
typedef float bf32x16 __attribute__((ext_vector_type(16)));
typedef float bf32x4 __attribute__((ext_vector_type(4)));

constexpr int kStS = 36;  // row stride (floats) of the transposed staging

template <int MT, int NL>
struct BwdMap {
  static constexpr int HP = 32 * MT;        // padded hidden width
  static constexpr int S0 = 17;             // row stride of the first layer (16 K-slots)
  static constexpr int SH = HP + 1;         // row stride of the other layers
  static constexpr int NH = NL - 2;         // hidden-to-hidden layers
  static constexpr int oW0 = 0;
  static constexpr int oWh = oW0 + HP * S0;
  static constexpr int oWo = oWh + NH * HP * SH;
  static constexpr int oB = (oWo + 32 * SH + 3) & ~3;  // bias fragments [layer 1..NL-1][mt][h][16]
  static constexpr int nB = (NH * MT + 1) * 32;
  static constexpr int oStage = (oB + nB + 3) & ~3;
  static constexpr int stage_rows = HP + (HP > 32 ? HP : 32);
  static constexpr int stage = stage_rows * kStS;    // Dt then At, per wavefront
  static constexpr int total = oStage + kBwdWaves * stage;
  __device__ static int bias(int l, int mt) { return oB + ((l - 1) * MT + mt) * 32; }  // l = 1 .. NL - 1
};

// Unit of the previous layer's tile fed to K-step s by lane half h.
__device__ __forceinline__ int chain_unit(int s, int h) {
  return 32 * (s >> 4) + 8 * ((s & 15) >> 2) + 4 * h + (s & 3);
}

// Feature index of first-layer K-slot 2 s + h (-1: padding, -2: the bias).
__device__ __forceinline__ int slot_feature(int s, int h, int n_levels) {
  if (s < 6) {
    const int lvl = 2 * h + s / 3;
    return lvl < n_levels ? 3 * lvl + s % 3 : -1;
  }
  if (s == 6) return 3 * n_levels + h;
  return h == 0 ? -2 : -1;
}

__device__ __forceinline__ bf32x16 mfma32(float a, float b, bf32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

template <int MT, int NL>
__global__ __launch_bounds__(64 * kBwdWaves) __attribute__((amdgpu_waves_per_eu(1, 1)))
void backward_mfma_kernel(BackwardArgs a) {
  using M = BwdMap<MT, NL>;
  constexpr int HP = M::HP;
  extern __shared__ float bwd_lds[];
  float *lds = bwd_lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63, h = lane >> 5, c32 = lane & 31;
  const int wave = tid >> 6;
  const int hid = a.dims[1], n_out = a.dims[NL], d0 = a.dims[0];
  const int n_levels = a.lat.n_levels;

  // ---- weights into LDS, zero-padded (every wavefront of the group shares them)
  for (int i = tid; i < HP * 16; i += 64 * kBwdWaves) {
    const int row = i >> 4, k = i & 15;
    const int f = slot_feature(k >> 1, k & 1, n_levels);
    float v = 0.0f;
    if (row < hid) v = f >= 0 ? a.W[0][row * d0 + f] : (f == -2 ? a.b[0][row] : 0.0f);
    lds[M::oW0 + row * M::S0 + k] = v;
  }
#pragma unroll
  for (int l = 1; l <= M::NH; ++l)
    for (int i = tid; i < HP * HP; i += 64 * kBwdWaves) {
      const int row = i / HP, col = i % HP;
      lds[M::oWh + (l - 1) * HP * M::SH + row * M::SH + col] = (row < hid && col < hid) ? a.W[l][row * hid + col] : 0.0f;
    }
  for (int i = tid; i < 32 * HP; i += 64 * kBwdWaves) {
    const int row = i / HP, col = i % HP;
    lds[M::oWo + row * M::SH + col] = (row < n_out && col < hid) ? a.W[NL - 1][row * hid + col] : 0.0f;
  }
  for (int i = tid; i < M::nB; i += 64 * kBwdWaves) {
    const int g = i / 32, e = i % 32;  // g = (l - 1) MT + mt, e = 16 h + 4 j + r
    const int l = g / MT + 1 < NL - 1 ? g / MT + 1 : NL - 1;
    const int mt = l == NL - 1 ? 0 : g % MT;
    const int row = 32 * mt + 8 * ((e & 15) >> 2) + 4 * (e >> 4) + (e & 3);
    const int rows = l == NL - 1 ? n_out : hid;
    lds[M::oB + i] = row < rows ? a.b[l][row] : 0.0f;
  }
  float *Dt = lds + M::oStage + wave * M::stage;
  float *At = Dt + HP * kStS;
  // the staging rows a layer input does not fill stay zero (first-layer K-slots 16..31)
  for (int i = lane; i < M::stage; i += 64) Dt[i] = 0.0f;
  __syncthreads();

  const float *W0s = lds + M::oW0;
  const float *Wo = lds + M::oWo;
  const bf32x16 zero = {};

  // weight-gradient accumulators: first layer [mt] (columns = K-slots), hidden
  // layers [l][mt][nt], output [nt]; bias gradients of rows `lane` (hidden)
  bf32x16 g0[MT], gh[M::NH > 0 ? M::NH : 1][MT][MT], go[MT];
  float gbh[M::NH > 0 ? M::NH : 1], gbo = 0.0f;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    g0[i] = zero;
    go[i] = zero;
#pragma unroll
    for (int l = 0; l < (M::NH > 0 ? M::NH : 1); ++l)
#pragma unroll
      for (int j = 0; j < MT; ++j) gh[l][i][j] = zero;
  }
#pragma unroll
  for (int l = 0; l < (M::NH > 0 ? M::NH : 1); ++l) gbh[l] = 0.0f;

  // staging helpers: a tile in accumulator layout -> rows [row0, row0 + 32)
  // of a transposed buffer (column of sample n: 16 (n % 2) + n / 2)
  const int scol = 16 * (c32 & 1) + (c32 >> 1);
  auto stage_tile = [&](float *buf, int row0, const bf32x16 &t) {
#pragma unroll
    for (int i = 0; i < 16; ++i) buf[(row0 + 8 * (i >> 2) + 4 * h + (i & 3)) * kStS + scol] = t[i];
  };
  // the 16 K-step operands of row `row` (samples 2 s + h, s < 16)
  auto stage_row = [&](const float *buf, int row, float (&v)[16]) {
    const bf32x4 *p = reinterpret_cast<const bf32x4 *>(buf + row * kStS + 16 * h);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const bf32x4 x = p[q];
      v[4 * q] = x[0];
      v[4 * q + 1] = x[1];
      v[4 * q + 2] = x[2];
      v[4 * q + 3] = x[3];
    }
  };
  // sum over the 32 samples of staged row `row`
  auto row_sum = [&](const float *buf, int row) {
    const bf32x4 *p = reinterpret_cast<const bf32x4 *>(buf + row * kStS);
    float sum = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bf32x4 x = p[q];
      sum += (x[0] + x[1]) + (x[2] + x[3]);
    }
    return sum;
  };
  // dW += Dt(MT_D tiles) At(NT_A tiles)^T over the 16 K-steps
  auto accum_dw = [&](auto &&acc, int mtn, int ntn) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int mt = 0; mt < mtn; ++mt) {
      float av[16];
      stage_row(Dt, 32 * mt + c32, av);
#pragma unroll
      for (int nt = 0; nt < ntn; ++nt) {
        float bv[16];
        stage_row(At, 32 * nt + c32, bv);
#pragma unroll
        for (int q = 0; q < 16; ++q) acc(mt, nt) = mfma32(av[q], bv[q], acc(mt, nt));
      }
    }
    asm volatile("" ::: "memory");
  };

  const int64_t n_chunks = (a.n + kBwdChunk - 1) / kBwdChunk;
  const int64_t stride = (int64_t)gridDim.x * kBwdWaves;
  for (int64_t chunk = (int64_t)blockIdx.x * kBwdWaves + wave; chunk < n_chunks; chunk += stride) {
    const int64_t smp = chunk * kBwdChunk + c32;
    const bool valid = smp < a.n;
    const float2 uv = a.uv[valid ? smp : a.n - 1];

    // ---- features of this lane half's K-slots
    float x[8];
    {
      const float3 c0 = sample_f32(a.lat.lv[2 * h], uv.x, uv.y, a.lat.address);
      const float3 c1 = sample_f32(a.lat.lv[2 * h + 1], uv.x, uv.y, a.lat.address);
      x[0] = c0.x; x[1] = c0.y; x[2] = c0.z;
      x[3] = c1.x; x[4] = c1.y; x[5] = c1.z;
      x[6] = h ? uv.y : uv.x;
      x[7] = h ? 0.0f : 1.0f;
    }

    // ---- forward
    bf32x16 act[NL - 1][MT];  // ReLU outputs of the hidden layers
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      bf32x16 z = zero;
#pragma unroll
      for (int s = 0; s < 8; ++s) z = mfma32(W0s[(32 * mt + c32) * M::S0 + 2 * s + h], x[s], z);
#pragma unroll
      for (int i = 0; i < 16; ++i) z[i] = fmaxf(z[i], 0.0f);
      act[0][mt] = z;
    }
#pragma unroll
    for (int l = 1; l <= M::NH; ++l) {
      const float *Wl = lds + M::oWh + (l - 1) * HP * M::SH;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bf32x4 *bp = reinterpret_cast<const bf32x4 *>(lds + M::bias(l, mt) + 16 * h);
        const bf32x4 b0 = bp[0], b1 = bp[1], b2 = bp[2], b3 = bp[3];
        bf32x16 z = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3],
                     b2[0], b2[1], b2[2], b2[3], b3[0], b3[1], b3[2], b3[3]};
#pragma unroll
        for (int s = 0; s < 16 * MT; ++s)
          z = mfma32(Wl[(32 * mt + c32) * M::SH + chain_unit(s, h)], act[l - 1][s >> 4][s & 15], z);
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = fmaxf(z[i], 0.0f);
        act[l][mt] = z;
      }
    }
    bf32x16 dout;
    {
      const bf32x4 *bp = reinterpret_cast<const bf32x4 *>(lds + M::bias(NL - 1, 0) + 16 * h);
      const bf32x4 b0 = bp[0], b1 = bp[1];
      bf32x16 z = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3], 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 16 * MT; ++s)
        z = mfma32(Wo[c32 * M::SH + chain_unit(s, h)], act[NL - 2][s >> 4][s & 15], z);
      // output deltas: g f (1 - f) on rows 8 j + 4 h + r < n_out (j < 2)
      dout = zero;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = 8 * (i >> 2) + 4 * h + (i & 3);
        if (row < n_out && valid) {
          const float f = 1.0f / (1.0f + expf(-z[i]));
          dout[i] = a.grad_out[smp * n_out + row] * f * (1.0f - f);
        }
      }
    }

    // ---- output layer: weight and bias gradients, delta of the last hidden layer
    stage_tile(Dt, 0, dout);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) stage_tile(At, 32 * mt, act[NL - 2][mt]);
    accum_dw([&](int, int nt) -> bf32x16 & { return go[nt]; }, 1, MT);
    if (lane < 16) gbo += row_sum(Dt, lane);
    bf32x16 del[MT];
    {
      const int tk = n_out > 8 ? 8 : 4;  // K-steps covering rows 0 .. n_out - 1
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        bf32x16 z = zero;
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (t < tk) z = mfma32(Wo[(8 * (t >> 2) + 4 * h + (t & 3)) * M::SH + 32 * mt + c32], dout[t], z);
#pragma unroll
        for (int i = 0; i < 16; ++i) del[mt][i] = act[NL - 2][mt][i] > 0.0f ? z[i] : 0.0f;
      }
    }
    // ---- hidden layers, top down
#pragma unroll
    for (int l = M::NH; l >= 1; --l) {
      const float *Wl = lds + M::oWh + (l - 1) * HP * M::SH;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        stage_tile(Dt, 32 * mt, del[mt]);
        stage_tile(At, 32 * mt, act[l - 1][mt]);
      }
      accum_dw([&](int mt, int nt) -> bf32x16 & { return gh[l - 1][mt][nt]; }, MT, MT);
      if (lane < HP) gbh[l - 1] += row_sum(Dt, lane);
      bf32x16 nd[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        bf32x16 z = zero;
#pragma unroll
        for (int s = 0; s < 16 * MT; ++s)
          z = mfma32(Wl[chain_unit(s, h) * M::SH + 32 * mt + c32], del[s >> 4][s & 15], z);
#pragma unroll
        for (int i = 0; i < 16; ++i) nd[mt][i] = act[l - 1][mt][i] > 0.0f ? z[i] : 0.0f;
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) del[mt] = nd[mt];
    }
    // ---- first layer: weight gradients over the K-slots (slot 14 = bias)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) stage_tile(Dt, 32 * mt, del[mt]);
#pragma unroll
    for (int s = 0; s < 8; ++s) At[(2 * s + h) * kStS + scol] = x[s];
    accum_dw([&](int mt, int) -> bf32x16 & { return g0[mt]; }, MT, 1);
    // ---- feature gradient dx = W0^T D0: rows = latent features
    {
      const int f = c32;  // feature of A-operand row c32
      const int lvl = f / 3;
      const int slot = (lvl < n_levels && f < 12) ? 2 * (3 * (lvl & 1) + f % 3) + (lvl >> 1) : -1;
      bf32x16 z = zero;
#pragma unroll
      for (int s = 0; s < 16 * MT; ++s) {
        const float w = slot >= 0 ? W0s[chain_unit(s, h) * M::S0 + slot] : 0.0f;
        z = mfma32(w, del[s >> 4][s & 15], z);
      }
      // the row of a.dx: the feature gradients, then u, v
      if (valid) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int row0 = 8 * j + 4 * h;
          if (row0 >= a.dx_stride) continue;
          float o[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            o[r] = row0 + r == a.n_feat ? uv.x : row0 + r == a.n_feat + 1 ? uv.y : z[4 * j + r];
          *reinterpret_cast<float4 *>(a.dx + smp * a.dx_stride + row0) = make_float4(o[0], o[1], o[2], o[3]);
        }
      }
    }
  }

  // ---- this wavefront's partial sums (parameters in unpadded order)
  float *part = a.wpart + ((int64_t)blockIdx.x * kBwdWaves + wave) * a.n_params;
  int off = 0;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = 32 * mt + 8 * (i >> 2) + 4 * h + (i & 3);
      const int k = c32;
      if (row < hid && k < 16) {
        const int f = slot_feature(k >> 1, k & 1, n_levels);
        if (f >= 0) part[off + row * d0 + f] = g0[mt][i];
        if (f == -2) part[off + hid * d0 + row] = g0[mt][i];
      }
    }
  off += hid * d0 + hid;
#pragma unroll
  for (int l = 0; l < M::NH; ++l) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < MT; ++nt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int row = 32 * mt + 8 * (i >> 2) + 4 * h + (i & 3), col = 32 * nt + c32;
          if (row < hid && col < hid) part[off + row * hid + col] = gh[l][mt][nt][i];
        }
    if (lane < hid) part[off + hid * hid + lane] = gbh[l];
    off += hid * hid + hid;
  }
#pragma unroll
  for (int nt = 0; nt < MT; ++nt)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = 8 * (i >> 2) + 4 * h + (i & 3), col = 32 * nt + c32;
      if (row < n_out && col < hid) part[off + row * hid + col] = go[nt][i];
    }
  if (lane < n_out) part[off + n_out * hid + lane] = gbo;
}

// ---------------------------------------------------------------------------
// Pass 2: latent gradients
// ---------------------------------------------------------------------------

// Sampling position on one level split into the left / top tap (not yet
// addressed) and the bilinear fractions, as tap_coords() does.
struct Cell {
  int ix, iy;
  float fx, fy;
};

__device__ __forceinline__ Cell cell_of(const LevelArgs &L, float2 uv) {
  float x = fmaf(uv.x, L.fw, -0.5f) + L.sx;
  float y = fmaf(uv.y, L.fh, -0.5f) + L.sy;
  x = fminf(fmaxf(x, -16777216.0f), 16777216.0f);
  y = fminf(fmaxf(y, -16777216.0f), 16777216.0f);
  const float xf = floorf(x), yf = floorf(y);
  return {(int)xf, (int)yf, x - xf, y - yf};
}

// Bin of a sample: the square of level-0 texels holding its addressed
// (clamped or wrapped) top left tap.
__device__ __forceinline__ int bin_of(const BackwardArgs &a, float2 uv) {
  const LevelArgs &L = a.lat.lv[0];
  const Cell c = cell_of(L, uv);
  return (address_coord(c.iy, L.h, a.lat.address) >> a.bin_shift) * a.bins_x +
         (address_coord(c.ix, L.w, a.lat.address) >> a.bin_shift);
}

// Per-bin sample counts: a histogram in LDS per workgroup, added to the
// global counts (which start at zero).
__global__ __launch_bounds__(256) void bin_count_kernel(BackwardArgs a) {
  extern __shared__ int32_t hist[];
  for (int k = threadIdx.x; k < a.n_bins; k += 256) hist[k] = 0;
  __syncthreads();
  const int64_t s0 = (int64_t)blockIdx.x * kBinSamplesPerBlock;
  for (int i = threadIdx.x; i < kBinSamplesPerBlock; i += 256) {
    const int64_t s = s0 + i;
    if (s < a.n) atomicAdd(&hist[bin_of(a, a.uv[s])], 1);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < a.n_bins; k += 256)
    if (hist[k]) atomicAdd(&a.bin_count[k], hist[k]);
}

// Inclusive prefix sums of one pair per thread over the 1024 threads of a
// workgroup.
__device__ __forceinline__ int2 scan1024(int2 v, int2 *part) {
  const int t = threadIdx.x;
  part[t] = v;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int2 u = t >= o ? part[t - o] : make_int2(0, 0);
    __syncthreads();
    part[t].x += u.x;
    part[t].y += u.y;
    __syncthreads();
  }
  return part[t];
}

// Exclusive prefix sum of the counts into the cursors, and the work list of
// bin_accum_kernel: every bin's samples cut into runs of at most kBinRun,
// as (bin, first sample, end) with the run count in front. One workgroup of
// 1024 threads.
__global__ __launch_bounds__(1024) void bin_scan_kernel(BackwardArgs a) {
  __shared__ int2 part[1024];
  const int t = threadIdx.x;
  const int per = (a.n_bins + 1023) / 1024;
  const int k0 = t * per, k1 = min(k0 + per, a.n_bins);
  int2 sum = make_int2(0, 0);
  for (int k = k0; k < k1; ++k) {
    sum.x += a.bin_count[k];
    sum.y += (a.bin_count[k] + kBinRun - 1) / kBinRun;
  }
  int2 run = scan1024(sum, part);
  if (t == 1023) a.runs[0] = make_int4(run.y, 0, 0, 0);
  run.x -= sum.x;
  run.y -= sum.y;
  for (int k = k0; k < k1; ++k) {
    const int32_t c = a.bin_count[k];
    a.bin_cursor[k] = run.x;
    for (int i = 0; i < c; i += kBinRun) a.runs[1 + run.y++] = make_int4(k, run.x + i, run.x + min(i + kBinRun, c), 0);
    run.x += c;
  }
}

// Sample indices grouped by bin: each workgroup ranks its samples per bin in
// LDS, reserves a range per bin with one global atomic, then writes. The
// order inside a bin depends on timing (as does the order of the atomics
// that follow it).
__global__ __launch_bounds__(256) void bin_scatter_kernel(BackwardArgs a) {
  extern __shared__ int32_t lds[];
  int32_t *local = lds, *base = lds + a.n_bins;
  for (int k = threadIdx.x; k < a.n_bins; k += 256) local[k] = 0;
  __syncthreads();
  constexpr int kPer = kBinSamplesPerBlock / 256;
  const int64_t s0 = (int64_t)blockIdx.x * kBinSamplesPerBlock;
  int key[kPer], rank[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int64_t s = s0 + threadIdx.x + 256 * i;
    key[i] = s < a.n ? bin_of(a, a.uv[s]) : -1;
    rank[i] = key[i] >= 0 ? atomicAdd(&local[key[i]], 1) : 0;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < a.n_bins; k += 256)
    if (local[k]) base[k] = atomicAdd(&a.bin_cursor[k], local[k]);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (key[i] >= 0) a.perm[base[key[i]] + rank[i]] = (int32_t)(s0 + threadIdx.x + 256 * i);
}

// Cells (left / top taps) of one level that one bin's samples fall into:
// columns c0 .. c0 + nc - 1, rows r0 .. r0 + nr - 1, before addressing (a
// clamped level's cells start at -1, a wrapped level's may pass either end).
// They touch the (nc + 1) x (nr + 1) texels from (c0, r0).
struct BinWindow {
  int c0, nc, r0, nr;
};

// Cells along one axis of level k for the level-0 cells [p, p + len) of a
// bin: the position maps linearly between levels. The range need not be
// exact: a sample that rounding puts outside it takes the global path.
__device__ __forceinline__ void window_axis(int k, int p, int len, int n0, float f0, float s0, int n, float fk,
                                            float sk, int mode, int &c0, int &nc) {
  const float q = fk / f0;
  int lo = k == 0 ? p : (int)floorf(((float)p + 0.5f - s0) * q - 0.5f + sk);
  int hi = k == 0 ? p + len - 1 : (int)floorf(((float)(p + len) + 0.5f - s0) * q - 0.5f + sk);
  if (mode == 1) {
    if (hi - lo + 1 >= n) {
      lo = 0;
      hi = n - 1;
    }
  } else {
    lo = p == 0 ? -1 : min(max(lo, -1), n - 1);
    hi = p + len >= n0 ? n - 1 : min(max(hi, lo), n - 1);
  }
  c0 = lo;
  nc = hi - lo + 1;
}

// i modulo n for |i| <= 2^25, with rn about 1 / n: the quotient is off by at
// most one (an integer division takes several times as long).
__device__ __forceinline__ int wrap_near(int i, int n, float rn) {
  int r = i - n * (int)floorf((float)i * rn);
  r += r < 0 ? n : 0;
  return r >= n ? r - n : r;
}

// Offset of cell coordinate i in a window axis (outside [0, nc): not in it).
__device__ __forceinline__ int window_coord(int i, int c0, int n, float rn, int mode) {
  return mode == 1 ? wrap_near(i - c0, n, rn) : min(max(i, -1), n - 1) - c0;
}

// Latent gradients of one level and one run of a bin's samples (at most
// kBinRun): one workgroup each.
//
// LDS float atomics bound the first form of this kernel (all levels of a bin
// in one workgroup, taps added to the window as they came): ds_add_f32 takes
// about 4.4 cycles per lane on gfx950 (SQ_LDS_IDX_ACTIVE), some 25 of them
// per sample. Here no float is added atomically in LDS. The run's samples
// are sorted by cell (a counting sort: integer LDS atomics, which are fast,
// and a scan), each carrying its fractions and its three gradient values;
// then every cell is summed in registers by the lanes that own it (several
// lanes per cell on the coarse levels) and its four taps are added to the
// window with plain reads and writes. Cells of one parity class (even or odd
// column, even or odd row) share no texel, so the four classes are taken one
// after the other with a barrier between them. At the end the window is added
// to the gradients, one global atomic per touched value. What is left is
// latency: a chain of about ten short steps between barriers, some 1 us each,
// which is why the levels are workgroups of their own (one workgroup taking
// all levels in turn: 90 us in place of the 57 below).
// 2^20 random samples on 1024^2..128^2 levels: 57 us (241 us with the LDS
// float atomics); 2^18 samples, wrapped 512^2..64^2 levels: 23 us (660 us
// with a global atomic per tap and channel).
// LDS: the window (bin_lds floats), five arrays of kBinRun floats, the cell
// counts: 40 KB with bins of 32 x 32 cells, so that four workgroups share a
// compute unit.
template <int kCtrl>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, true));
}

// Sum of the payloads start, start + step, ... < end of one cell per tap and
// channel.
__device__ __forceinline__ void cell_sum(const float *pay, int start, int end, int step, float (&g)[4][3]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) g[q][0] = g[q][1] = g[q][2] = 0.0f;
  for (int j = start; j < end; j += step) {
    const float x = pay[j], y = pay[kBinRun + j];
    const float gx = 1.0f - x, gy = 1.0f - y;
    const float w[4] = {gx * gy, x * gy, gx * y, x * y};
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float z = pay[(2 + ch) * kBinRun + j];
#pragma unroll
      for (int q = 0; q < 4; ++q) g[q][ch] = fmaf(w[q], z, g[q][ch]);
    }
  }
}

// Adds a cell's sums to its four texels; p: the top left one, tc texels a row.
__device__ __forceinline__ void cell_add(float *p, int tc, const float (&g)[4][3]) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) p[3 * ((q & 1) + (q >> 1) * tc) + ch] += g[q][ch];
}

__global__ __launch_bounds__(kAccThreads) void bin_accum_kernel(BackwardArgs a) {
  constexpr int kT = kAccThreads, kWaves = kT / 64;
  extern __shared__ float win[];
  float *pay = win + a.bin_lds;                                   // [5][kBinRun]
  int32_t *cnt = reinterpret_cast<int32_t *>(pay + 5 * kBinRun);  // [bin_cells + 1]
  __shared__ int32_t wsum[kWaves];
  // the levels of one run are neighbours on one XCD (workgroups go to the 8
  // XCDs in turn), whose L2 then holds the run's rows for all of them
  const int n_levels = a.lat.n_levels, mode = a.lat.address;
  const int k = (int)(blockIdx.x >> 3) % n_levels;
  const int item = ((int)(blockIdx.x >> 3) / n_levels) * 8 + (int)(blockIdx.x & 7);
  if (item >= a.runs[0].x) return;
  const int4 run = a.runs[1 + item];
  const int bx = run.x % a.bins_x, by = run.x / a.bins_x;
  const int m = run.z - run.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const LevelArgs &L0 = a.lat.lv[0];

  const LevelArgs &L = a.lat.lv[k];

  // this thread's samples: tid, tid + kT, ...
  constexpr int kPer = (kBinRun + kT - 1) / kT;
  float d[kPer][3];
  float2 uv[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const float *g = a.dx + (int64_t)a.perm[run.y + min(tid + kT * i, m - 1)] * a.dx_stride;
    uv[i] = make_float2(g[a.n_feat], g[a.n_feat + 1]);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) d[i][ch] = g[3 * k + ch];
  }
  const int lw = L.w, lh = L.h;
  const float rw = 1.0f / L.fw, rh = 1.0f / L.fh;
  BinWindow wk;
  window_axis(k, bx << a.bin_shift, 1 << a.bin_shift, L0.w, L0.fw, L0.sx, lw, L.fw, L.sx, mode, wk.c0, wk.nc);
  window_axis(k, by << a.bin_shift, 1 << a.bin_shift, L0.h, L0.fh, L0.sy, lh, L.fh, L.sy, mode, wk.r0, wk.nr);
  const int tc = wk.nc + 1, size = 3 * tc * (wk.nr + 1), cells = wk.nc * wk.nr;
  const bool fits = size <= a.bin_lds && cells <= a.bin_cells;
  if (fits) {
    for (int i = tid; i < size; i += kT) win[i] = 0.0f;
    for (int i = tid; i < cells; i += kT) cnt[i] = 0;
  }
  __syncthreads();
  // cell and rank of every sample
  int cell[kPer], rank[kPer];
  float fx[kPer], fy[kPer];
  bool direct = false;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const Cell c = cell_of(L, uv[i]);
    fx[i] = c.fx;
    fy[i] = c.fy;
    const int col = window_coord(c.ix, wk.c0, lw, rw, mode), line = window_coord(c.iy, wk.r0, lh, rh, mode);
    const bool in = fits && (unsigned)col < (unsigned)wk.nc && (unsigned)line < (unsigned)wk.nr;
    cell[i] = in ? line * wk.nc + col : -1;
    if (tid + kT * i >= m) {
      cell[i] = -1;
    } else if (in) {
      rank[i] = atomicAdd(&cnt[cell[i]], 1);
    } else {
      direct = true;
    }
  }
  if (direct) {  // samples outside the window go straight to the gradients
#pragma unroll 1
    for (int j = tid; j < m; j += kT) {
      const float *g = a.dx + (int64_t)a.perm[run.y + j] * a.dx_stride;
      const Cell c = cell_of(L, make_float2(g[a.n_feat], g[a.n_feat + 1]));
      const int col = window_coord(c.ix, wk.c0, lw, rw, mode), row = window_coord(c.iy, wk.r0, lh, rh, mode);
      if (fits && (unsigned)col < (unsigned)wk.nc && (unsigned)row < (unsigned)wk.nr) continue;
#pragma unroll 1
      for (int q = 0; q < 4; ++q) {
        const int ti = address_coord(c.ix + (q & 1), lw, mode), tj = address_coord(c.iy + (q >> 1), lh, mode);
        const float w = ((q & 1) ? c.fx : 1.0f - c.fx) * ((q >> 1) ? c.fy : 1.0f - c.fy);
        float *p = a.grad_lat[k] + ((int64_t)tj * lw + ti) * 3;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) unsafeAtomicAdd(p + ch, w * g[3 * k + ch]);
      }
    }
  }
  if (!fits) return;
  __syncthreads();
  // exclusive scan of the counts
  const int per = (cells + kT - 1) / kT;
  const int e0 = min(tid * per, cells), e1 = min(e0 + per, cells);
  int sum = 0;
  for (int e = e0; e < e1; ++e) sum += cnt[e];
  int v = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  if (lane == 63) wsum[wave] = v;
  __syncthreads();
  v -= sum;
#pragma unroll
  for (int w = 0; w < kWaves - 1; ++w) v += w < wave ? wsum[w] : 0;
  for (int e = e0; e < e1; ++e) {
    const int c = cnt[e];
    cnt[e] = v;
    v += c;
  }
  if (tid == kT - 1) cnt[cells] = v;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (cell[i] >= 0) {
      const int at = cnt[cell[i]] + rank[i];
      pay[at] = fx[i];
      pay[kBinRun + at] = fy[i];
      pay[2 * kBinRun + at] = d[i][0];
      pay[3 * kBinRun + at] = d[i][1];
      pay[4 * kBinRun + at] = d[i][2];
    }
  }
  __syncthreads();
  float g[4][3];
  if (cells <= kT) {
    // every cell at once, 2^ts lanes each (at most 16, a DPP row), then the
    // classes one after the other
    int ts = 0;
    while (ts < 4 && (cells << (ts + 1)) <= kT) ++ts;
    const int e = tid >> ts, row = (int)(((float)e + 0.5f) * (1.0f / (float)wk.nc)), col = e - row * wk.nc;
    const int start = e < cells ? cnt[e] : 0, end = e < cells ? cnt[e + 1] : 0;
    cell_sum(pay, start + (tid & ((1 << ts) - 1)), end, 1 << ts, g);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        if (ts > 0) g[q][ch] = dpp_add<0xB1>(g[q][ch]);   // quad_perm 1,0,3,2
        if (ts > 1) g[q][ch] = dpp_add<0x4E>(g[q][ch]);   // quad_perm 2,3,0,1
        if (ts > 2) g[q][ch] = dpp_add<0x141>(g[q][ch]);  // row_half_mirror
        if (ts > 3) g[q][ch] = dpp_add<0x140>(g[q][ch]);  // row_mirror
      }
    const int own = (tid & ((1 << ts) - 1)) == 0 && end > start ? (col & 1) + 2 * (row & 1) : -1;
#pragma unroll 1
    for (int par = 0; par < 4; ++par) {
      if (own == par) cell_add(win + 3 * (row * tc + col), tc, g);
      __syncthreads();
    }
  } else {
#pragma unroll 1
    for (int par = 0; par < 4; ++par) {
      const int pc = par & 1, pr = par >> 1;
      const int ncol = (wk.nc + 1 - pc) >> 1, count = ncol * ((wk.nr + 1 - pr) >> 1);
      const float rcol = 1.0f / (float)ncol;
      for (int e = tid; e < count; e += kT) {
        const int er = (int)(((float)e + 0.5f) * rcol);
        const int row = pr + 2 * er, col = pc + 2 * (e - er * ncol);
        const int start = cnt[row * wk.nc + col], end = cnt[row * wk.nc + col + 1];
        if (end > start) {
          cell_sum(pay, start, end, 1, g);
          cell_add(win + 3 * (row * tc + col), tc, g);
        }
      }
      __syncthreads();
    }
  }
  // the window's touched values, a row of texels per wavefront
  for (int r = wave; r <= wk.nr; r += kWaves) {
    float *G = a.grad_lat[k] + (int64_t)address_coord(wk.r0 + r, lh, mode) * lw * 3;
    for (int i = lane; i < 3 * tc; i += 64) {
      const float x = win[3 * r * tc + i];
      const int c = i / 3;
      const int cg = mode == 1 ? wrap_near(wk.c0 + c, lw, rw) : min(max(wk.c0 + c, 0), lw - 1);
      if (x != 0.0f) unsafeAtomicAdd(G + 3 * cg + (i - 3 * c), x);
    }
  }
}

// Too many samples for the bins' 32-bit indices: every tap of every sample is
// a global atomic.
__global__ __launch_bounds__(256) void scatter_direct_kernel(BackwardArgs a) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= a.n) return;
  const float2 uv = a.uv[s];
  const float *g = a.dx + s * a.dx_stride;
#pragma unroll
  for (int k = 0; k < kMaxLevels; ++k) {
    if (k < a.lat.n_levels) {
      const LevelArgs &L = a.lat.lv[k];
      const Taps t = tap_coords(uv.x, uv.y, L, a.lat.address);
      const float gx = 1.0f - t.fx, gy = 1.0f - t.fy;
      const float w[4] = {gx * gy, t.fx * gy, gx * t.fy, t.fx * t.fy};
      const int ii[4] = {t.i0, t.i1, t.i0, t.i1};
      const int jj[4] = {t.j0, t.j0, t.j1, t.j1};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float *p = a.grad_lat[k] + ((int64_t)jj[q] * L.w + ii[q]) * 3;
        unsafeAtomicAdd(p + 0, w[q] * g[3 * k]);
        unsafeAtomicAdd(p + 1, w[q] * g[3 * k + 1]);
        unsafeAtomicAdd(p + 2, w[q] * g[3 * k + 2]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Forward decode of continuous (float) latents on the FP32 matrix cores: the
// forward half of backward_mfma_kernel (same LDS weight layout, same
// 32-sample steps), ending in the sigmoid and the store. Weights come from
// the packed FP32 image (per layer W [rows_pad][cols_pad], then b).
// ---------------------------------------------------------------------------
template <int MT, int NL>
__global__ __launch_bounds__(64 * kBwdWaves) void forward_mfma_kernel(DecodeArgs a) {
  using M = BwdMap<MT, NL>;
  constexpr int HP = M::HP;
  extern __shared__ float fwd_lds[];
  float *lds = fwd_lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63, h = lane >> 5, c32 = lane & 31;
  const int wave = tid >> 6;
  const PackLayout &L = a.lay;
  const int n_out = a.n_out, n_levels = a.lat.n_levels;
  const float *W0 = reinterpret_cast<const float *>(a.packed + L.w_off[0]);
  const float *B0 = reinterpret_cast<const float *>(a.packed + L.b_off[0]);
  const int hid = L.rows_pad[0] < HP ? L.rows_pad[0] : HP;  // padded rows hold zero weights

  for (int i = tid; i < HP * 16; i += 64 * kBwdWaves) {
    const int row = i >> 4, k = i & 15;
    const int f = slot_feature(k >> 1, k & 1, n_levels);
    float v = 0.0f;
    if (row < hid) v = f >= 0 ? W0[row * L.cols_pad[0] + f] : (f == -2 ? B0[row] : 0.0f);
    lds[M::oW0 + row * M::S0 + k] = v;
  }
#pragma unroll
  for (int l = 1; l <= M::NH; ++l) {
    const float *Wl = reinterpret_cast<const float *>(a.packed + L.w_off[l]);
    for (int i = tid; i < HP * HP; i += 64 * kBwdWaves) {
      const int row = i / HP, col = i % HP;
      lds[M::oWh + (l - 1) * HP * M::SH + row * M::SH + col] =
          (row < L.rows_pad[l] && col < L.cols_pad[l]) ? Wl[row * L.cols_pad[l] + col] : 0.0f;
    }
  }
  {
    const float *Wo = reinterpret_cast<const float *>(a.packed + L.w_off[NL - 1]);
    for (int i = tid; i < 32 * HP; i += 64 * kBwdWaves) {
      const int row = i / HP, col = i % HP;
      lds[M::oWo + row * M::SH + col] =
          (row < L.rows_pad[NL - 1] && col < L.cols_pad[NL - 1]) ? Wo[row * L.cols_pad[NL - 1] + col] : 0.0f;
    }
  }
  for (int i = tid; i < M::nB; i += 64 * kBwdWaves) {
    const int g = i / 32, e = i % 32;  // g = (l - 1) MT + mt, e = 16 h + 4 j + r
    const int l = g / MT + 1 < NL - 1 ? g / MT + 1 : NL - 1;
    const int mt = l == NL - 1 ? 0 : g % MT;
    const int row = 32 * mt + 8 * ((e & 15) >> 2) + 4 * (e >> 4) + (e & 3);
    const float *Bl = reinterpret_cast<const float *>(a.packed + L.b_off[l]);
    lds[M::oB + i] = row < L.rows_pad[l] ? Bl[row] : 0.0f;
  }
  __syncthreads();

  const float *W0s = lds + M::oW0;
  const float *Wos = lds + M::oWo;
  const bf32x16 zero = {};
  const int64_t n_chunks = (a.n + kBwdChunk - 1) / kBwdChunk;
  const int64_t stride = (int64_t)gridDim.x * kBwdWaves;
  for (int64_t chunk = (int64_t)blockIdx.x * kBwdWaves + wave; chunk < n_chunks; chunk += stride) {
    const int64_t smp = chunk * kBwdChunk + c32;
    const bool valid = smp < a.n;
    const float2 uv = a.uv[valid ? smp : a.n - 1];
    float x[8];
    {
      const float3 c0 = sample_f32(a.lat.lv[2 * h], uv.x, uv.y, a.lat.address);
      const float3 c1 = sample_f32(a.lat.lv[2 * h + 1], uv.x, uv.y, a.lat.address);
      x[0] = c0.x; x[1] = c0.y; x[2] = c0.z;
      x[3] = c1.x; x[4] = c1.y; x[5] = c1.z;
      x[6] = h ? uv.y : uv.x;
      x[7] = h ? 0.0f : 1.0f;
    }
    bf32x16 act[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      bf32x16 z = zero;
#pragma unroll
      for (int s = 0; s < 8; ++s) z = mfma32(W0s[(32 * mt + c32) * M::S0 + 2 * s + h], x[s], z);
#pragma unroll
      for (int i = 0; i < 16; ++i) z[i] = fmaxf(z[i], 0.0f);
      act[mt] = z;
    }
#pragma unroll
    for (int l = 1; l <= M::NH; ++l) {
      const float *Wl = lds + M::oWh + (l - 1) * HP * M::SH;
      bf32x16 nx[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bf32x4 *bp = reinterpret_cast<const bf32x4 *>(lds + M::bias(l, mt) + 16 * h);
        const bf32x4 b0 = bp[0], b1 = bp[1], b2 = bp[2], b3 = bp[3];
        bf32x16 z = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3],
                     b2[0], b2[1], b2[2], b2[3], b3[0], b3[1], b3[2], b3[3]};
#pragma unroll
        for (int s = 0; s < 16 * MT; ++s)
          z = mfma32(Wl[(32 * mt + c32) * M::SH + chain_unit(s, h)], act[s >> 4][s & 15], z);
#pragma unroll
        for (int i = 0; i < 16; ++i) z[i] = fmaxf(z[i], 0.0f);
        nx[mt] = z;
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) act[mt] = nx[mt];
    }
    const bf32x4 *bp = reinterpret_cast<const bf32x4 *>(lds + M::bias(NL - 1, 0) + 16 * h);
    const bf32x4 b0 = bp[0], b1 = bp[1];
    bf32x16 z = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3], 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < 16 * MT; ++s) z = mfma32(Wos[c32 * M::SH + chain_unit(s, h)], act[s >> 4][s & 15], z);
    if (valid) {
      // rows 8 j + 4 h + r (j < 2, r < 4) of this lane's sample
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int row0 = 8 * j + 4 * h;
        if (row0 >= n_out) continue;
        float f[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) f[r] = 1.0f / (1.0f + expf(-z[4 * j + r]));
        if (a.out_f16) {
          _Float16 *o = reinterpret_cast<_Float16 *>(a.out) + smp * n_out + row0;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (row0 + r < n_out) o[r] = (_Float16)f[r];
        } else {
          float *o = reinterpret_cast<float *>(a.out) + smp * n_out + row0;
          if ((n_out & 3) == 0) {
            *reinterpret_cast<float4 *>(o) = make_float4(f[0], f[1], f[2], f[3]);
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (row0 + r < n_out) o[r] = f[r];
          }
        }
      }
    }
  }
}

hipError_t launch_forward_f32(const DecodeArgs &a, const MlpShape &s, hipStream_t st) {
  const int groups = backward_groups(a.n);
  auto go = [&](auto kernel, size_t floats) {
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(64 * kBwdWaves), floats * sizeof(float), st, a);
    return hipGetLastError();
  };
  const int mt = s.hid > 32 ? 2 : 1;
  if (mt == 1) {
    switch (s.n_layers) {
      case 2: return go(forward_mfma_kernel<1, 2>, BwdMap<1, 2>::oStage);
      case 3: return go(forward_mfma_kernel<1, 3>, BwdMap<1, 3>::oStage);
      case 4: return go(forward_mfma_kernel<1, 4>, BwdMap<1, 4>::oStage);
      default: return hipErrorInvalidValue;
    }
  }
  switch (s.n_layers) {
    case 2: return go(forward_mfma_kernel<2, 2>, BwdMap<2, 2>::oStage);
    case 3: return go(forward_mfma_kernel<2, 3>, BwdMap<2, 3>::oStage);
    case 4: return go(forward_mfma_kernel<2, 4>, BwdMap<2, 4>::oStage);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_backward(const BackwardArgs &a, const MlpShape &s, float *const *grad_W, float *const *grad_b,
                           hipStream_t st) {
  // latent gradients start at zero (fill kernel: no memset nodes in graphs)
  for (int k = 0; k < a.lat.n_levels; ++k) {
    hipError_t e = launch_fill_f32(a.grad_lat[k], (int64_t)a.lat.lv[k].w * a.lat.lv[k].h * 3, 0.0f, st);
    if (e != hipSuccess) return e;
  }
  hipError_t e;
  {
    const int groups = a.n_blocks / kBwdWaves;
    auto go = [&](auto kernel, size_t floats) {
      hipLaunchKernelGGL(kernel, dim3(groups), dim3(64 * kBwdWaves), floats * sizeof(float), st, a);
      return hipGetLastError();
    };
    const int mt = s.hid > 32 ? 2 : 1;
    if (mt == 1) {
      switch (s.n_layers) {
        case 2: e = go(backward_mfma_kernel<1, 2>, BwdMap<1, 2>::total); break;
        case 3: e = go(backward_mfma_kernel<1, 3>, BwdMap<1, 3>::total); break;
        case 4: e = go(backward_mfma_kernel<1, 4>, BwdMap<1, 4>::total); break;
        default: return hipErrorInvalidValue;
      }
    } else {
      switch (s.n_layers) {
        case 2: e = go(backward_mfma_kernel<2, 2>, BwdMap<2, 2>::total); break;
        case 3: e = go(backward_mfma_kernel<2, 3>, BwdMap<2, 3>::total); break;
        case 4: e = go(backward_mfma_kernel<2, 4>, BwdMap<2, 4>::total); break;
        default: return hipErrorInvalidValue;
      }
    }
  }
  if (e != hipSuccess) return e;
  ReduceArgs r;
  r.part = a.wpart;
  r.n_blocks = a.n_blocks;
  r.n_params = a.n_params;
  r.n_layers = s.n_layers;
  for (int l = 0; l <= s.n_layers; ++l) r.dims[l] = a.dims[l];
  for (int l = 0; l < s.n_layers; ++l) {
    r.W[l] = grad_W[l];
    r.b[l] = grad_b[l];
  }
  hipLaunchKernelGGL(reduce_f64_kernel, dim3((a.n_params + 63) / 64), dim3(64 * kReduceWaves), 0, st, r);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // latent gradients from dx
  if (a.n_bins == 0) {
    hipLaunchKernelGGL(scatter_direct_kernel, dim3((unsigned)((a.n + 255) / 256)), dim3(256), 0, st, a);
    return hipGetLastError();
  }
  if ((e = launch_fill_f32(reinterpret_cast<float *>(a.bin_count), a.n_bins, 0.0f, st)) != hipSuccess) return e;
  const unsigned grid = (unsigned)((a.n + kBinSamplesPerBlock - 1) / kBinSamplesPerBlock);
  hipLaunchKernelGGL(bin_count_kernel, dim3(grid), dim3(256), a.n_bins * sizeof(int32_t), st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(bin_scan_kernel, dim3(1), dim3(1024), 0, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(bin_scatter_kernel, dim3(grid), dim3(256), 2 * a.n_bins * sizeof(int32_t), st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(bin_accum_kernel, dim3((unsigned)((a.n_runs + 7) / 8 * 8 * a.lat.n_levels)), dim3(kAccThreads),
                     (size_t)(a.bin_lds + 5 * kBinRun + a.bin_cells + 1) * sizeof(float), st, a);
  return hipGetLastError();
}

}  // namespace ntc
