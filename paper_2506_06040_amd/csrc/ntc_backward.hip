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
// channel (taps outside a window, and the samples of sparse bins, go straight to
// global atomics).
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

// Matrix-core backward: workgroups of 4 or 8 wavefronts (one or two per SIMD),
// each wavefront taking kBwdChunk samples per step; one row of partial
// weight-gradient sums per wavefront that has samples.
constexpr int kBwdChunk = 32;
constexpr int kBwdMaxGroups = 256;

// Wavefronts per workgroup: two per SIMD (256 registers each) cover each
// other's waits; the 64-wide networks of four layers need the registers of
// one per SIMD for their gradient accumulators.
static constexpr int backward_waves(int mt, int n_layers) { return mt == 2 && n_layers > 3 ? 4 : 8; }

// A short batch spreads over the compute units first: two wavefronts of a SIMD halve
// each other's matrix rate (forward of 300 to 4096 samples: 14-64-64-64-8 16.3 ->
// 11.3 us, 14-64-64-8 11.3 -> 8.2).
static int backward_groups(int64_t n) {
  const int64_t chunks = (n + kBwdChunk - 1) / kBwdChunk;
  return (int)(chunks > kBwdMaxGroups ? kBwdMaxGroups : (chunks < 1 ? 1 : chunks));
}

// First chunk of a wavefront of this workgroup, and its row of partial sums:
// neighbours in one workgroup where every wavefront has one (`full`; rows 256
// apart cost 3.5 us for 14-64-64-8), over the workgroups first where not.
__device__ __forceinline__ int first_chunk(bool full, int waves, int wave) {
  return full ? (int)blockIdx.x * waves + wave : wave * (int)gridDim.x + (int)blockIdx.x;
}

// Wavefronts that have a chunk, each of which writes a row of partial sums.
static int backward_blocks(const MlpShape &s, int64_t n) {
  const int64_t chunks = (n + kBwdChunk - 1) / kBwdChunk;
  const int all = backward_waves(s.hid > 32 ? 2 : 1, s.n_layers) * backward_groups(n);
  return (int)(chunks > all ? all : (chunks < 1 ? 1 : chunks));
}

// Spatial bins of the latent-gradient scatter: squares of 2^kBinShift (or a
// larger power of two, keeping at most kMaxBins bins) level-0 texels.
constexpr int kBinShift = 5;
constexpr int kMaxBins = 4096;
// Samples and threads per workgroup of the count / scatter passes. Larger
// shares need fewer global atomics (one per workgroup and bin) but leave CUs
// idle; more threads hide the latency of the loads, which are requested
// together (us, count + scatter at 2^20 / 2^18 samples: 4096 by 256 threads 12.5
// + 17.4 / 9.6 + 10.4, by 512 9.3 + 14.9 / 5.5 + 7.9, by 1024 8.5 + 14.1 /
// 4.9 + 7.3; 8192 by 1024 7.1 + 13.6 / 6.5 + 10.9; 2048 by 512 12.9 + 20.9 /
// 5.3 + 6.9).
constexpr int kBinSamplesPerBlock = 4096;
constexpr int kBinThreads = 1024;
constexpr int kBinRun = 1120;              // samples of a bin taken by one workgroup of the accumulation
constexpr int kAccThreads = 512;           // threads of that workgroup
constexpr int kBinWindowFloats = 12288;    // largest LDS of a bin's texel window (48 KB)
constexpr int kBinWindowCells = 4096;      // largest number of cells of one window
// Samples of a bin up to which they are added straight to the gradients (a run
// costs its window, whatever it holds), and the mean per bin up to which bins are
// looked at for that (the look costs 10 us at 2^18 samples). Random samples, whole
// backward in us, runs alone / with sparse bins: 2048^2..256^2 levels, mean of 4 per
// bin 231 / 108, 16 269 / 206, 32 314 / 316, 64 396 / 402; 1024^2..128^2, 16 90 / 79,
// 32 93 / 97; up to 16 and 48 samples in place of 32: 226 and 205 in place of 206.
constexpr int kBinSparse = 32;
constexpr int kBinSparseMean = 24;

// LDS of one bin: floats and cells of its largest texel window that fits (none
// where no level's does).
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
    const int64_t f = 3 * (nc + 1) * (nr + 1), c = nc * nr;
    if (f > kBinWindowFloats || c > kBinWindowCells) continue;
    most_f = std::max(most_f, f);
    most_c = std::max(most_c, c);
  }
  floats = (int)most_f;
  cells = (int)most_c;
}

static size_t align256(size_t v) { return (v + 255) / 256 * 256; }

BwdLayout backward_layout(const MlpShape &s, const LatArgs &lat, int64_t n) {
  BwdLayout L{};
  L.n_blocks = backward_blocks(s, n);
  L.n_params = n_params_of(s);
  L.n_feat = 3 * lat.n_levels;
  L.dx_stride = (L.n_feat + 2 + 3) & ~3;
  // Sample indices of the bins are int32, and so is the end of the run that
  // follows the last one of a bin holding all samples.
  int t = kBinShift;
  if (n <= INT32_MAX - kBinRun) {
    const int w = lat.lv[0].w, h = lat.lv[0].h;
    auto bins = [&](int len) { return (len + (1 << t) - 1) >> t; };
    while ((int64_t)bins(w) * bins(h) > kMaxBins) ++t;
    bin_window(lat, t, L.bin_lds, L.bin_cells);
    const int64_t n_bins = (int64_t)bins(w) * bins(h);
    L.bin_sparse = n <= n_bins * kBinSparseMean ? kBinSparse : 0;
    if (L.bin_cells > 0 && n > L.bin_sparse) {
      L.bin_shift = t;
      L.bins_x = bins(w);
      L.n_bins = (int32_t)n_bins;
      L.n_runs = (int32_t)(std::min<int64_t>(n_bins, n / (L.bin_sparse + 1)) + n / kBinRun);
    }
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
// Pass 1 on the matrix cores (FP32 operands and accumulation)
//
// A wavefront takes 32 samples per step. The products over hidden units are
// v_mfma_f32_32x32x2 tiles of units x samples: the weights are the A operand
// (row = output unit, one float per lane), the layer input the B operand. In
// the accumulator a lane holds rows 8 j + 4 h + r (j, r < 4, h = lane / 32)
// of sample lane % 32; K-step t of a product whose input is such a tile takes
// element t of it (lane half h supplying unit 8 (t / 4) + 4 h + t % 4 of the
// tile), so layers chain in registers in both directions. The first layer's
// K-slots hold per lane half two levels' features: slot 2 s + h is channel
// s % 3 of level 2 h + s / 3 (s < 6), u or v (s = 6), the constant 1 that
// carries the bias (s = 7, h = 0) or padding.
//
// Products with at most 16 output rows (the output layer, the feature
// gradients) take v_mfma_f32_16x16x1_4b, half the matrix time of a padded
// 32-row tile: block b = lane / 16 multiplies its own 16 columns, which are
// samples 16 (b % 2) .. + 15 and the units of lane half b / 2, so an
// accumulator tile is its B operand as it stands; blocks b and b + 2 are added
// at the end, and a lane then holds rows 4 (lane / 16) + r of samples
// lane % 16 and 16 + lane % 16.
//
// Weight gradients contract over the samples: the deltas and layer inputs
// are written to LDS as [unit][sample] and read back with a unit per lane,
// 32x32x2 tiles for hidden layers (lane half h: samples 16 h ..), 16x16x4
// tiles where one side has at most 16 rows (lane / 16 = g: samples 8 g ..).
// The buffers are [sample / 4][unit][sample % 4] with a pad of one unit, so
// that neither the writes (32 samples of a unit) nor the reads (float4s of
// consecutive units) meet bank conflicts and every offset is an immediate.
// Bias gradients are row sums of the staged deltas.
//
// Matrix time bounds both kernels, and the vector instructions add to it:
// FP32 matrix and vector work of one SIMD hardly overlap (64 instructions
// less per step were worth 10 us of 2^20 samples). Hence the float4 weight
// reads, the 16-row products (280 in place of 344 units of 64 matrix cycles
// per step of 14-64-64-8) and two wavefronts per SIMD, which cover each
// other's texel loads and LDS round trips. 2^20 random samples, 14-64-64-8,
// 1024^2..128^2 levels: backward 558 -> 363 us (95 TFLOP/s of products that
// count), forward 188 -> 145 us, against one wavefront per SIMD, padded
// 32-row output tiles and level parameters fetched per lane.
// ---------------------------------------------------------------------------
typedef float bf32x16 __attribute__((ext_vector_type(16)));
typedef float bf32x4 __attribute__((ext_vector_type(4)));

constexpr int kLevelFloats = sizeof(LevelSel) / sizeof(float) + 2;  // a multiple of 4

__device__ __forceinline__ void load_levels(float *tab, const LatArgs &lat, int tid) {
  if (tid < kMaxLevels) *reinterpret_cast<LevelSel *>(tab + kLevelFloats * tid) = level_sel(lat.lv[tid]);
}

template <int MT, int NL>
struct BwdMap {
  static constexpr int waves = backward_waves(MT, NL);
  static constexpr int HP = 32 * MT;        // padded hidden width
  static constexpr int S0 = 20;             // row stride of the first layer (K-slots, lane half 0's 8 first)
  static constexpr int SH = HP + 4;         // row stride of the other layers (float4 reads of 8 rows: no conflicts)
  static constexpr int NH = NL - 2;         // hidden-to-hidden layers
  static constexpr int oW0 = 0;
  static constexpr int oWh = oW0 + HP * S0;
  static constexpr int oWo = oWh + NH * HP * SH;         // 16 output rows
  static constexpr int oB = oWo + 16 * SH;               // bias fragments [layer 1..NL-2][mt][h][16]
  static constexpr int oBo = oB + NH * MT * 32;          // output biases [16]
  static constexpr int oLv = oBo + 16;                   // level parameters
  static constexpr int oStage = oLv + kLevelFloats * kMaxLevels;
  static constexpr int SQ = 4 * (HP + 1);                // stride of a staged group of 4 samples
  static constexpr int stage = 2 * 8 * SQ;               // per wavefront: two buffers of HP units
  static constexpr int total = oStage + waves * stage;
  __device__ static int bias(int l, int mt) { return oB + ((l - 1) * MT + mt) * 32; }  // l = 1 .. NL - 2
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

// Weights and biases into LDS, zero-padded, shared by the workgroup's
// T threads. W(l), b(l): element functions of layer l's matrix and bias.
template <int MT, int NL, int T, class FW, class FB>
__device__ __forceinline__ void load_weights(float *lds, int tid, int n_levels, FW W, FB b) {
  using M = BwdMap<MT, NL>;
  constexpr int HP = M::HP;
  for (int i = tid; i < HP * 16; i += T) {
    const int row = i >> 4, k = i & 15;
    const int f = slot_feature(k >> 1, k & 1, n_levels);
    lds[M::oW0 + row * M::S0 + 8 * (k & 1) + (k >> 1)] = f >= 0 ? W(0, row, f) : (f == -2 ? b(0, row) : 0.0f);
  }
#pragma unroll
  for (int l = 1; l <= M::NH; ++l)
    for (int i = tid; i < HP * HP; i += T)
      lds[M::oWh + (l - 1) * HP * M::SH + (i / HP) * M::SH + i % HP] = W(l, i / HP, i % HP);
  for (int i = tid; i < 16 * HP; i += T) lds[M::oWo + (i / HP) * M::SH + i % HP] = W(NL - 1, i / HP, i % HP);
  for (int i = tid; i < M::NH * MT * 32; i += T) {
    const int g = i / 32, e = i % 32;  // g = (l - 1) MT + mt, e = 16 h + 4 j + r
    lds[M::oB + i] = b(g / MT + 1, 32 * (g % MT) + 8 * ((e & 15) >> 2) + 4 * (e >> 4) + (e & 3));
  }
  if (tid < 16) lds[M::oBo + tid] = b(NL - 1, tid);
}

// Features of a lane half's K-slots: the values of sample_f32(), with the
// loads of both levels in flight together (the level parameters come from
// LDS, the address mode is one uniform branch).
__device__ __forceinline__ void first_slots(const float *tab, int mode, float2 uv, int h, float (&x)[8]) {
  LevelSel L[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) L[j] = *reinterpret_cast<const LevelSel *>(tab + kLevelFloats * (2 * h + j));
  float fx[2], fy[2];
  int i0[2], i1[2], j0[2], j1[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    float px = fmaf(uv.x, L[j].fw, -0.5f) + L[j].sx;
    float py = fmaf(uv.y, L[j].fh, -0.5f) + L[j].sy;
    px = fminf(fmaxf(px, -16777216.0f), 16777216.0f);
    py = fminf(fmaxf(py, -16777216.0f), 16777216.0f);
    const float xf = floorf(px), yf = floorf(py);
    fx[j] = px - xf;
    fy[j] = py - yf;
    i0[j] = (int)xf;
    j0[j] = (int)yf;
  }
  if (mode == 1) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      i0[j] = wrap_near(i0[j], L[j].w, L[j].rw);
      j0[j] = wrap_near(j0[j], L[j].h, L[j].rh);
      i1[j] = i0[j] + 1 == L[j].w ? 0 : i0[j] + 1;
      j1[j] = j0[j] + 1 == L[j].h ? 0 : j0[j] + 1;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      i1[j] = min(max(i0[j] + 1, 0), L[j].w - 1);
      j1[j] = min(max(j0[j] + 1, 0), L[j].h - 1);
      i0[j] = min(max(i0[j], 0), L[j].w - 1);
      j0[j] = min(max(j0[j], 0), L[j].h - 1);
    }
  }
  float t[2][4][3];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const auto *p = (const __attribute__((address_space(1))) float *)L[j].grid +
                      ((int64_t)((q >> 1) ? j1[j] : j0[j]) * L[j].w + ((q & 1) ? i1[j] : i0[j])) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) t[j][q][c] = p[c];
    }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const float gx = 1.0f - fx[j], gy = 1.0f - fy[j];
    const float w[4] = {gx * gy, fx[j] * gy, gx * fy[j], fx[j] * fy[j]};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float v = 0.0f;
#pragma unroll
      for (int q = 0; q < 4; ++q) v = fmaf(w[q], t[j][q][c], v);
      x[3 * j + c] = v;
    }
  }
  x[6] = h ? uv.y : uv.x;
  x[7] = h ? 0.0f : 1.0f;
}

// max(z, 0), 0 for NaN, as a median with an infinity that the compiler does
// not see: fmaxf() costs a second instruction that quiets NaN first.
__device__ __forceinline__ float relu(float z) {
  float inf;
  asm("s_mov_b32 %0, 0x7f800000" : "=s"(inf));
  return __builtin_amdgcn_fmed3f(z, 0.0f, inf);
}

// ReLU outputs of tile mt of the first layer, and of hidden layer l from its
// input tiles.
template <int MT, int NL>
__device__ __forceinline__ bf32x16 first_tile(const float *lds, int mt, int c32, int h, const float (&x)[8]) {
  using M = BwdMap<MT, NL>;
  bf32x16 z = {};
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bf32x4 w = *reinterpret_cast<const bf32x4 *>(lds + M::oW0 + (32 * mt + c32) * M::S0 + 8 * h + 4 * q);
#pragma unroll
    for (int r = 0; r < 4; ++r) z = mfma32(w[r], x[4 * q + r], z);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = relu(z[i]);
  return z;
}

template <int MT, int NL>
__device__ __forceinline__ bf32x16 hidden_tile(const float *lds, int l, int mt, int c32, int h,
                                               const bf32x16 (&in)[MT]) {
  using M = BwdMap<MT, NL>;
  const float *Wl = lds + M::oWh + (l - 1) * M::HP * M::SH;
  const bf32x4 *bp = reinterpret_cast<const bf32x4 *>(lds + M::bias(l, mt) + 16 * h);
  const bf32x4 b0 = bp[0], b1 = bp[1], b2 = bp[2], b3 = bp[3];
  bf32x16 z = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3],
               b2[0], b2[1], b2[2], b2[3], b3[0], b3[1], b3[2], b3[3]};
#pragma unroll
  for (int q = 0; q < 4 * MT; ++q) {
    const bf32x4 w = *reinterpret_cast<const bf32x4 *>(Wl + (32 * mt + c32) * M::SH + 8 * q + 4 * h);
#pragma unroll
    for (int r = 0; r < 4; ++r) z = mfma32(w[r], in[q >> 2][4 * (q & 3) + r], z);
  }
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = relu(z[i]);
  return z;
}

// Outputs of 32 samples as rows16 gives them, spread over the lanes: with at
// most 8 rows the lanes that hold rows 8 .. 15 take the second samples of the
// others (one value per lane and row instead of two, half of them padding).
struct OutRows {
  int n, row0, smp[2];  // vectors of 4 rows from row0, of samples smp[..]
  bf32x4 z[2];
};
__device__ __forceinline__ OutRows spread_rows(int n_out, int g16, int c16, const bf32x4 &first, const bf32x4 &second) {
  OutRows o;
  o.z[0] = first;
  o.z[1] = second;
  o.n = 2;
  o.row0 = 4 * g16;
  o.smp[0] = c16;
  o.smp[1] = 16 + c16;
  if (n_out <= 8) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // lanes 32 .. 63 get `second` of lanes 0 .. 31
      const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(first[r]), __float_as_uint(second[r]), false, false);
      o.z[0][r] = __uint_as_float(t[0]);
    }
    o.n = 1;
    o.row0 = 4 * (g16 & 1);
    o.smp[0] = 16 * (g16 >> 1) + c16;
  }
  return o;
}

// Product of a 16-row matrix (wt(q): this lane's elements for K-steps 4 q ..
// 4 q + 3) with MT accumulator tiles, plus `bias` rows: rows 4 (lane / 16) + r of samples
// lane % 16 (first) and 16 + lane % 16 (second).
template <int MT, class FW>
__device__ __forceinline__ void rows16(FW wt, const bf32x16 (&in)[MT], bf32x4 bias, bf32x4 &first, bf32x4 &second) {
  bf32x16 z = {bias[0], bias[1], bias[2], bias[3], bias[0], bias[1], bias[2], bias[3], 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < 4 * MT; ++q) {
    const bf32x4 w = wt(q);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      z = __builtin_amdgcn_mfma_f32_16x16x1f32(w[r], in[q >> 2][4 * (q & 3) + r], z, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    first[r] = z[r] + z[8 + r];
    second[r] = z[4 + r] + z[12 + r];
  }
}

template <int MT, int NL>
__global__ __launch_bounds__((64 * backward_waves(MT, NL)))
__attribute__((amdgpu_waves_per_eu((backward_waves(MT, NL) / 4), (backward_waves(MT, NL) / 4))))
void backward_mfma_kernel(BackwardArgs a) {
  using M = BwdMap<MT, NL>;
  constexpr int HP = M::HP, NH1 = M::NH > 0 ? M::NH : 1;
  extern __shared__ float bwd_lds[];
  float *lds = bwd_lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63, h = lane >> 5, c32 = lane & 31, c16 = lane & 15, g16 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hid = a.dims[1], n_out = a.dims[NL], d0 = a.dims[0];
  const int n_levels = a.lat.n_levels;

  load_weights<MT, NL, 64 * M::waves>(
      lds, tid, n_levels,
      [&](int l, int row, int col) {
        const int rows = l == NL - 1 ? n_out : hid, cols = l == 0 ? d0 : hid;
        return row < rows && col < cols ? a.W[l][row * cols + col] : 0.0f;
      },
      [&](int l, int row) { return row < (l == NL - 1 ? n_out : hid) ? a.b[l][row] : 0.0f; });
  load_levels(lds + M::oLv, a.lat, tid);
  float *Dt = lds + M::oStage + wave * M::stage;  // deltas
  float *At = Dt + 8 * M::SQ;                     // layer inputs
  __syncthreads();

  const bf32x16 zero = {};

  // weight-gradient accumulators: first layer (16-row tiles, columns =
  // K-slots), hidden layers [l][mt][nt], output layer (16-column tiles); bias
  // gradients of rows `lane`
  bf32x4 g0[2 * MT] = {}, go[2 * MT] = {};
  bf32x16 gh[NH1][MT][MT];
  float gbh[NH1], gbo = 0.0f;
#pragma unroll
  for (int l = 0; l < NH1; ++l) {
    gbh[l] = 0.0f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j) gh[l][i][j] = zero;
  }

  // element (row, sample) of a staged buffer, and float4 q of a row
  auto at = [](int row, int smp) { return (smp >> 2) * M::SQ + 4 * row + (smp & 3); };
  auto quad = [](const float *buf, int row, int q) {
    return *reinterpret_cast<const bf32x4 *>(buf + q * M::SQ + 4 * row);
  };
  // a tile in accumulator layout -> rows [row0, row0 + 32) of a buffer
  // (tile_at: this lane's first element)
  auto stage_tile = [](float *buf, int tile_at, int row0, const bf32x16 &t) {
#pragma unroll
    for (int i = 0; i < 16; ++i) buf[4 * (row0 + 8 * (i >> 2) + (i & 3)) + tile_at] = t[i];
  };
  // ReLU mask: v where the activation staged in rows [row0, row0 + 32) of At
  // is positive (read back from LDS: its registers are free after staging)
  auto mask_tile = [](const float *buf, int tile_at, int row0, const bf32x16 &v) {
    bf32x16 m;
#pragma unroll
    for (int i = 0; i < 16; ++i) m[i] = buf[4 * (row0 + 8 * (i >> 2) + (i & 3)) + tile_at] > 0.0f ? v[i] : 0.0f;
    return m;
  };
  // sum over the 32 samples of staged row `row`
  auto row_sum = [&](const float *buf, int row) {
    float sum = 0.0f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bf32x4 x = quad(buf, row, q);
      sum += (x[0] + x[1]) + (x[2] + x[3]);
    }
    return sum;
  };
  auto lds_order = [] { asm volatile("" ::: "memory"); };  // a wavefront's LDS accesses complete in order

  const int64_t n_chunks = (a.n + kBwdChunk - 1) / kBwdChunk;
  const int64_t stride = (int64_t)gridDim.x * M::waves;
  const int64_t first = first_chunk(a.n_blocks == M::waves * (int)gridDim.x, M::waves, wave);
  auto load_uv = [&](int64_t chunk) {
    const int64_t smp = chunk * kBwdChunk + c32;
    return a.uv[smp < a.n ? smp : a.n - 1];
  };
  float2 uv_next = load_uv(first);
  for (int64_t chunk = first; chunk < n_chunks; chunk += stride) {
    const float2 uv = uv_next;
    uv_next = load_uv(chunk + stride < n_chunks ? chunk + stride : chunk);
    const int64_t s0 = chunk * kBwdChunk;
    // weights, level parameters and addresses are read or computed where they
    // are used, not held in registers across steps (opaque_zero)
    const float *wl = lds + opaque_zero((int)chunk);
    const int ln = lane + opaque_zero((int)chunk);
    const int h = ln >> 5, c32 = ln & 31, c16 = ln & 15, g16 = ln >> 4;
    const int tile_at = at(4 * h, c32);

    // ---- forward
    float x[8];
    first_slots(wl + M::oLv, a.lat.address, uv, h, x);
    bf32x16 act[NL - 1][MT];  // ReLU outputs of the hidden layers
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) act[0][mt] = first_tile<MT, NL>(wl, mt, c32, h, x);
#pragma unroll
    for (int l = 1; l <= M::NH; ++l)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) act[l][mt] = hidden_tile<MT, NL>(wl, l, mt, c32, h, act[l - 1]);
    bf32x4 zo[2];
    rows16<MT>([&](int q) { return *reinterpret_cast<const bf32x4 *>(wl + M::oWo + c16 * M::SH + 8 * q + 4 * h); }, act[NL - 2],
               *reinterpret_cast<const bf32x4 *>(wl + M::oBo + 4 * g16), zo[0], zo[1]);

    // ---- output deltas g f (1 - f), staged
    lds_order();
    const OutRows zr = spread_rows(n_out, g16, c16, zo[0], zo[1]);
    auto out_delta = [&](int e) {
      float g[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t smp = min(s0 + zr.smp[e], a.n - 1);
        g[r] = a.grad_out[smp * n_out + min(zr.row0 + r, n_out - 1)];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = zr.row0 + r;
        const float f = 1.0f / (1.0f + expf(-zr.z[e][r]));
        const int keep = row < n_out && s0 + zr.smp[e] < a.n ? -1 : 0;  // a select here becomes branches
        Dt[at(row, zr.smp[e])] = __int_as_float(__float_as_int(g[r] * f * (1.0f - f)) & keep);
      }
    };
    out_delta(0);
    if (zr.n > 1) {
      out_delta(1);
    } else {  // rows 8 .. 15 of the padded product
#pragma unroll
      for (int r = 0; r < 4; ++r) Dt[at(8 + zr.row0 + r, zr.smp[0])] = 0.0f;
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) stage_tile(At, tile_at, 32 * mt, act[NL - 2][mt]);
    lds_order();
    // ---- output layer: delta of the last hidden layer, weight and bias gradients
    bf32x16 del[MT];
    {
      auto steps = [&](int t0) {
#pragma unroll
        for (int t = t0; t < t0 + 4; ++t) {
          const float dv = Dt[at(2 * t + h, c32)];
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            del[mt] = mfma32(wl[M::oWo + (2 * t + h) * M::SH + 32 * mt + c32], dv, del[mt]);
        }
      };
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) del[mt] = zero;
      steps(0);
      if (n_out > 8) steps(4);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) del[mt] = mask_tile(At, tile_at, 32 * mt, del[mt]);
    }
    {
      const bf32x4 a0 = quad(Dt, c16, 2 * g16), a1 = quad(Dt, c16, 2 * g16 + 1);
#pragma unroll
      for (int nt = 0; nt < 2 * MT; ++nt) {
        const bf32x4 b0 = quad(At, 16 * nt + c16, 2 * g16), b1 = quad(At, 16 * nt + c16, 2 * g16 + 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) go[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[q], b0[q], go[nt], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) go[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[q], b1[q], go[nt], 0, 0, 0);
      }
      if (ln < 16) gbo += row_sum(Dt, ln);
    }
    // ---- hidden layers, top down
#pragma unroll
    for (int l = M::NH; l >= 1; --l) {
      const float *Wl = wl + M::oWh + (l - 1) * HP * M::SH;
      lds_order();
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        stage_tile(Dt, tile_at, 32 * mt, del[mt]);
        stage_tile(At, tile_at, 32 * mt, act[l - 1][mt]);
      }
      lds_order();
      bf32x16 nd[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) nd[mt] = zero;
#pragma unroll
      for (int q = 0; q < 4 * MT; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            nd[mt] = mfma32(Wl[(8 * q + 4 * h + r) * M::SH + 32 * mt + c32], del[q >> 2][4 * (q & 3) + r], nd[mt]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) nd[mt] = mask_tile(At, tile_at, 32 * mt, nd[mt]);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        bf32x4 av[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) av[q] = quad(Dt, 32 * mt + c32, 4 * h + q);
#pragma unroll
        for (int nt = 0; nt < MT; ++nt)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bf32x4 bv = quad(At, 32 * nt + c32, 4 * h + q);
#pragma unroll
            for (int r = 0; r < 4; ++r) gh[l - 1][mt][nt] = mfma32(av[q][r], bv[r], gh[l - 1][mt][nt]);
          }
      }
      if (ln < HP) gbh[l - 1] += row_sum(Dt, ln);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) del[mt] = nd[mt];
    }
    // ---- first layer: weight gradients over the K-slots (slot 14 = bias)
    lds_order();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) stage_tile(Dt, tile_at, 32 * mt, del[mt]);
#pragma unroll
    for (int s = 0; s < 8; ++s) At[at(2 * s + h, c32)] = x[s];
    lds_order();
    {
      const bf32x4 b0 = quad(At, c16, 2 * g16), b1 = quad(At, c16, 2 * g16 + 1);
#pragma unroll
      for (int mt = 0; mt < 2 * MT; ++mt) {
        const bf32x4 a0 = quad(Dt, 16 * mt + c16, 2 * g16), a1 = quad(Dt, 16 * mt + c16, 2 * g16 + 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) g0[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[q], b0[q], g0[mt], 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) g0[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[q], b1[q], g0[mt], 0, 0, 0);
      }
    }
    // ---- feature gradient dx = W0^T D0, one row of a.dx per sample: the
    // latent features' gradients, then u, v (slots 12 and 13)
    {
      const int lvl = c16 / 3;
      const int slot = lvl < n_levels && c16 < 12 ? 8 * (lvl >> 1) + 3 * (lvl & 1) + c16 % 3 : 15;  // 15: zeros
      bf32x4 dx[2];
      const bf32x4 none = {};
      rows16<MT>(
          [&](int q) {
            const float *w = wl + M::oW0 + (8 * q + 4 * h) * M::S0 + slot;
            return bf32x4{w[0], w[M::S0], w[2 * M::S0], w[3 * M::S0]};
          },
          del, none, dx[0], dx[1]);
      if (4 * g16 < a.dx_stride) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int smp = 16 * e + c16;
          const float u = At[at(12, smp)], v = At[at(13, smp)];
          float4 o;
          float *po = &o.x;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            po[r] = 4 * g16 + r == a.n_feat ? u : 4 * g16 + r == a.n_feat + 1 ? v : dx[e][r];
          if (s0 + smp < a.n) *reinterpret_cast<float4 *>(a.dx + (s0 + smp) * a.dx_stride + 4 * g16) = o;
        }
      }
    }
  }

  // ---- this wavefront's partial sums (parameters in unpadded order)
  const int part_row = first_chunk(a.n_blocks == M::waves * (int)gridDim.x, M::waves, wave);
  if (part_row >= a.n_blocks) return;
  float *part = a.wpart + (int64_t)part_row * a.n_params;
  int off = 0;
  {
    const int f = slot_feature(c16 >> 1, c16 & 1, n_levels);
#pragma unroll
    for (int mt = 0; mt < 2 * MT; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * mt + 4 * g16 + r;
        if (row < hid && f >= 0) part[off + row * d0 + f] = g0[mt][r];
        if (row < hid && f == -2) part[off + hid * d0 + row] = g0[mt][r];
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
  for (int nt = 0; nt < 2 * MT; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * g16 + r, col = 16 * nt + c16;
      if (row < n_out && col < hid) part[off + row * hid + col] = go[nt][r];
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
__global__ __launch_bounds__(kBinThreads) void bin_count_kernel(BackwardArgs a) {
  extern __shared__ int32_t hist[];
  for (int k = threadIdx.x; k < a.n_bins; k += kBinThreads) hist[k] = 0;
  __syncthreads();
  const int64_t s0 = (int64_t)blockIdx.x * kBinSamplesPerBlock;
  constexpr int kPer = kBinSamplesPerBlock / kBinThreads;
  float2 uv[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int64_t s = s0 + threadIdx.x + kBinThreads * i;
    uv[i] = a.uv[s < a.n ? s : a.n - 1];
  }
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (s0 + threadIdx.x + kBinThreads * i < a.n) atomicAdd(&hist[bin_of(a, uv[i])], 1);
  __syncthreads();
  for (int k = threadIdx.x; k < a.n_bins; k += kBinThreads)
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
// bin_accum_kernel: the samples of every bin of more than bin_sparse cut into runs of at most kBinRun,
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
    sum.y += a.bin_count[k] > a.bin_sparse ? (a.bin_count[k] + kBinRun - 1) / kBinRun : 0;
  }
  int2 run = scan1024(sum, part);
  if (t == 1023) a.runs[0] = make_int4(run.y, 0, 0, 0);
  run.x -= sum.x;
  run.y -= sum.y;
  for (int k = k0; k < k1; ++k) {
    const int32_t c = a.bin_count[k];
    a.bin_cursor[k] = run.x;
    for (int i = 0; i < c && c > a.bin_sparse; i += kBinRun) a.runs[1 + run.y++] = make_int4(k, run.x + i, run.x + min(i + kBinRun, c), 0);
    run.x += c;
  }
}

// Sample indices grouped by bin: each workgroup ranks its samples per bin in
// LDS, reserves a range per bin with one global atomic, then writes. The
// order inside a bin depends on timing (as does the order of the atomics
// that follow it).
__global__ __launch_bounds__(kBinThreads) void bin_scatter_kernel(BackwardArgs a) {
  extern __shared__ int32_t lds[];
  int32_t *local = lds, *base = lds + a.n_bins;
  for (int k = threadIdx.x; k < a.n_bins; k += kBinThreads) local[k] = 0;
  __syncthreads();
  constexpr int kPer = kBinSamplesPerBlock / kBinThreads;
  const int64_t s0 = (int64_t)blockIdx.x * kBinSamplesPerBlock;
  int key[kPer], rank[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int64_t s = s0 + threadIdx.x + kBinThreads * i;
    key[i] = s < a.n ? bin_of(a, a.uv[s]) : -1;
    rank[i] = key[i] >= 0 ? atomicAdd(&local[key[i]], 1) : 0;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < a.n_bins; k += kBinThreads)
    if (local[k]) base[k] = atomicAdd(&a.bin_cursor[k], local[k]);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPer; ++i)
    if (key[i] >= 0) a.perm[base[key[i]] + rank[i]] = (int32_t)(s0 + threadIdx.x + kBinThreads * i);
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
// A level whose windows do not fit (bins of 64 texels and more, levels finer than
// level 0) has no window: its taps are global atomics, four lanes a sample, and
// it does not size the LDS (2^14 samples on 4096^2..512^2 levels: backward 485 -> 234
// us, 112 with its sparse bins added sample by sample).
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

// Adds tap q of sample s on level k straight to the gradients.
__device__ __forceinline__ void tap_direct(const BackwardArgs &a, int64_t s, int k, int q) {
  const LevelArgs &L = a.lat.lv[k];
  const float *g = a.dx + s * a.dx_stride;
  const Cell c = cell_of(L, make_float2(g[a.n_feat], g[a.n_feat + 1]));
  const int i = address_coord(c.ix + (q & 1), L.w, a.lat.address);
  const int j = address_coord(c.iy + (q >> 1), L.h, a.lat.address);
  const float w = ((q & 1) ? c.fx : 1.0f - c.fx) * ((q >> 1) ? c.fy : 1.0f - c.fy);
  float *p = a.grad_lat[k] + ((int64_t)j * L.w + i) * 3;
#pragma unroll
  for (int ch = 0; ch < 3; ++ch) unsafeAtomicAdd(p + ch, w * g[3 * k + ch]);
}

// Samples of sparse bins: 16 lanes each, a level and tap per lane, global
// atomics.
constexpr int kDirectSamples = kAccThreads / 16;
__device__ __forceinline__ void sparse_samples(const BackwardArgs &a, int64_t block) {
  const int64_t s = block * kDirectSamples + (threadIdx.x >> 4);
  const int k = (int)(threadIdx.x >> 2) & 3, q = (int)threadIdx.x & 3;
  if (s >= a.n || k >= a.lat.n_levels) return;
  if (a.n_bins > 0 && a.bin_count[bin_of(a, a.uv[s])] > a.bin_sparse) return;
  tap_direct(a, s, k, q);
}

template <bool SPARSE>
__global__ __launch_bounds__(kAccThreads) void bin_accum_kernel(BackwardArgs a, unsigned run_blocks) {
  constexpr int kT = kAccThreads, kWaves = kT / 64;
  if (SPARSE && blockIdx.x >= run_blocks) {
    sparse_samples(a, blockIdx.x - run_blocks);
    return;
  }
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
  if (!fits) {  // no window: every tap goes straight to the gradients
    for (int i = tid; i < 4 * m; i += kT) tap_direct(a, a.perm[run.y + (i >> 2)], k, i & 3);
    return;
  }
  if (direct) {  // samples outside the window go straight to the gradients
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (cell[i] >= 0 || tid + kT * i >= m) continue;
#pragma unroll 1
      for (int q = 0; q < 4; ++q) tap_direct(a, a.perm[run.y + tid + kT * i], k, q);
    }
  }
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

// No bins: every sample's taps are global atomics.
__global__ __launch_bounds__(kAccThreads) void scatter_direct_kernel(BackwardArgs a) {
  for (int64_t b = blockIdx.x; b * kDirectSamples < a.n; b += gridDim.x) sparse_samples(a, b);
}

// ---------------------------------------------------------------------------
// Forward decode of continuous (float) latents on the FP32 matrix cores: the
// forward half of backward_mfma_kernel (same LDS weight layout, same
// 32-sample steps), ending in the sigmoid and the store. Weights come from
// the packed FP32 image (per layer W [rows_pad][cols_pad], then b).
// ---------------------------------------------------------------------------
constexpr int kFwdWaves = 8;  // wavefronts per workgroup, two per SIMD

template <int MT, int NL>
__global__ __launch_bounds__(64 * kFwdWaves) __attribute__((amdgpu_waves_per_eu(kFwdWaves / 4)))
void forward_mfma_kernel(DecodeArgs a) {
  using M = BwdMap<MT, NL>;
  extern __shared__ float fwd_lds[];
  float *lds = fwd_lds;
  const int tid = threadIdx.x;
  const int lane = tid & 63, h = lane >> 5, c32 = lane & 31, c16 = lane & 15, g16 = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const PackLayout &L = a.lay;
  const int n_out = a.n_out;

  load_weights<MT, NL, 64 * kFwdWaves>(
      lds, tid, a.lat.n_levels,
      [&](int l, int row, int col) {  // padded rows and columns hold zero weights
        return row < L.rows_pad[l] && col < L.cols_pad[l]
                   ? reinterpret_cast<const float *>(a.packed + L.w_off[l])[row * L.cols_pad[l] + col]
                   : 0.0f;
      },
      [&](int l, int row) {
        return row < L.rows_pad[l] ? reinterpret_cast<const float *>(a.packed + L.b_off[l])[row] : 0.0f;
      });
  load_levels(lds + M::oLv, a.lat, tid);
  __syncthreads();

  const int64_t n_chunks = (a.n + kBwdChunk - 1) / kBwdChunk;
  const int64_t stride = (int64_t)gridDim.x * kFwdWaves;
  const int64_t first = first_chunk(n_chunks >= stride, kFwdWaves, wave);
  auto load_uv = [&](int64_t chunk) {
    const int64_t smp = chunk * kBwdChunk + c32;
    return a.uv[smp < a.n ? smp : a.n - 1];
  };
  float2 uv_next = load_uv(first);
  for (int64_t chunk = first; chunk < n_chunks; chunk += stride) {
    const float2 uv = uv_next;
    uv_next = load_uv(chunk + stride < n_chunks ? chunk + stride : chunk);
    const float *wl = lds + opaque_zero((int)chunk);  // as in the backward
    float x[8];
    first_slots(wl + M::oLv, a.lat.address, uv, h, x);
    bf32x16 act[MT], nx[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) act[mt] = first_tile<MT, NL>(wl, mt, c32, h, x);
#pragma unroll
    for (int l = 1; l <= M::NH; ++l) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) nx[mt] = hidden_tile<MT, NL>(wl, l, mt, c32, h, act);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) act[mt] = nx[mt];
    }
    bf32x4 zo[2];
    rows16<MT>([&](int q) { return *reinterpret_cast<const bf32x4 *>(wl + M::oWo + c16 * M::SH + 8 * q + 4 * h); }, act,
               *reinterpret_cast<const bf32x4 *>(wl + M::oBo + 4 * g16), zo[0], zo[1]);
    const OutRows zr = spread_rows(n_out, g16, c16, zo[0], zo[1]);
    auto store = [&](int e) {
      const int64_t smp = chunk * kBwdChunk + zr.smp[e];
      const int row0 = zr.row0;
      float f[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) f[r] = 1.0f / (1.0f + expf(-zr.z[e][r]));
      if (smp >= a.n || row0 >= n_out) return;
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
    };
    store(0);
    if (zr.n > 1) store(1);
  }
}

hipError_t launch_forward_f32(const DecodeArgs &a, const MlpShape &s, hipStream_t st) {
  const int mt = s.hid > 32 ? 2 : 1;
  auto go = [&](auto kernel, size_t floats) {
    hipLaunchKernelGGL(kernel, dim3(backward_groups(a.n)), dim3(64 * kFwdWaves), floats * sizeof(float), st, a);
    return hipGetLastError();
  };
  switch (10 * mt + s.n_layers) {
    case 12: return go(forward_mfma_kernel<1, 2>, BwdMap<1, 2>::oStage);
    case 13: return go(forward_mfma_kernel<1, 3>, BwdMap<1, 3>::oStage);
    case 14: return go(forward_mfma_kernel<1, 4>, BwdMap<1, 4>::oStage);
    case 22: return go(forward_mfma_kernel<2, 2>, BwdMap<2, 2>::oStage);
    case 23: return go(forward_mfma_kernel<2, 3>, BwdMap<2, 3>::oStage);
    case 24: return go(forward_mfma_kernel<2, 4>, BwdMap<2, 4>::oStage);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_backward(const BackwardArgs &a, const MlpShape &s, float *const *grad_W, float *const *grad_b,
                           hipStream_t st) {
  // latent gradients and bin counts start at zero (a kernel: no memset nodes in
  // graphs; one launch: five of 3 to 5 us each took 24 us of a step)
  ZeroArgs z{};
  for (int k = 0; k < a.lat.n_levels; ++k) {
    z.p[k] = a.grad_lat[k];
    z.n[k] = (int64_t)a.lat.lv[k].w * a.lat.lv[k].h * 3;
  }
  z.p[kMaxLevels] = reinterpret_cast<float *>(a.bin_count);
  z.n[kMaxLevels] = a.n_bins;
  if (hipError_t e0 = launch_zero(z, st); e0 != hipSuccess) return e0;
  hipError_t e;
  {
    const int mt = s.hid > 32 ? 2 : 1;
    const int waves = backward_waves(mt, s.n_layers);
    auto go = [&](auto kernel, size_t floats) {
      hipLaunchKernelGGL(kernel, dim3(backward_groups(a.n)), dim3(64 * waves), floats * sizeof(float), st, a);
      return hipGetLastError();
    };
    switch (10 * mt + s.n_layers) {
      case 12: e = go(backward_mfma_kernel<1, 2>, BwdMap<1, 2>::total); break;
      case 13: e = go(backward_mfma_kernel<1, 3>, BwdMap<1, 3>::total); break;
      case 14: e = go(backward_mfma_kernel<1, 4>, BwdMap<1, 4>::total); break;
      case 22: e = go(backward_mfma_kernel<2, 2>, BwdMap<2, 2>::total); break;
      case 23: e = go(backward_mfma_kernel<2, 3>, BwdMap<2, 3>::total); break;
      case 24: e = go(backward_mfma_kernel<2, 4>, BwdMap<2, 4>::total); break;
      default: return hipErrorInvalidValue;
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
  const unsigned sparse = (unsigned)std::min<int64_t>((a.n + kDirectSamples - 1) / kDirectSamples, 1 << 20);
  if (a.n_bins == 0) {
    hipLaunchKernelGGL(scatter_direct_kernel, dim3(sparse), dim3(kAccThreads), 0, st, a);
    return hipGetLastError();
  }
  const unsigned grid = (unsigned)((a.n + kBinSamplesPerBlock - 1) / kBinSamplesPerBlock);
  hipLaunchKernelGGL(bin_count_kernel, dim3(grid), dim3(kBinThreads), a.n_bins * sizeof(int32_t), st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(bin_scan_kernel, dim3(1), dim3(1024), 0, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  hipLaunchKernelGGL(bin_scatter_kernel, dim3(grid), dim3(kBinThreads), 2 * a.n_bins * sizeof(int32_t), st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const unsigned run_blocks = (unsigned)((a.n_runs + 7) / 8 * 8 * a.lat.n_levels);
  const size_t lds = (size_t)(a.bin_lds + 5 * kBinRun + a.bin_cells + 1) * sizeof(float);
  if (a.bin_sparse > 0)
    hipLaunchKernelGGL(bin_accum_kernel<true>, dim3(run_blocks + sparse), dim3(kAccThreads), lds, st, a, run_blocks);
  else
    hipLaunchKernelGGL(bin_accum_kernel<false>, dim3(run_blocks), dim3(kAccThreads), lds, st, a, run_blocks);
  return hipGetLastError();
}

}  // namespace ntc
