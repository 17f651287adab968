// The batch plan of a classified frame, built on the device.
//
// The pixels of every material are known on the device once the frame is
// classified (mat_offsets). Taking them to the host, packing work items there
// and copying the plan back costs two waits and several copies, more than the
// frame's GPU work; so one kernel writes the plan that decode_batched_kernel
// walks, and the host enqueues classification, plan and decode in one go.
//
// Items: the materials' 64-pixel tiles, ordered by (MLP shape, material), are
// laid on one axis of estimated cost and the axis is cut into a range per
// wave, at tiles. A wave gets few materials, so weights load once per wave and
// material, and the waves differ by a tile, where packing whole items longest
// first leaves them an item apart.
// Measured at 2560 x 1440 with 64 materials: this kernel 11 us, the decode
// 111 us against 116 with the host's plan, the whole frame 815 -> 150 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <vector>

#include "ntc.h"
#include "ntc_internal.hpp"

namespace ntc {

namespace {

constexpr int kPlanThreads = 1024;
constexpr int kCopyMats = 16;  // materials a copying workgroup fills in

// A material in the order of the items: index, shape and cost of a tile, in
// units of two matrix issue slots.
constexpr uint32_t kMaxTileCost = 127;
// Share of sampling, in matrix issue slots, of a tile of listed pixels: one
// material over 2560 x 1440 takes 88 us at 16 x 2 (width x layers), 92 at
// 64 x 2, 101 at 64 x 3, 114 at 64 x 4, which is nearly flat. Frame of 64
// materials at 2560 x 1440, decode: 111 us with 100 to 150, 114 to 122 with
// 200 to 400, 148 with the 12 of the batch, whose waves mix all shapes.
constexpr double kListedSampling = 150.0;
__host__ __device__ inline uint32_t order_word(uint32_t mat, uint32_t shape, uint32_t cost) {
  return mat | (shape << 12) | (cost << 16);
}
__device__ __forceinline__ uint32_t order_mat(uint32_t o) { return o & 0xFFFu; }
__device__ __forceinline__ uint32_t order_shape(uint32_t o) { return (o >> 12) & 15u; }
__device__ __forceinline__ uint32_t order_cost(uint32_t o) { return o >> 16; }

struct FrameArgs {
  FrameTable t;
  const uint8_t *table;
  const int32_t *list;
  const int32_t *mat_offsets;  // [n_mats + 1]
  const float2 *uv;
  void *image;
  int64_t img_px;
  uint8_t *plan;
};

// Exclusive prefix sums of one value a thread over the workgroup.
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t *part, uint32_t &total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = (uint32_t)__shfl_up((int)inc, o);
    if (lane >= o) inc += u;
  }
  if (lane == 63) part[wave] = inc;
  __syncthreads();
  uint32_t before = 0;
  total = 0;
#pragma unroll
  for (int i = 0; i < kPlanThreads / 64; ++i) {
    const uint32_t u = part[i];
    before += i < wave ? u : 0u;
    total += u;
  }
  __syncthreads();
  return before + inc - v;
}

// Workgroup 0: header, work items and the waves' ranges of them. The others:
// the material table, each word copied and the frame's fields filled in.
// LDS: 2 (n_mats + 1) words. Sums of costs fit 32 bits: mat_offsets, being
// int32, count less than 2^31 pixels, so there are at most 2^25 + n_mats tiles,
// of a cost of at most kMaxTileCost each.
static_assert(((1ull << 25) + NTC_MAX_CLASSIFY_MATERIALS) * kMaxTileCost < (1ull << 32), "32-bit sums of costs");
__global__ __launch_bounds__(kPlanThreads) void frame_plan_kernel(FrameArgs f) {
  const int n_mats = f.t.plan.n_mats;
  if (blockIdx.x > 0) {
    const int m0 = (blockIdx.x - 1) * kCopyMats, m1 = min(m0 + kCopyMats, n_mats);
    constexpr int kWords = sizeof(BatchMaterial) / 4;
    const uint32_t *src = reinterpret_cast<const uint32_t *>(f.table + f.t.mats_off) + (int64_t)m0 * kWords;
    BatchMaterial *mats = reinterpret_cast<BatchMaterial *>(f.plan + f.t.plan.mats_off);
    uint32_t *dst = reinterpret_cast<uint32_t *>(mats + m0);
    for (int i = threadIdx.x; i < (m1 - m0) * kWords; i += kPlanThreads) dst[i] = src[i];
    __syncthreads();
    const int m = m0 + threadIdx.x;
    if (m < m1) {
      const int32_t o0 = f.mat_offsets[m], n = f.mat_offsets[m + 1] - o0;
      DecodeArgs &a = mats[m].a;
      a.uv = f.uv;
      a.out = f.image;
      a.n = n;
      a.n_tiles = ((int64_t)n + 63) / 64;
      a.pix = f.list + o0;
      a.img_px = f.img_px;
    }
    return;
  }
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t part[kPlanThreads / 64];
  uint32_t *start = lds;             // start of the s-th material with pixels on the cost axis; [n]: the whole cost
  uint32_t *who = lds + n_mats + 1;  // its word of `order`
  const uint32_t *order = reinterpret_cast<const uint32_t *>(f.table + f.t.order_off);
  // materials with pixels, in order, and where they start
  const int per = (n_mats + kPlanThreads - 1) / kPlanThreads;
  const int k0 = min((int)threadIdx.x * per, n_mats), k1 = min(k0 + per, n_mats);
  auto tiles_of = [&](uint32_t o) {
    const uint32_t m = order_mat(o);
    return (uint32_t)(f.mat_offsets[m + 1] - f.mat_offsets[m] + 63) >> 6;
  };
  uint32_t my_n = 0, my_c = 0;
  for (int k = k0; k < k1; ++k) {
    const uint32_t o = order[k], t = tiles_of(o);
    my_n += t > 0;
    my_c += t * order_cost(o);
  }
  uint32_t n, total;
  uint32_t s = block_prefix(my_n, part, n);
  uint32_t c = block_prefix(my_c, part, total);
  for (int k = k0; k < k1; ++k) {
    const uint32_t o = order[k], t = tiles_of(o);
    if (t > 0) {
      start[s] = c;
      who[s++] = o;
      c += t * order_cost(o);
    }
  }
  if (threadIdx.x == 0) start[n] = total;
  __syncthreads();
  // where the range of wave w begins: (material s, tile t), (n, 0) for the end
  const int n_waves = f.t.plan.n_waves;
  const double step = (double)total / n_waves;
  auto locate = [&](int w, uint32_t &ms, uint32_t &mt) {
    const uint32_t b = (uint32_t)(w * step);
    uint32_t lo = 0, hi = n;  // the last material starting at or before b
    while (lo + 1 < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (start[mid] <= b) lo = mid; else hi = mid;
    }
    const bool end = w >= n_waves || n == 0;
    ms = end ? n : lo;
    mt = end ? 0u : min((b - start[lo]) / order_cost(who[lo]), (start[lo + 1] - start[lo]) / order_cost(who[lo]));
  };
  // emit(wave) before the wave's items, emit(order word, first tile, tiles) for each
  const int wper = (n_waves + kPlanThreads - 1) / kPlanThreads;
  const int w0 = min((int)threadIdx.x * wper, n_waves), w1 = min(w0 + wper, n_waves);
  auto walk = [&](auto begin, auto emit) {
    uint32_t s0, t0, s1, t1;
    locate(w0, s0, t0);
    for (int w = w0; w < w1; ++w) {
      begin(w);
      locate(w + 1, s1, t1);
      for (uint32_t q = s0; q <= s1 && q < n; ++q) {
        const uint32_t a = q == s0 ? t0 : 0u;
        const uint32_t e = q == s1 ? t1 : (start[q + 1] - start[q]) / order_cost(who[q]);
        if (e > a) emit(who[q], a, e - a);
      }
      s0 = s1;
      t0 = t1;
    }
  };
  uint32_t my_items = 0;
  walk([](int) {}, [&](uint32_t, uint32_t, uint32_t) { ++my_items; });
  uint32_t n_items;
  uint32_t it = block_prefix(my_items, part, n_items);
  BatchItem *items = reinterpret_cast<BatchItem *>(f.plan + f.t.plan.items_off);
  int32_t *wstart = reinterpret_cast<int32_t *>(f.plan + f.t.plan.wave_start_off);
  walk([&](int w) { wstart[w] = (int32_t)it; },
       [&](uint32_t o, uint32_t first, uint32_t tiles) {
         BatchItem b;
         b.mat = (int32_t)order_mat(o);
         b.shape_id = (int32_t)order_shape(o);
         b.first_tile = first;
         b.n_tiles = tiles;
         items[it++] = b;
       });
  if (threadIdx.x == 0) {
    wstart[n_waves] = (int32_t)n_items;
    BatchPlanHeader h = f.t.plan;
    h.n_items = (int32_t)n_items;
    *reinterpret_cast<BatchPlanHeader *>(f.plan) = h;
  }
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

size_t frame_table_bytes(int n_mats) {
  return align256(sizeof(FrameTable)) + align256((size_t)n_mats * sizeof(BatchMaterial)) +
         align256((size_t)n_mats * sizeof(uint32_t));
}

void build_frame_table(const BatchMaterial *mats, int n_mats, int n_waves, int stage_cap, uint8_t *out, size_t bytes) {
  memset(out, 0, bytes);
  FrameTable t;
  memset(&t, 0, sizeof t);
  t.mats_off = align256(sizeof(FrameTable));
  t.order_off = t.mats_off + align256((size_t)n_mats * sizeof(BatchMaterial));
  t.total_bytes = frame_table_bytes(n_mats);
  t.n_out = mats[0].a.n_out;
  t.out_f16 = mats[0].a.out_f16;
  // every wave and every material start an item
  const int64_t n_items = (int64_t)n_waves + n_mats;
  BatchPlanHeader &h = t.plan;
  h.magic = kFrameMagic;
  h.version = kPlanVersion;
  h.n_mats = n_mats;
  h.n_waves = n_waves;
  h.stage_cap = stage_cap;
  h.mats_off = align256(sizeof(BatchPlanHeader));
  h.items_off = align256(h.mats_off + (size_t)n_mats * sizeof(BatchMaterial));
  h.wave_start_off = align256(h.items_off + (size_t)n_items * sizeof(BatchItem));
  h.total_bytes = align256(h.wave_start_off + (size_t)(n_waves + 1) * sizeof(int32_t));
  memcpy(out, &t, sizeof t);
  memcpy(out + t.mats_off, mats, (size_t)n_mats * sizeof(BatchMaterial));
  std::vector<int32_t> by_shape(n_mats);
  for (int m = 0; m < n_mats; ++m) by_shape[m] = m;
  std::stable_sort(by_shape.begin(), by_shape.end(),
                   [&](int32_t x, int32_t y) { return mats[x].shape_id < mats[y].shape_id; });
  uint32_t *order = reinterpret_cast<uint32_t *>(out + t.order_off);
  for (int k = 0; k < n_mats; ++k) {
    const BatchMaterial &M = mats[by_shape[k]];
    order[k] = order_word(by_shape[k], M.shape_id,
                          std::min<uint32_t>(kMaxTileCost,
                                             (uint32_t)(0.5 * tile_cost(M.hid, M.n_layers, kListedSampling))));
  }
}

hipError_t launch_frame_plan(FrameTable &t, const uint8_t *table_dev, const int32_t *list,
                             const int32_t *mat_offsets, const float *uv, void *image, int64_t img_px,
                             uint8_t *plan_dev, hipStream_t st) {
  const int n_mats = t.plan.n_mats;
  // no more waves than the frame can have tiles
  t.plan.n_waves = (int)std::min<int64_t>(t.plan.n_waves, img_px / 64 + n_mats);
  FrameArgs f;
  f.t = t;
  f.table = table_dev;
  f.list = list;
  f.mat_offsets = mat_offsets;
  f.uv = reinterpret_cast<const float2 *>(uv);
  f.image = image;
  f.img_px = img_px;
  f.plan = plan_dev;
  hipLaunchKernelGGL(frame_plan_kernel, dim3(1 + (n_mats + kCopyMats - 1) / kCopyMats), dim3(kPlanThreads),
                     2 * (size_t)(n_mats + 1) * sizeof(uint32_t), st, f);
  return hipGetLastError();
}

}  // namespace ntc
