// Fused BC1 + MLP decode on the CDNA4 matrix cores (FP16 or E4M3 operands,
// FP32 accumulation), one persistent wavefront per workgroup.
//
// The paper evaluates the MLP per 8x4 pixel tile on the matrix engines of its
// GPUs through cooperative vectors, with all threads of a workgroup sharing
// one weight matrix (Sec. 4). Here a wavefront keeps the whole MLP in
// registers and walks spans of 256 or 512 pixels; every layer is a product of
// 32x32 tiles (v_mfma_f32_32x32x16_f16, or the 32x32x64 E4M3 form), the
// full-rate matrix instructions of gfx950. The tile-level data flow is
// described in ntc_mfma_tile.hpp.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ntc_device.hpp"
#include "ntc_internal.hpp"
#include "ntc_mfma_tile.hpp"

namespace ntc {

constexpr int kWrapTiles = 2;  // 64-pixel tiles per span with wrap addressing (4: 88 in place of 82 us, see decode_span_wrap)

// One kernel per address mode: the wrapped one is rolled and small, the
// clamped one keeps the registers and the schedule that it has alone (both
// with staging in one kernel: 1 to 3% slower clamped decodes). The mode stays a
// run-time value in the clamped spans of FP32 texels (as a constant: 1% slower)
// and of the 64-wide FP16 networks of four and more layers (as a constant the
// five-layer ones spill 28 registers in place of 17, the four-layer ones 1 in place
// of none; 14-64-64-64-64-8: 2048x1024 pixels 68 -> 65 us, 1501x999 54 -> 52).
template <class P, int HID, int NL, int VEC4, int ADDR>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NTC_WAVES_PER_SIMD, NTC_WAVES_PER_SIMD))) void decode_mfma_kernel(DecodeArgs a) {
  constexpr int kMode = P::kF16Tex && !(HID == 64 && NL >= 4) ? kClampOnly : kEitherMode;
  constexpr int ST = ADDR == kWrapOnly ? kWrapTiles : span_tiles_for(HID, NL, P::kF16Tex);
  constexpr int SPX = 64 * ST;
  extern __shared__ f32x4 smem[];
  f32x4 *stage = smem;
  f32x4 *bias = smem + a.stage_cap;
  f32x4 *ltab = bias + BiasLds<HID, NL>::kCount;
  // output staging for widths that are not a multiple of 4 (32 x 16 floats)
  float *obuf = VEC4 ? nullptr : reinterpret_cast<float *>(ltab + LevelTab::kCount);
  const int lane = threadIdx.x;

  MfmaWeights<P, HID, NL> W;
  W.load(a.packed, a.lay, lane);
  BiasLds<HID, NL>::fill(bias, a.packed, a.lay, lane);
  LevelTab::fill(ltab, a.lat, lane);
  W.ready();
  __syncthreads();

  // XCD-aware numbering: consecutive workgroups land on different XCDs;
  // renumber so that each XCD walks a contiguous range of spans at a time.
  const int nb = gridDim.x;
  int vb = blockIdx.x;
  if ((nb & 7) == 0) vb = (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3);
  const int64_t n_spans = (a.n + SPX - 1) / SPX;
  SpanUv<ST> uvs;
  if (vb < n_spans) {
    uvs.load(a.uv, (int64_t)vb * SPX, a.n);
    // completed before the loop, so that the loop is entered with the same
    // pending loads as its back edge has
    uvs.ready();
  }
  for (int64_t it = vb; it < n_spans; it += nb) {
    const int64_t nx = it + nb;
    const int64_t next = nx < n_spans ? nx * SPX : -1;
    if constexpr (ADDR == kWrapOnly)
      decode_span_wrap<P, HID, NL, ST, VEC4>(a, it * SPX, a.n, stage, bias, ltab, W, uvs, next, a.n, obuf);
    else
      decode_span<P, HID, NL, ST, VEC4, false, kMode>(a, it * SPX, a.n, stage, bias, ltab, W, uvs, next, a.n, obuf);
  }
}

template <class P, int HID, int VEC4>
static hipError_t launch_mfma_v(const DecodeArgs &a, int n_layers, int grid, hipStream_t st) {
  const size_t lds =
      (size_t)(a.stage_cap + BiasLds<HID, 5>::kCount + LevelTab::kCount + (VEC4 ? 0 : 32 * 16 / 4)) * sizeof(f32x4);
  auto go = [&](auto clamped, auto wrapped) {
    if (a.lat.address == 0)
      hipLaunchKernelGGL(clamped, dim3(grid), dim3(64), lds, st, a);
    else
      hipLaunchKernelGGL(wrapped, dim3(grid), dim3(64), lds, st, a);
    return hipGetLastError();
  };
  switch (n_layers) {
    case 2: return go(decode_mfma_kernel<P, HID, 2, VEC4, kClampOnly>, decode_mfma_kernel<P, HID, 2, VEC4, kWrapOnly>);
    case 3: return go(decode_mfma_kernel<P, HID, 3, VEC4, kClampOnly>, decode_mfma_kernel<P, HID, 3, VEC4, kWrapOnly>);
    case 4: return go(decode_mfma_kernel<P, HID, 4, VEC4, kClampOnly>, decode_mfma_kernel<P, HID, 4, VEC4, kWrapOnly>);
    case 5: return go(decode_mfma_kernel<P, HID, 5, VEC4, kClampOnly>, decode_mfma_kernel<P, HID, 5, VEC4, kWrapOnly>);
    default: return hipErrorInvalidValue;
  }
}

template <class P, int HID>
static hipError_t launch_mfma_hid(const DecodeArgs &a, int n_layers, int grid, hipStream_t st) {
  switch (out_class(a.n_out)) {
    case kOut4: return launch_mfma_v<P, HID, kOut4>(a, n_layers, grid, st);
    case kOut4x2: return launch_mfma_v<P, HID, kOut4x2>(a, n_layers, grid, st);
    default: return launch_mfma_v<P, HID, kOutAny>(a, n_layers, grid, st);
  }
}

template <class P>
static hipError_t launch_mfma_prec(const DecodeArgs &a, const MlpShape &s, int grid, hipStream_t st) {
  switch (s.hid) {
    case 16: return launch_mfma_hid<P, 16>(a, s.n_layers, grid, st);
    case 32: return launch_mfma_hid<P, 32>(a, s.n_layers, grid, st);
    case 64: return launch_mfma_hid<P, 64>(a, s.n_layers, grid, st);
    default: return hipErrorInvalidValue;
  }
}

int decode_span_tiles(int hid, int n_layers, int compute) {
  return span_tiles_for(hid, n_layers, compute == 1 ? PrecF16::kF16Tex : (compute == 2 ? PrecBF16::kF16Tex : PrecF8::kF16Tex));
}

hipError_t launch_decode_mfma(const DecodeArgs &a, const MlpShape &s, int compute, int n_cus, int waves_per_cu,
                              hipStream_t st) {
  int64_t grid = (int64_t)n_cus * waves_per_cu;
  const int span = a.lat.address == 0 ? decode_span_tiles(s.hid, s.n_layers, compute) : kWrapTiles;
  // Batches that long spans would fill badly: tiles (64 pixels) one by one, all
  // of them or after a long span per wave. A pass is that of the waves that run at
  // once, however many are to be launched (1024x1024 pixels of 14-32-32-8, 32 per
  // compute unit: long spans 16 us, one tile 27). The lines are where the two meet
  // for pixels in 8x8 tiles or rows of whole spans, which long spans favour (for odd
  // rows and random order they lie further up); the less matrix work a tile has, the
  // more of its time is what a long span shares. Measured (us, long spans / tiles /
  // one long span, then tiles; pixels in 8x8 tiles, then in odd rows), tiles a wave:
  //   spans of 8, FP16: 14-16-8      3: 14/14 21/14; 4: 13/15 21/16;
  //                     14-32-32-8   1/2: 20/8 20/8; 3.5: 13/13 21/13; 4: 13/14 21/15;
  //       8.25: 22/24/16 40/28/28; 9: 25/26/17 56/29/30; 10: 25/28/20 56/33/32;
  //       12: 25/33/25 56/37/37; 14: 25/38/30 57/42/48;
  //                     14-64-64-8   4: 16/16 24/17; 9: 33/30/23 64/33/33;
  //   spans of 4, FP16: 14-64-64-64-8  1/2: 15/9 15/8; 2: 13/12 16/13; 3: 15/15
  //       20/16; 5: 25/21 33/22; 6: 24/24 33/26; 7: 25/27 33/30;
  //               BF16: 14-64-8      5: 19/19 27/20; 6: 19/22 27/23;
  //               E4M3: 14-64-64-8   2: 12/12 15/13; 5: 23/20 30/21; 6: 22/23 30/24.
  // BF16 and E4M3 meet at the same lines, within half a tile.
  if (a.lat.address == 0) {
    const int64_t waves = std::min(grid, (int64_t)n_cus * 4 * NTC_WAVES_PER_SIMD);
    const int64_t pass = span * waves, rest = a.n_tiles % pass;
    // sixteenths of a pass; a wave alone on its SIMD gains by tiles up to half of one
    // (512x512 pixels, 4 waves per compute unit, BF16 14-32-32-8: 19 / 13)
    const int line = waves < (int64_t)n_cus * 4 * NTC_WAVES_PER_SIMD ? 8 : (s.n_layers == 2 ? 6 : (s.hid < 64 ? 7 : 8));
    const bool head = span == NTC_SPAN_TILES_SMALL && a.n_tiles > pass;
    if (a.n_tiles < 2 * pass && rest > 0 && (head ? 2 * rest <= pass : 16 * rest <= line * pass))
      return launch_decode_short(a, s, compute, (int)std::min(a.n_tiles, waves), head, st);
  }
  const int64_t n_iter = (a.n_tiles + span - 1) / span;
  // a multiple of 8 for the XCD numbering: rounded up where the spans are
  // fewer than the waves (down, the spans left over would take a second pass)
  if (grid > n_iter) grid = n_iter < 8 ? n_iter : (n_iter + 7) & ~(int64_t)7;
  else if (grid >= 8) grid &= ~(int64_t)7;
  if (grid < 1) grid = 1;
  if (compute == 1) return launch_mfma_prec<PrecF16>(a, s, (int)grid, st);
  if (compute == 2) return launch_mfma_prec<PrecBF16>(a, s, (int)grid, st);
  if (compute == 3) return launch_mfma_prec<PrecF8>(a, s, (int)grid, st);
  return hipErrorInvalidValue;
}

}  // namespace ntc
