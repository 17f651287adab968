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
  // Spans of one tile where long ones would leave more than half of the first
  // or of the second pass of the waves empty. Measured (us, one tile / spans
  // of 4 or 8; FP16, pixels in rows of whole spans, and in odd rows, whose
  // wrapped spans seldom fit the staging region); tiles a wave:
  //   14-64-64-64-8, spans of 4: 1/2 8 / 13 to 15, 2 12 / 13, 2 1/2 14 / 13
  //   and 15 to 22, 4 18 / 14 and 20 to 23, 5 24 / 28 and 29 / 34, 6 26 / 26
  //   and 27 / 40, 7 29 / 27 and 29 / 38, 10 38 / 37;
  //   14-32-32-8, spans of 8: 1/2 7 / 19, 2 10 / 21, 3 15 / 21, 5 16 / 16 and
  //   22 / 31, 6 19 / 16 and 21 / 31, 8 24 / 16, 9 26 / 27 and 29 / 56,
  //   10 29 / 42, 11.4 35 / 42 (odd).
  if (a.lat.address == 0) {
    // a pass is that of the waves that run at once, however many are to be
    // launched (1024x1024 pixels of 14-32-32-8, 32 per compute unit: long spans 16 us,
    // one tile 27)
    const int64_t waves = std::min(grid, (int64_t)n_cus * 4 * NTC_WAVES_PER_SIMD);
    const int64_t pass = span * waves, rest = a.n_tiles % pass;
    if (a.n_tiles < 2 * pass && rest > 0 && 2 * rest <= pass)
      return launch_decode_short(a, s, compute, (int)std::min(a.n_tiles, waves), st);
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
