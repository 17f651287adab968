// Short batches of the matrix-core decode: the same walk as ntc_mfma.hip with
// spans of one 64-pixel tile, for the networks with spans of 8 tiles after one
// long span per wavefront where a batch fills them once and a little more.
//
// A batch of fewer spans of 256 or 512 pixels than the card has wavefronts to
// run leaves SIMDs idle, and its time is that of one wavefront working through
// one span, tile after tile (300 to 65536 pixels, FP16 14-64-64-64-8: 14.5 -> 8
// us in a stream of launches; 14-32-32-8 19 -> 7.5).
#include <hip/hip_runtime.h>

#include "ntc_device.hpp"
#include "ntc_internal.hpp"
#include "ntc_mfma_tile.hpp"

namespace ntc {

// A kernel of their own for batches with a long span first: in one kernel the
// others pay for it (14-32-32-32-9, 2177x139 pixels 20.8 -> 21.3 us).
template <class P, int HID, int NL, int VEC4, bool HEAD>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(NTC_WAVES_PER_SIMD, NTC_WAVES_PER_SIMD))) void decode_short_kernel(DecodeArgs a) {
  constexpr int ST = span_tiles_for(HID, NL, P::kF16Tex);
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

  // HEAD: the first ST tiles of every wavefront are one span, of neighbours on an
  // XCD as in ntc_mfma.hip, or tiles too where the span cannot be staged (9 tiles a
  // wave of odd rows, 14-32-32-8: 30 us, 34 with direct fetches)
  const int nb = gridDim.x;
  int64_t head_it = 0, head_end = 0, it = blockIdx.x;
  if constexpr (HEAD) {
    const int vb = (nb & 7) == 0 ? (blockIdx.x & 7) * (nb >> 3) + (blockIdx.x >> 3) : blockIdx.x;
    SpanUv<ST> uvs;
    uvs.load(a.uv, (int64_t)vb * (64 * ST), a.n);
    uvs.ready();
    if (!decode_span<P, HID, NL, ST, VEC4, false, P::kF16Tex ? kClampOnly : kEitherMode, true>(
            a, (int64_t)vb * (64 * ST), a.n, stage, bias, ltab, W, uvs, -1, a.n, obuf)) {
      head_it = (int64_t)vb * ST;
      head_end = head_it + ST;
    }
    it += (int64_t)ST * nb;
  }
#pragma unroll 1
  for (int part = HEAD ? 0 : 1; part < 2; ++part) {
    const int64_t end = part ? a.n_tiles : head_end, step = part ? nb : 1;
    int64_t t = part ? it : head_it;
    if (t >= end) continue;
    SpanUv<1> uvs;
    uvs.load(a.uv, t * 64, a.n);
    uvs.ready();
    for (; t < end; t += step) {
      const int64_t nx = t + step;
      decode_span<P, HID, NL, 1, VEC4, false, kClampOnly>(a, t * 64, a.n, stage, bias, ltab, W, uvs,
                                                          nx < end ? nx * 64 : -1, a.n, obuf);
    }
  }
}

template <class P, int HID, int NL, int VEC4>
static void launch_short_nl(const DecodeArgs &a, int grid, bool head, hipStream_t st) {
  const size_t lds =
      (size_t)(a.stage_cap + BiasLds<HID, 5>::kCount + LevelTab::kCount + (VEC4 ? 0 : 32 * 16 / 4)) * sizeof(f32x4);
  if constexpr (span_tiles_for(HID, NL, P::kF16Tex) == NTC_SPAN_TILES_SMALL)
    if (head) {
      hipLaunchKernelGGL((decode_short_kernel<P, HID, NL, VEC4, true>), dim3(grid), dim3(64), lds, st, a);
      return;
    }
  hipLaunchKernelGGL((decode_short_kernel<P, HID, NL, VEC4, false>), dim3(grid), dim3(64), lds, st, a);
}

template <class P, int HID, int VEC4>
static hipError_t launch_short_v(const DecodeArgs &a, int n_layers, int grid, bool head, hipStream_t st) {
  switch (n_layers) {
    case 2: launch_short_nl<P, HID, 2, VEC4>(a, grid, head, st); break;
    case 3: launch_short_nl<P, HID, 3, VEC4>(a, grid, head, st); break;
    case 4: launch_short_nl<P, HID, 4, VEC4>(a, grid, head, st); break;
    case 5: launch_short_nl<P, HID, 5, VEC4>(a, grid, head, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <class P, int HID>
static hipError_t launch_short_hid(const DecodeArgs &a, int n_layers, int grid, bool head, hipStream_t st) {
  switch (out_class(a.n_out)) {
    case kOut4: return launch_short_v<P, HID, kOut4>(a, n_layers, grid, head, st);
    case kOut4x2: return launch_short_v<P, HID, kOut4x2>(a, n_layers, grid, head, st);
    default: return launch_short_v<P, HID, kOutAny>(a, n_layers, grid, head, st);
  }
}

template <class P>
static hipError_t launch_short_prec(const DecodeArgs &a, const MlpShape &s, int grid, bool head, hipStream_t st) {
  switch (s.hid) {
    case 16: return launch_short_hid<P, 16>(a, s.n_layers, grid, head, st);
    case 32: return launch_short_hid<P, 32>(a, s.n_layers, grid, head, st);
    case 64: return launch_short_hid<P, 64>(a, s.n_layers, grid, head, st);
    default: return hipErrorInvalidValue;
  }
}

// Clamp addressing; 1 <= grid <= a.n_tiles. head: a span of 8 tiles per wavefront
// first (networks with such spans, grid * 8 <= a.n_tiles).
hipError_t launch_decode_short(const DecodeArgs &a, const MlpShape &s, int compute, int grid, bool head,
                               hipStream_t st) {
  if (compute == 1) return launch_short_prec<PrecF16>(a, s, grid, head, st);
  if (compute == 2) return launch_short_prec<PrecBF16>(a, s, grid, head, st);
  if (compute == 3) return launch_short_prec<PrecF8>(a, s, grid, head, st);
  return hipErrorInvalidValue;
}

}  // namespace ntc
