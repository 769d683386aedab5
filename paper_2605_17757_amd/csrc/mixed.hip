// bf16 tokens of the mixed-precision cache in a launch of their own
// (oscar_decode_attn_mixed; a decode step runs them with its prologue).
#include <algorithm>

#include "seg_partial.h"

namespace oscar {
namespace {

template <int NH>
__global__ __launch_bounds__(512)
__attribute__((amdgpu_waves_per_eu(NH > 8 ? 2 : 4, NH > 8 ? 2 : 4))) void seg_partial_kernel(SegArgs args) {
  __shared__ SegSmem<NH> sm;
  seg_partial_body<NH>(sm, blockIdx.x, blockDim.x >> 6, args);
}

template <int NH>
hipError_t launch_seg_nh(const uint16_t* seg, int Hkv, int S0, int W, int B, int Hq,
                         const int32_t* seq_lens, int max_pages, const uint16_t* q, float qscale,
                         int num_splits, float* part_o, float* part_ml, hipStream_t st) {
  const int nw = std::min(kSegWaves, std::max(1, (S0 + W + kP - 1) / kP));
  return by_seqs(B, launch_seqs(Hq), [&](int b0, int nb) {
    const size_t row = (size_t)b0 * Hq, part = row * (num_splits + 1);
    const SegArgs args{seg ? seg + (size_t)b0 * Hkv * 2 * (S0 + W) * kD : nullptr, nullptr, nullptr, Hkv,
                       S0, W, Hq, seq_lens + b0, max_pages, q + row * kD, qscale, num_splits,
                       part_o + part * kD, part_ml + part * 2};
    hipLaunchKernelGGL(seg_partial_kernel<NH>, dim3((unsigned)(nb * Hkv)), dim3(64 * nw), 0, st, args);
    return hipGetLastError();
  });
}

}  // namespace

hipError_t launch_seg_partial(const uint16_t* seg, int Hkv, int S0, int W, int B, int Hq,
                              const int32_t* seq_lens, int max_pages, const uint16_t* q,
                              float qscale, int num_splits, float* part_o, float* part_ml,
                              hipStream_t st) {
  const int g = Hq / Hkv;
  if (g <= 4)
    return launch_seg_nh<4>(seg, Hkv, S0, W, B, Hq, seq_lens, max_pages, q, qscale, num_splits,
                            part_o, part_ml, st);
  if (g <= 8)
    return launch_seg_nh<8>(seg, Hkv, S0, W, B, Hq, seq_lens, max_pages, q, qscale, num_splits,
                            part_o, part_ml, st);
  return launch_seg_nh<16>(seg, Hkv, S0, W, B, Hq, seq_lens, max_pages, q, qscale, num_splits,
                           part_o, part_ml, st);
}

}  // namespace oscar
