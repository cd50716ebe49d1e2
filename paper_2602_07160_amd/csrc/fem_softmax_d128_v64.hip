// Softmax-prior reads at d_qk = 128, d_v = 64 (kernel: fem_softmax_kernel.h).

#include "fem_softmax_kernel.h"

namespace fem {

template <>
hipError_t softmax_causal<128, 64>(FEM_SOFTMAX_ARGS, void* out, bool obf16, float* lse) {
  return obf16 ? launch_kg<128, 64, kFem, true, true>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream, lse)
               : launch_kg<128, 64, kFem, true, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream, lse);
}

template <>
hipError_t softmax_encoder<128, 64>(FEM_SOFTMAX_ARGS, void* out, bool obf16) {
  return obf16 ? launch_kg<128, 64, kFem, false, true>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream)
               : launch_kg<128, 64, kFem, false, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream);
}

}  // namespace fem
