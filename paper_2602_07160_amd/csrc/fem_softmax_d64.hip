// Softmax-prior reads at widths 64 (kernel: fem_softmax_kernel.h).

#include "fem_softmax_kernel.h"

namespace fem {

template <>
hipError_t softmax_causal<64, 64>(FEM_SOFTMAX_ARGS, void* out, bool obf16, float* lse) {
  return obf16 ? launch_kg<64, 64, kFem, true, true>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream, lse)
               : launch_kg<64, 64, kFem, true, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream, lse);
}

template <>
hipError_t softmax_encoder<64, 64>(FEM_SOFTMAX_ARGS, void* out, bool obf16) {
  return obf16 ? launch_kg<64, 64, kFem, false, true>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream)
               : launch_kg<64, 64, kFem, false, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream);
}

// mu into out, then the free-energy pass that mixes it
template <>
hipError_t softmax_gated<64>(FEM_SOFTMAX_ARGS, const float* lam, const float* gate, float* out) {
  const hipError_t e = launch_kg<64, 64, kMean, true, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream);
  if (e != hipSuccess) return e;
  return launch_kg<64, 64, kGated, true, false>(Q, K, V, beta, lam, gate, out, B, H, T, stream);
}

}  // namespace fem
