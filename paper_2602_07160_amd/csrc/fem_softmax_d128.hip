// Causal softmax-prior reads at widths 128 (kernel: fem_softmax_kernel.h).

#include "fem_softmax_kernel.h"

namespace fem {

template <>
hipError_t softmax_causal<128, 128>(FEM_SOFTMAX_ARGS, void* out, bool obf16, float* lse) {
  return obf16 ? launch_kg<128, 128, kFem, true, true>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream, lse)
               : launch_kg<128, 128, kFem, true, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream, lse);
}

}  // namespace fem
