// Encoder softmax-prior reads at widths 128 (kernel: fem_softmax_kernel.h).

#include "fem_softmax_kernel.h"

namespace fem {

template <>
hipError_t softmax_encoder<128, 128>(FEM_SOFTMAX_ARGS, void* out, bool obf16) {
  return obf16 ? launch_kg<128, 128, kFem, false, true>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream)
               : launch_kg<128, 128, kFem, false, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream);
}

}  // namespace fem
