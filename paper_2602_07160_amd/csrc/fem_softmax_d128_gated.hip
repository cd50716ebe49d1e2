// Two-level gated read at width 128 (kernel: fem_softmax_kernel.h).

#include "fem_softmax_kernel.h"

namespace fem {

// mu into out, then the free-energy pass that mixes it
template <>
hipError_t softmax_gated<128>(FEM_SOFTMAX_ARGS, const float* lam, const float* gate, float* out) {
  const hipError_t e = launch_kg<128, 128, kMean, true, false>(Q, K, V, beta, nullptr, nullptr, out, B, H, T, stream);
  if (e != hipSuccess) return e;
  return launch_kg<128, 128, kGated, true, false>(Q, K, V, beta, lam, gate, out, B, H, T, stream);
}

}  // namespace fem
