// Dispatch of the bf16 softmax-prior reads on their widths (the kernel is in
// fem_softmax_kernel.h, its instantiations in fem_softmax_d*.hip).

#include "fem_internal.h"

namespace fem {

hipError_t launch_softmax_bf16(const void* Q, const void* K, const void* V, const float* beta,
                               float* out, int B, int H, int T, int d, hipStream_t stream) {
  return launch_softmax_ex_bf16(Q, K, V, beta, out, B, H, T, d, d, true, false, stream);
}

hipError_t launch_softmax_ex_bf16(const void* Q, const void* K, const void* V, const float* beta,
                                  void* out, int B, int H, int T, int dk, int dv, bool causal,
                                  bool obf16, hipStream_t stream) {
#define FEM_PAIR(DK, DV)                                                                     \
  if (dk == DK && dv == DV)                                                                  \
    return causal ? softmax_causal<DK, DV>(Q, K, V, beta, B, H, T, stream, out, obf16, nullptr) \
                  : softmax_encoder<DK, DV>(Q, K, V, beta, B, H, T, stream, out, obf16);
  FEM_PAIR(32, 32)
  FEM_PAIR(64, 64)
  FEM_PAIR(128, 128)
  FEM_PAIR(64, 32)
  FEM_PAIR(128, 64)
#undef FEM_PAIR
  return hipErrorInvalidValue;
}

hipError_t launch_softmax_train_bf16(const void* Q, const void* K, const void* V,
                                     const float* beta, float* out, float* lse, int B, int H,
                                     int T, int d, hipStream_t stream) {
  switch (d) {
    case 32: return softmax_causal<32, 32>(Q, K, V, beta, B, H, T, stream, out, false, lse);
    case 64: return softmax_causal<64, 64>(Q, K, V, beta, B, H, T, stream, out, false, lse);
    case 128: return softmax_causal<128, 128>(Q, K, V, beta, B, H, T, stream, out, false, lse);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_softmax_gated_bf16(const void* Q, const void* K, const void* V,
                                     const float* beta_max, const float* lam, const float* gate,
                                     float* out, int B, int H, int T, int d, hipStream_t stream) {
  switch (d) {
    case 32: return softmax_gated<32>(Q, K, V, beta_max, B, H, T, stream, lam, gate, out);
    case 64: return softmax_gated<64>(Q, K, V, beta_max, B, H, T, stream, lam, gate, out);
    case 128: return softmax_gated<128>(Q, K, V, beta_max, B, H, T, stream, lam, gate, out);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fem
