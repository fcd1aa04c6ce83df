// Shared by the surrogate's kernels: matrix-core vector types, GELU, the
// error text of the C entry points.
#pragma once

#include <hip/hip_runtime.h>

namespace sbp_nn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// GELU, tanh form: gelu(z) = z/2 (1 + tanh(s (z + 0.044715 z^3))), s = sqrt(2/pi)
__device__ __forceinline__ float gelu(float z) {
  const float s = 0.7978845608028654f;
  return 0.5f * z * (1.f + tanhf(s * (z + 0.044715f * z * z * z)));
}
__device__ __forceinline__ float gelu_grad(float z) {
  const float s = 0.7978845608028654f;
  const float u = s * (z + 0.044715f * z * z * z);
  const float t = tanhf(u);
  return 0.5f * (1.f + t) + 0.5f * z * (1.f - t * t) * s * (1.f + 3.f * 0.044715f * z * z);
}

// sets the calling thread's error text, returns SBP_NN_EINVAL
int set_error(const char* msg);
// SBP_NN_OK, or SBP_NN_EHIP with the text of the last HIP error
int status();

}  // namespace sbp_nn
