// Middle of the gated FFN, one element: used by the GEMM epilogue that fuses it and by the separate kernel.
#pragma once
#include <hip/hip_runtime.h>

namespace kvpr {

__device__ __forceinline__ float silu_mul(float gate, float up) { return gate / (1.0f + __expf(-gate)) * up; }

}  // namespace kvpr
