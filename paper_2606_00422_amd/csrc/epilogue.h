// GELU of fp32 models (device code, header-only).
#pragma once

#include "upr_internal.h"

namespace upr {

__device__ __forceinline__ float gelu_tanh_f(float x) {
    // 0.5 x (1 + tanh(sqrt(2/pi) (x + 0.044715 x^3)))
    const float k0 = 0.7978845608028654f;
    const float y = k0 * (x + 0.044715f * x * x * x);
    return 0.5f * x * (1.0f + tanhf(y));
}

}  // namespace upr
