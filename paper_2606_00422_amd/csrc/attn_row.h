// Causal attention of one history row by one wave that touches the keys and
// values of positions 0..i only (device code, header-only).
//
// The matrix-core kernels multiply the probabilities of a block of keys, zero
// for those after the query, by all of the block's values: an infinite or NaN
// value of a later position turns 0 * v into NaN for the queries before it.
// Those of fp32 models and of head_dim 32 send the queries whose sums come out
// non-finite here, so that such a position stays behind the causal mask.
// Speed is of no concern: few registers (the row is computed inside kernels
// that have none to spare), the logits twice.
#pragma once

#include "upr_internal.h"

namespace upr {

// Inf or NaN.  (Opaque bits: in a file built without NaN semantics the compiler
// drops the NaN half of a test whose operand it knows to be a float.)
__device__ __forceinline__ bool nonfinite_bits(float x) {
    unsigned u = __float_as_uint(x);
    asm("" : "+v"(u));
    return (u & 0x7f800000u) == 0x7f800000u;
}

// q: the query's D values, K and V: rows of the user's positions from 0.
// Queries are pre-scaled (the softmax uses exp2).  All 64 lanes call it with
// the same arguments; lane e < D gets output e.
template <typename T, int D>
__device__ __forceinline__ float causal_row(const T* q, const T* K, const T* V, int i) {
    const int lane = threadIdx.x & 63;
    auto logit = [&](int t) {
        float s = 0.f;
#pragma unroll 4
        for (int e = 0; e < D; ++e) s = fmaf((float)q[e], (float)K[(int64_t)t * D + e], s);
        return s;
    };
    float m = -INFINITY;
    for (int t = lane; t <= i; t += 64) m = fmaxf(m, logit(t));
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) m = fmaxf(m, __shfl_xor(m, x, 64));
    float l = 0.f, acc = 0.f;
    for (int t0 = 0; t0 <= i; t0 += 64) {
        const int n = i + 1 - t0 < 64 ? i + 1 - t0 : 64;        // keys of this pass
        const float p = lane < n ? __builtin_amdgcn_exp2f(logit(t0 + lane) - m) : 0.f;
        l += p;
        for (int j = 0; j < n; ++j)
            acc = fmaf(__shfl(p, j, 64), (float)V[(int64_t)(t0 + j) * D + lane % D], acc);
    }
#pragma unroll
    for (int x = 32; x >= 1; x >>= 1) l += __shfl_xor(l, x, 64);
    return acc / l;
}

}  // namespace upr
