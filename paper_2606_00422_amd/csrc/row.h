// One row of d features (d a multiple of 64, at most 1024) in the registers of
// one 64-lane wave: statistics, the MXFP8 LayerNorm and the score head, shared
// by the row kernels and the MXFP8 layer tail (same bits in both).  Device
// code, header-only.
#pragma once

#include "mx.h"
#include "upr_internal.h"

namespace upr {

namespace row_detail {

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

template <int N>
__device__ __forceinline__ void wave_sum(float (&v)[N]) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
        for (int k = 0; k < N; ++k) v[k] += __shfl_xor(v[k], m, 64);
}

constexpr int kMaxPerLane = 16;      // d <= 1024

// Per-lane feature index of register slot i.
template <bool VEC>
__device__ __forceinline__ int feat(int lane, int i) {
    return VEC ? (i >> 2) * 256 + 4 * lane + (i & 3) : lane + 64 * i;
}

template <bool VEC>
__device__ __forceinline__ void load_row(const float* __restrict__ x, int d, int lane,
                                         float (&v)[kMaxPerLane]) {
    const int per = d >> 6;
    if (VEC) {
#pragma unroll
        for (int j = 0; j < kMaxPerLane / 4; ++j)
            if (4 * j < per) {
                const float4 q = *reinterpret_cast<const float4*>(x + j * 256 + 4 * lane);
                v[4 * j] = q.x; v[4 * j + 1] = q.y; v[4 * j + 2] = q.z; v[4 * j + 3] = q.w;
            }
    } else {
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) v[i] = x[lane + 64 * i];
    }
}

// (mean, 1/sqrt(var + eps)) of the N rows held in v, their sums side by side.
template <int N>
__device__ __forceinline__ void row_stats(const float (&v)[N][kMaxPerLane], int d, float eps, float (&mu)[N],
                                          float (&rstd)[N]) {
    const int per = d >> 6;
    float s[N];
#pragma unroll
    for (int k = 0; k < N; ++k) {
        s[k] = 0.f;
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) s[k] += v[k][i];
    }
    wave_sum(s);
#pragma unroll
    for (int k = 0; k < N; ++k) {
        mu[k] = s[k] / (float)d;
        s[k] = 0.f;
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) { const float t = v[k][i] - mu[k]; s[k] = fmaf(t, t, s[k]); }
    }
    wave_sum(s);
#pragma unroll
    for (int k = 0; k < N; ++k) rstd[k] = 1.0f / sqrtf(s[k] / (float)d + eps);
}
__device__ __forceinline__ void row_stats(const float (&v)[kMaxPerLane], int d, float eps, float& mu, float& rstd) {
    float m[1], r[1];
    row_stats(reinterpret_cast<const float (&)[1][kMaxPerLane]>(v), d, eps, m, r);
    mu = m[0];
    rstd = r[0];
}

// Writes LN(v) for the row as MXFP8 (fp8 projection inputs): the VEC layout
// gives a lane four consecutive features per 256-feature group, so one
// 32-feature block is eight consecutive lanes; codes[c] is feature c's E4M3
// code, scales[c / 32] its block's E8M0 byte.
__device__ __forceinline__ void store_normed_mx(uint8_t* __restrict__ codes,
                                                uint8_t* __restrict__ scales,
                                                const float (&v)[kMaxPerLane], int d, int lane,
                                                float mu, float rstd,
                                                const float* __restrict__ gain,
                                                const float* __restrict__ shift, bool store = true) {
    const int per = d >> 6;
#pragma unroll
    for (int j = 0; j < kMaxPerLane / 4; ++j)
        if (4 * j < per) {
            const int c = j * 256 + 4 * lane;
            const float4 gq = *reinterpret_cast<const float4*>(gain + c);
            const float4 bq = *reinterpret_cast<const float4*>(shift + c);
            const float y0 = keep_f32(fmaf((v[4 * j] - mu) * rstd, gq.x, bq.x));
            const float y1 = keep_f32(fmaf((v[4 * j + 1] - mu) * rstd, gq.y, bq.y));
            const float y2 = keep_f32(fmaf((v[4 * j + 2] - mu) * rstd, gq.z, bq.z));
            const float y3 = keep_f32(fmaf((v[4 * j + 3] - mu) * rstd, gq.w, bq.w));
            float amax = fmaxf(fmaxf(fabsf(y0), fabsf(y1)), fmaxf(fabsf(y2), fabsf(y3)));
            amax = fmaxf(amax, __shfl_xor(amax, 1, 64));
            amax = fmaxf(amax, __shfl_xor(amax, 2, 64));
            amax = fmaxf(amax, __shfl_xor(amax, 4, 64));
            const int e = mx_block_exp(amax);
            const float inv = mx_inv_scale(e);
            const uint32_t q = mx_pack4(y0 * inv, y1 * inv, y2 * inv, y3 * inv);
            if (!store) continue;
            *reinterpret_cast<uint32_t*>(codes + c) = q;
            if ((lane & 7) == 0) scales[c >> 5] = (uint8_t)(e + 127);
        }
}

// LN(v) . w for the row, in every lane.
template <bool VEC>
__device__ __forceinline__ float score_row(const float (&v)[kMaxPerLane], int d, int lane, float mu, float rstd,
                                           const float* __restrict__ gain, const float* __restrict__ shift,
                                           const float* __restrict__ w) {
    const int per = d >> 6;
    float acc = 0.f;
    if (VEC) {
#pragma unroll
        for (int j = 0; j < kMaxPerLane / 4; ++j)
            if (4 * j < per) {
                const int c = j * 256 + 4 * lane;
                const float4 gq = *reinterpret_cast<const float4*>(gain + c);
                const float4 bq = *reinterpret_cast<const float4*>(shift + c);
                const float4 wq = *reinterpret_cast<const float4*>(w + c);
                acc = fmaf(fmaf((v[4 * j] - mu) * rstd, gq.x, bq.x), wq.x, acc);
                acc = fmaf(fmaf((v[4 * j + 1] - mu) * rstd, gq.y, bq.y), wq.y, acc);
                acc = fmaf(fmaf((v[4 * j + 2] - mu) * rstd, gq.z, bq.z), wq.z, acc);
                acc = fmaf(fmaf((v[4 * j + 3] - mu) * rstd, gq.w, bq.w), wq.w, acc);
            }
    } else {
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) {
                const int c = lane + 64 * i;
                acc = fmaf(fmaf((v[i] - mu) * rstd, gain[c], shift[c]), w[c], acc);
            }
    }
    return wave_sum(acc);
}

}  // namespace row_detail

}  // namespace upr
