// Row-wise kernels: residual-stream initialisation, LayerNorm, score head.
//
// One 64-lane wave owns one row of d features (d a multiple of 64, at most
// 1024).  For d a multiple of 256 a lane holds float4 groups j*256 + 4*lane
// (16-byte loads, 8-byte half stores); otherwise features lane + 64 i.
// Statistics are two-pass in fp32 over the registers: mean, then the mean
// of squared deviations (population variance), as LayerNorm defines them.
#include "row.h"
#include "worklist.h"

namespace upr {

namespace {

using namespace row_detail;

template <typename T> __device__ __forceinline__ float to_f(T v) { return (float)v; }

// Four consecutive token values (8 bytes for bf16, 16 for fp32) as floats.
template <typename T>
__device__ __forceinline__ void load4(const T* __restrict__ p, float* v) {
    typedef __attribute__((ext_vector_type(4))) T t4;
    const t4 x = *reinterpret_cast<const t4*>(p);
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = (float)x[t];
}

constexpr int kRowsPerBlock = 4;     // 4 waves, one row each

// Writes LN(v) (gain/shift) for the row to out (model operand type TA).
template <bool VEC, typename TA>
__device__ __forceinline__ void store_normed(TA* __restrict__ out, const float (&v)[kMaxPerLane],
                                             int d, int lane, float mu, float rstd,
                                             const float* __restrict__ gain,
                                             const float* __restrict__ shift) {
    const int per = d >> 6;
    if constexpr (VEC && sizeof(TA) == 2) {
        typedef __attribute__((ext_vector_type(4))) TA t4;
#pragma unroll
        for (int j = 0; j < kMaxPerLane / 4; ++j)
            if (4 * j < per) {
                const int c = j * 256 + 4 * lane;
                const float4 gq = *reinterpret_cast<const float4*>(gain + c);
                const float4 bq = *reinterpret_cast<const float4*>(shift + c);
                t4 o;
                o[0] = (TA)keep_f32(fmaf((v[4 * j] - mu) * rstd, gq.x, bq.x));
                o[1] = (TA)keep_f32(fmaf((v[4 * j + 1] - mu) * rstd, gq.y, bq.y));
                o[2] = (TA)keep_f32(fmaf((v[4 * j + 2] - mu) * rstd, gq.z, bq.z));
                o[3] = (TA)keep_f32(fmaf((v[4 * j + 3] - mu) * rstd, gq.w, bq.w));
                *reinterpret_cast<t4*>(out + c) = o;
            }
    } else {
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) {
                const int c = feat<VEC>(lane, i);
                out[c] = (TA)keep_f32(fmaf((v[i] - mu) * rstd, gain[c], shift[c]));
            }
    }
}

// g = float(x); a = LN(g)  (residual stream initialisation fused with the
// first layer's LayerNorm).  g may be null: the first residual update then
// reads x itself.
//
// LIST: block 0 builds the attention's work list meanwhile: the launch that
// used to do only that took 4.7 us of every call.
template <bool VEC, bool LIST, typename TKV, typename TA>
__global__ __launch_bounds__(256) void k_init_layernorm(const TKV* __restrict__ x,
                                                        float* __restrict__ g, TA* __restrict__ a,
                                                        int64_t rows, int d,
                                                        const float* __restrict__ gain,
                                                        const float* __restrict__ shift, float eps,
                                                        WorkList wl) {
    if constexpr (LIST) {
        if (blockIdx.x == 0) {
            build_worklist<256, kListMaxUsers>(wl);
            return;
        }
    }
    const int64_t row = (int64_t)(blockIdx.x - LIST) * kRowsPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    const int per = d >> 6;
    float v[kMaxPerLane];
    const TKV* xr = x + row * d;
    float* gr = g + row * d;
    if (VEC) {
#pragma unroll
        for (int j = 0; j < kMaxPerLane / 4; ++j)
            if (4 * j < per) load4(xr + j * 256 + 4 * lane, v + 4 * j);
    } else {
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) v[i] = to_f(xr[lane + 64 * i]);
    }
    if (g == nullptr) {
    } else if (VEC) {
#pragma unroll
        for (int j = 0; j < kMaxPerLane / 4; ++j)
            if (4 * j < per)
                *reinterpret_cast<float4*>(gr + j * 256 + 4 * lane) =
                    make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < kMaxPerLane; ++i)
            if (i < per) gr[lane + 64 * i] = v[i];
    }
    float mu, rstd;
    row_stats(v, d, eps, mu, rstd);
    store_normed<VEC>(a + row * d, v, d, lane, mu, rstd, gain, shift);
}

template <bool VEC, typename TA>
__global__ __launch_bounds__(256) void k_layernorm(const float* __restrict__ g, TA* __restrict__ a,
                                                   int64_t rows, int d,
                                                   const float* __restrict__ gain,
                                                   const float* __restrict__ shift, float eps) {
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    float v[kMaxPerLane], mu, rstd;
    load_row<VEC>(g + row * d, d, lane, v);
    row_stats(v, d, eps, mu, rstd);
    store_normed<VEC>(a + row * d, v, d, lane, mu, rstd, gain, shift);
}

// MXFP8 LayerNorm outputs (d a multiple of 256).  INIT: the residual stream
// starts here, g = float(x).
template <bool INIT, typename TKV>
__global__ __launch_bounds__(256) void k_layernorm_mx(const TKV* __restrict__ x,
                                                      float* __restrict__ g,
                                                      uint8_t* __restrict__ codes,
                                                      uint8_t* __restrict__ scales, int64_t rows,
                                                      int d, const float* __restrict__ gain,
                                                      const float* __restrict__ shift, float eps) {
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    const int per = d >> 6;
    float v[kMaxPerLane], mu, rstd;
    if constexpr (INIT) {
        const TKV* xr = x + row * d;
        float* gr = g + row * d;
#pragma unroll
        for (int j = 0; j < kMaxPerLane / 4; ++j)
            if (4 * j < per) {
                const int c = j * 256 + 4 * lane;
                load4(xr + c, v + 4 * j);
                if (g != nullptr)      // null: the first residual update reads x
                    *reinterpret_cast<float4*>(gr + c) =
                        make_float4(v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]);
            }
    } else {
        load_row<true>(g + row * d, d, lane, v);
    }
    row_stats(v, d, eps, mu, rstd);
    store_normed_mx(codes + row * d, scales + row * (d / kMxBlock), v, d, lane, mu, rstd, gain,
                    shift);
}

template <bool VEC>
__global__ __launch_bounds__(256) void k_score_head(const float* __restrict__ g,
                                                    float* __restrict__ scores, int64_t rows, int d,
                                                    const float* __restrict__ gain,
                                                    const float* __restrict__ shift,
                                                    const float* __restrict__ w,
                                                    const float* __restrict__ b, float eps) {
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    float v[kMaxPerLane], mu, rstd;
    load_row<VEC>(g + row * d, d, lane, v);
    row_stats(v, d, eps, mu, rstd);
    const float acc = score_row<VEC>(v, d, lane, mu, rstd, gain, shift, w);
    if (lane == 0) scores[row] = acc + b[0];
}

// LayerNorm (fp16 output) or, with `scores`, the score head of fp32 rows of at
// most 512 values in the association tree of the GEMMs' whole-row epilogue
// (EPI_RESID_LN, EPI_RESID_SCORE), so that a residual update on small tiles
// followed by this kernel gives the bits of that epilogue: statistics per
// 64-column block over 16 lanes of four columns (exchanges 8, 4, 2, 1 apart),
// then the blocks in order (Chan et al.'s pairwise update).
template <bool SCORE>
__global__ __launch_bounds__(256) void k_block_layernorm(const float* __restrict__ g, f16* __restrict__ a,
                                                         int64_t rows, int d, const float* __restrict__ gain,
                                                         const float* __restrict__ shift, float eps,
                                                         const float* __restrict__ w,
                                                         const float* __restrict__ b,
                                                         float* __restrict__ scores) {
    const int64_t row = (int64_t)blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (row >= rows) return;
    auto row16_sum = [](float t) {
        t += __shfl_xor(t, 8, 64);
        t += __shfl_xor(t, 4, 64);
        t += __shfl_xor(t, 2, 64);
        return t + __shfl_xor(t, 1, 64);
    };
    // lane l holds columns 256j + 4l .. +3, of block 4j + l / 16
    float4 h[2], gq[2], bq[2], wq[2];
    bool on[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = 256 * j + 4 * lane;
        on[j] = c < d;
        h[j] = gq[j] = bq[j] = wq[j] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on[j]) {
            h[j] = *reinterpret_cast<const float4*>(g + row * d + c);
            gq[j] = *reinterpret_cast<const float4*>(gain + c);
            bq[j] = *reinterpret_cast<const float4*>(shift + c);
            if constexpr (SCORE) wq[j] = *reinterpret_cast<const float4*>(w + c);
        }
    }
    float mean[2], m2[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        mean[j] = row16_sum((h[j].x + h[j].y) + (h[j].z + h[j].w)) / 64.0f;
        const float u0 = h[j].x - mean[j], u1 = h[j].y - mean[j], u2 = h[j].z - mean[j], u3 = h[j].w - mean[j];
        m2[j] = row16_sum(fmaf(u0, u0, fmaf(u1, u1, fmaf(u2, u2, u3 * u3))));
    }
    const int blocks = d >> 6;
    float mean_w[8], m2_w[8], tot = 0.f, sum = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        mean_w[k] = __shfl(mean[k >> 2], 16 * (k & 3), 64);
        m2_w[k] = __shfl(m2[k >> 2], 16 * (k & 3), 64);
        if (k < blocks) {
            tot += 64.0f;
            sum = fmaf(64.0f, mean_w[k], sum);
        }
    }
    const float mu = sum / tot;
    float M2 = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (k < blocks) {
            const float dm = mean_w[k] - mu;
            M2 += fmaf(64.0f * dm, dm, m2_w[k]);
        }
    const float rstd = 1.0f / sqrtf(M2 / tot + eps);
    if constexpr (SCORE) {
        float part[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            float d4 = 0.f;
            if (on[j]) {
                d4 = fmaf(fmaf((h[j].x - mu) * rstd, gq[j].x, bq[j].x), wq[j].x, d4);
                d4 = fmaf(fmaf((h[j].y - mu) * rstd, gq[j].y, bq[j].y), wq[j].y, d4);
                d4 = fmaf(fmaf((h[j].z - mu) * rstd, gq[j].z, bq[j].z), wq[j].z, d4);
                d4 = fmaf(fmaf((h[j].w - mu) * rstd, gq[j].w, bq[j].w), wq[j].w, d4);
            }
            part[j] = row16_sum(d4);
        }
        float sc = __shfl(part[0], 0, 64);
#pragma unroll
        for (int k = 1; k < 8; ++k) sc += __shfl(part[k >> 2], 16 * (k & 3), 64);
        if (lane == 0) scores[row] = sc + b[0];
    } else {
        typedef __attribute__((ext_vector_type(4))) _Float16 h4;
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (on[j]) {
                h4 o;
                o[0] = (f16)keep_f32(fmaf((h[j].x - mu) * rstd, gq[j].x, bq[j].x));
                o[1] = (f16)keep_f32(fmaf((h[j].y - mu) * rstd, gq[j].y, bq[j].y));
                o[2] = (f16)keep_f32(fmaf((h[j].z - mu) * rstd, gq[j].z, bq[j].z));
                o[3] = (f16)keep_f32(fmaf((h[j].w - mu) * rstd, gq[j].w, bq[j].w));
                *reinterpret_cast<h4*>(a + row * d + 256 * j + 4 * lane) = o;
            }
    }
}

inline unsigned grid_rows(int64_t rows) {
    return (unsigned)((rows + kRowsPerBlock - 1) / kRowsPerBlock);
}

}  // namespace

template <typename TKV, typename TA>
hipError_t launch_init_layernorm(const TKV* x, float* g, TA* a, int64_t rows, int d,
                                 const float* gain, const float* shift, float eps, const WorkList* wl,
                                 hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (wl != nullptr && wl->U > kListMaxUsers) return hipErrorInvalidValue;
    const unsigned grid = grid_rows(rows) + (wl != nullptr);
    const WorkList w = wl != nullptr ? *wl : WorkList{};
    if (d % 256 == 0 && wl != nullptr)
        k_init_layernorm<true, true, TKV, TA><<<grid, 256, 0, s>>>(x, g, a, rows, d, gain, shift, eps, w);
    else if (d % 256 == 0)
        k_init_layernorm<true, false, TKV, TA><<<grid, 256, 0, s>>>(x, g, a, rows, d, gain, shift, eps, w);
    else if (wl != nullptr)
        k_init_layernorm<false, true, TKV, TA><<<grid, 256, 0, s>>>(x, g, a, rows, d, gain, shift, eps, w);
    else
        k_init_layernorm<false, false, TKV, TA><<<grid, 256, 0, s>>>(x, g, a, rows, d, gain, shift, eps, w);
    return hipGetLastError();
}

template <typename TA>
hipError_t launch_layernorm(const float* g, TA* a, int64_t rows, int d, const float* gain,
                            const float* shift, float eps, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (d % 256 == 0)
        k_layernorm<true, TA><<<grid_rows(rows), 256, 0, s>>>(g, a, rows, d, gain, shift, eps);
    else
        k_layernorm<false, TA><<<grid_rows(rows), 256, 0, s>>>(g, a, rows, d, gain, shift, eps);
    return hipGetLastError();
}

template <typename TKV>
hipError_t launch_init_layernorm_mx(const TKV* x, float* g, uint8_t* codes, uint8_t* scales,
                                    int64_t rows, int d, const float* gain, const float* shift,
                                    float eps, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (d % 256 != 0) return hipErrorInvalidValue;
    k_layernorm_mx<true, TKV><<<grid_rows(rows), 256, 0, s>>>(x, g, codes, scales, rows, d, gain,
                                                             shift, eps);
    return hipGetLastError();
}

hipError_t launch_layernorm_mx(const float* g, uint8_t* codes, uint8_t* scales, int64_t rows,
                               int d, const float* gain, const float* shift, float eps,
                               hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (d % 256 != 0) return hipErrorInvalidValue;
    k_layernorm_mx<false, float><<<grid_rows(rows), 256, 0, s>>>(nullptr, const_cast<float*>(g),
                                                                codes, scales, rows, d, gain,
                                                                shift, eps);
    return hipGetLastError();
}

hipError_t launch_score_head(const float* g, float* scores, int64_t rows, int d,
                             const FinalWeights& fw, float eps, hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (d % 256 == 0)
        k_score_head<true><<<grid_rows(rows), 256, 0, s>>>(g, scores, rows, d, fw.lnf_g, fw.lnf_b,
                                                           fw.w_score, fw.b_score, eps);
    else
        k_score_head<false><<<grid_rows(rows), 256, 0, s>>>(g, scores, rows, d, fw.lnf_g,
                                                            fw.lnf_b, fw.w_score, fw.b_score, eps);
    return hipGetLastError();
}

hipError_t launch_block_layernorm(const float* g, f16* a, int64_t rows, int d, const float* gain,
                                  const float* shift, float eps, const FinalWeights* fw, float* scores,
                                  hipStream_t s) {
    if (rows == 0) return hipSuccess;
    if (d % 64 != 0 || d > kResidLnMaxN) return hipErrorInvalidValue;
    if (scores != nullptr)
        k_block_layernorm<true><<<grid_rows(rows), 256, 0, s>>>(g, nullptr, rows, d, gain, shift, eps,
                                                               fw->w_score, fw->b_score, scores);
    else
        k_block_layernorm<false><<<grid_rows(rows), 256, 0, s>>>(g, a, rows, d, gain, shift, eps, nullptr,
                                                                nullptr, nullptr);
    return hipGetLastError();
}

template hipError_t launch_init_layernorm<float, float>(const float*, float*, float*, int64_t, int,
                                                        const float*, const float*, float,
                                                        const WorkList*, hipStream_t);
template hipError_t launch_init_layernorm<bf16, f16>(const bf16*, float*, f16*, int64_t, int,
                                                     const float*, const float*, float,
                                                     const WorkList*, hipStream_t);
template hipError_t launch_init_layernorm_mx<bf16>(const bf16*, float*, uint8_t*, uint8_t*,
                                                   int64_t, int, const float*, const float*,
                                                   float, hipStream_t);
template hipError_t launch_layernorm<float>(const float*, float*, int64_t, int, const float*,
                                            const float*, float, hipStream_t);
template hipError_t launch_layernorm<f16>(const float*, f16*, int64_t, int, const float*,
                                          const float*, float, hipStream_t);

}  // namespace upr
