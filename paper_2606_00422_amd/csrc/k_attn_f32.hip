// Attention of fp32 models on the fp32 matrix instructions
// (v_mfma_f32_16x16x4_f32, exact fp32 products, fp32 sums): the ranking pass
// and the causal encode pass, as k_attn_mfma.hip defines them.
//
// One workgroup = one work item (user, head, up to 32 queries); its four
// waves are two groups of 16 queries times two halves of the keys, so that a
// wave's serial walk is half the history and a small call still spreads over
// the device (2132 candidates, 4 heads: 280 workgroups).  K/V stream through
// LDS in double-buffered 16 KB stages shared by all four waves; key half kh
// takes the stage's keys [kh kKS/2, (kh+1) kKS/2), 16 at a time:
//   S^T = K Q^T   (keys x queries): a lane holds the logits of keys 4g + r of
//                 one query (g = lane / 16, r = 0..3);
//   O^T += V^T P^T: register r of the probabilities is the B operand whose
//                 four k-indices are keys 4g + r, one per lane group.
// The contraction over features takes 16-byte chunks (lane group g chunk
// 4c + g, MFMA i its value i) and V's columns are dealt out as e = kEB m + j
// (e-block j, m = lane % 16), so that one 16- or 8-byte LDS read of a V row
// feeds every e-block and a lane ends with 4 kEB consecutive outputs.
//
// The softmax is exact: a running maximum per query (fp32 logits, starting
// from the query's own logit), probabilities and sums fp32, O rescaled when
// the maximum moves; the two key halves are merged through LDS.  (The bare
// exponential instruction: probabilities below 2^-126 of the largest are 0.)
//
// Bound by the fp32 matrix rate (157 TFLOP/s nominal): per 16 keys a wave
// issues D/2 MFMAs of 32 cycles and about 60 VALU instructions.  Ranking 4
// users (150-450 rows, 300-700 candidates, 4 heads of 64): 21.2 us per layer
// (20.7 with one chain per sum), 175 on the one-wave-per-row kernel.
#include <type_traits>

#include "attn_row.h"
#include "upr_plan.h"

namespace upr {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;

__device__ __forceinline__ float quad_max(float v) {
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ float quad_sum(float v) {
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}

// qsrc: ranking, q|k|v rows (stride 3d); encode, query rows (stride d, own
// keys in the cache).  Queries are pre-scaled by log2(e)/sqrt(D).
template <bool CAUSAL, int D>
__global__ __launch_bounds__(256, 2) void k_attn_f32(const float* __restrict__ qsrc, int64_t qstride,
                                                     float* __restrict__ out, int64_t row0, int H,
                                                     const int4* __restrict__ work,
                                                     const float* __restrict__ cache_k,
                                                     const float* __restrict__ cache_v, int64_t cap) {
    constexpr int kKS = 4096 / D;           // keys per stage (16 KB each of K and V)
    constexpr int kCR = D / 4;              // 16-byte chunks per row
    constexpr int kC = D / 16;              // chunks per lane of a K or Q row
    constexpr int kEB = D / 16;             // 16-column blocks of O
    constexpr int kRPL = 64 / kCR;          // rows per 64-lane load
    constexpr int kLoads = kKS / 4 / kRPL;  // loads per wave and matrix
    __shared__ __attribute__((aligned(16))) float sK0[kKS * D], sK1[kKS * D], sV0[kKS * D], sV1[kKS * D];

    const int4 item = work[blockIdx.x];
    const int h = item.w & 0xffff, kc = item.w >> 16;
    if (kc <= 0) return;
    const int64_t c0 = item.z, hb = item.x;
    const int n = item.y;
    if (hb < 0 || n < 0 || hb + n > cap) return;    // (never, for an item of the work list)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qg = wave & 1, kh = wave >> 1;
    const int g = lane >> 4, l16 = lane & 15;
    const int d = H * D;
    const int ipos0 = CAUSAL ? (int)(c0 - hb) : 0;
    const int nkeys = CAUSAL ? ipos0 + kc : n;
    const int nst = (nkeys + kKS - 1) / kKS;
    const bool active = qg * 16 < kc;               // wave-uniform

    // rows past the history end read as zeros; slot s of K row r holds chunk
    // s ^ key(r): 16 consecutive rows at one chunk fall on distinct bank
    // groups (V rows are read whole and need no swizzle)
    const __amdgpu_buffer_rsrc_t rsK = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(cache_k + ((int64_t)h * cap + hb) * D), (short)0, n * D * 4, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsV = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(cache_v + ((int64_t)h * cap + hb) * D), (short)0, n * D * 4, 0x00020000);
    auto key = [](int row) { return D == 64 ? row & 15 : (row >> 1) & 7; };
    static_assert(kLoads == 4, "the same for either head_dim");
    int offK[4], offV[4];   // (fixed size: a template-dependent one makes the host pass drop the launch stub)
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int row = (wave * kLoads + i) * kRPL + lane / kCR, slot = lane % kCR;
        offK[i] = row * D * 4 + ((slot ^ key(row)) << 4);
        offV[i] = row * D * 4 + (slot << 4);
    }
    auto issue = [&](float* dK, float* dV, int st) __attribute__((always_inline)) {
        const int base = st * kKS * D * 4;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsK, (__attribute__((address_space(3))) void*)(dK + (wave * kLoads + i) * kRPL * D), 16,
                offK[i] + base, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsV, (__attribute__((address_space(3))) void*)(dV + (wave * kLoads + i) * kRPL * D), 16,
                offV[i] + base, 0, 0, 0);
        }
    };
    if (nst > 0) issue(sK0, sV0, 0);

    // ---- the lane's query (clamped in a ragged tail), own logit, start
    int qi = qg * 16 + l16;
    qi = qi < kc ? qi : kc - 1;
    const int qpos = ipos0 + qi;
    const float* const qrow = qsrc + (c0 - row0 + qi) * qstride + h * D;
    const float* const krow = CAUSAL ? cache_k + ((int64_t)h * cap + c0 + qi) * D : qrow + d;
    f32x4 q[kC];
    float own = 0.f;
#pragma unroll
    for (int c = 0; c < kC; ++c) {
        q[c] = *reinterpret_cast<const f32x4*>(qrow + (4 * c + g) * 4);
        const f32x4 k = *reinterpret_cast<const f32x4*>(krow + (4 * c + g) * 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) own = fmaf(q[c][i], k[i], own);
    }
    float m = quad_sum(own);
    // ranking: the own key and value belong to key half 0 (encode streams
    // the diagonal key)
    const bool with_own = !CAUSAL && kh == 0;
    float l = with_own && g == 0 ? 1.f : 0.f;
    // o[j][r]: e = kEB (4g + r) + j; the odd keys of a lane group in oo (two sums
    // of half the length each, added at the end: half their rounding error)
    f32x4 o[kEB], oo[kEB];
#pragma unroll
    for (int j = 0; j < kEB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            o[j][r] = with_own ? qrow[2 * d + kEB * (4 * g + r) + j] : 0.f;
            oo[j][r] = 0.f;
        }

    // 16 keys, rows kb .. kb + 15 of the stage, keys kabs .. of the user
    auto block = [&](const float* cK, const float* cV, int kb, int kabs) __attribute__((always_inline)) {
        f32x4 s = {0.f, 0.f, 0.f, 0.f}, so = s;     // (two sums, as for o)
        const int row = kb + l16;
#pragma unroll
        for (int c = 0; c < kC; ++c) {
            const f32x4 k = *reinterpret_cast<const f32x4*>(cK + row * D + (((4 * c + g) ^ key(row)) << 2));
#pragma unroll
            for (int i = 0; i < 4; i += 2) {
                s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i], q[c][i], s, 0, 0, 0);
                so = __builtin_amdgcn_mfma_f32_16x16x4f32(k[i + 1], q[c][i + 1], so, 0, 0, 0);
            }
        }
        mfma_settled<16>();
        s += so;
        if (__builtin_expect(CAUSAL ? kabs + 15 > ipos0 + qg * 16 : kabs + 16 > n, 0)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int kk = kabs + 4 * g + r;
                if (CAUSAL ? kk > qpos : kk >= n) s[r] = -INFINITY;
            }
        }
        const float top = quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
        if (__any(top > m)) {                       // the same test for all lanes of the wave
            const float mn = fmaxf(m, top);
            const float alpha = __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= alpha;
#pragma unroll
            for (int j = 0; j < kEB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    o[j][r] *= alpha;
                    oo[j][r] *= alpha;
                }
        }
        float p[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(s[r] - m);
        l += (p[0] + p[1]) + (p[2] + p[3]);
        typedef std::conditional_t<D == 64, f32x4, f32x2> vrow;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const vrow v = *reinterpret_cast<const vrow*>(cV + (kb + 4 * g + r) * D + kEB * l16);
#pragma unroll
            for (int j = 0; j < kEB; ++j) {
                f32x4& sum = r & 1 ? oo[j] : o[j];
                sum = __builtin_amdgcn_mfma_f32_16x16x4f32(v[j], p[r], sum, 0, 0, 0);
            }
        }
    };
    const int wave_last = ipos0 + min(qg * 16 + 16, kc) - 1;    // encode: the wave's last query position
    auto stage = [&](const float* cK, const float* cV, float* nK, float* nV, int st) __attribute__((always_inline)) {
        if (st + 1 < nst) issue(nK, nV, st + 1);
        if (active) {
            for (int kb = kh * (kKS / 2); kb < (kh + 1) * (kKS / 2); kb += 16) {
                const int kabs = st * kKS + kb;
                if (kabs >= nkeys || (CAUSAL && kabs > wave_last)) break;
                block(cK, cV, kb, kabs);
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);         // vmcnt(0): next stage landed
        __syncthreads();
    };
    if (nst > 0) __builtin_amdgcn_s_waitcnt(0x0F70);
    __syncthreads();
    int st = 0;
    for (; st + 2 <= nst; st += 2) {
        stage(sK0, sV0, sK1, sV1, st);
        stage(sK1, sV1, sK0, sV0, st + 1);
    }
    if (st < nst) stage(sK0, sV0, sK1, sV1, st);

    mfma_settled<16>();
#pragma unroll
    for (int j = 0; j < kEB; ++j) o[j] += oo[j];
    // ---- key half 1 hands its state to half 0 through LDS (all reads of the
    // stages ended at the last barrier)
    float* const x = sK0 + qg * (64 * (4 * kEB + 2));
    if (kh == 1) {
#pragma unroll
        for (int j = 0; j < kEB; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) x[(4 * j + r) * 64 + lane] = o[j][r];
        x[4 * kEB * 64 + lane] = m;
        x[(4 * kEB + 1) * 64 + lane] = l;
    }
    __syncthreads();
    if (kh == 1) return;
    const float m1 = x[4 * kEB * 64 + lane];
    const float mm = fmaxf(m, m1);
    const float a0 = __builtin_amdgcn_exp2f(m - mm), a1 = __builtin_amdgcn_exp2f(m1 - mm);
    l = l * a0 + x[(4 * kEB + 1) * 64 + lane] * a1;
    const float inv = 1.0f / quad_sum(l);
    const bool valid = qg * 16 + l16 < kc;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kEB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            o[j][r] = (o[j][r] * a0 + x[(4 * j + r) * 64 + lane] * a1) * inv;
            bad |= nonfinite_bits(o[j][r]);
        }
    if constexpr (CAUSAL) {
        // queries that a later position's infinite or NaN value may have reached
        const unsigned long long any = __ballot(bad && valid);
        for (int i = 0; any != 0 && i < 16; ++i) {
            if ((any & (0x0001000100010001ull << i)) == 0) continue;
            const int qr = qg * 16 + i;
            const float v = causal_row<float, D>(qsrc + (c0 - row0 + qr) * qstride + h * D,
                                                 cache_k + ((int64_t)h * cap + hb) * D,
                                                 cache_v + ((int64_t)h * cap + hb) * D, ipos0 + qr);
#pragma unroll
            for (int j = 0; j < kEB; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float e = __shfl(v, kEB * (4 * g + r) + j, 64);
                    if (l16 == i) o[j][r] = e;
                }
        }
    }
    if (!valid) return;
    float* const orow = out + (c0 - row0 + qi) * d + h * D + 4 * kEB * g;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        typedef std::conditional_t<D == 64, f32x4, f32x2> vrow;
        vrow v;
#pragma unroll
        for (int j = 0; j < kEB; ++j) v[j] = o[j][r];
        *reinterpret_cast<vrow*>(orow + kEB * r) = v;
    }
}

}  // namespace

hipError_t launch_attn_f32(bool causal, const float* q, float* o, int64_t row0, int H, int D, const int32_t* work,
                           int64_t items, const float* cache_k, const float* cache_v, int64_t cache_cap,
                           hipStream_t s) {
    if (items == 0) return hipSuccess;
    if (D != 64 && D != 32) return hipErrorInvalidValue;
    const int4* w = reinterpret_cast<const int4*>(work);
    const int64_t ld = (int64_t)(causal ? 1 : 3) * H * D;
    if (causal && D == 64)
        k_attn_f32<true, 64><<<(unsigned)items, 256, 0, s>>>(q, ld, o, row0, H, w, cache_k, cache_v, cache_cap);
    else if (causal)
        k_attn_f32<true, 32><<<(unsigned)items, 256, 0, s>>>(q, ld, o, row0, H, w, cache_k, cache_v, cache_cap);
    else if (D == 64)
        k_attn_f32<false, 64><<<(unsigned)items, 256, 0, s>>>(q, ld, o, row0, H, w, cache_k, cache_v, cache_cap);
    else
        k_attn_f32<false, 32><<<(unsigned)items, 256, 0, s>>>(q, ld, o, row0, H, w, cache_k, cache_v, cache_cap);
    return hipGetLastError();
}

}  // namespace upr
