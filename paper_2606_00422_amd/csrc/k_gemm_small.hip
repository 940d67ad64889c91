// Projection GEMM on small tiles: out = A[M,K] W[N,K]^T (+ epilogue), the
// product of k_gemm_mfma.hip for calls whose large tiles would leave compute
// units idle (fp16 operands), and the projections of fp32 models
// (v_mfma_f32_16x16x4_f32).
//
// What bounds a small call is latency: a workgroup walks its whole K with
// nobody beside it on the compute unit.  So the block tile is small and four
// waves take a quarter of it each: 64 x 64 for fp16, 32 x 32 for fp32 (whose
// MFMAs run 16 times longer per K value: in a 64 x 64 block their dependent
// chain alone takes twice as long), 128 x 128 for large fp32 calls.  Every wave
// issues a share of the loads, straight into LDS, and four LDS stages of one
// 128-byte K-step each (two for 128 x 128, where another workgroup's work
// covers the latency) keep three K-steps in flight with a single barrier per
// step: wait for the own loads of step t, barrier, refill the stage that step
// t - 1 read, read the fragments of step t, multiply those of step t - 1.  (Eight stages were no faster for any
// K up to 4096: the steps are bound by the LDS port, 16 KB written and 32 KB
// read per step, and by the barrier, not by the loads' latency.)
//
// fp16: every output element is the same chain of MFMAs over K in the same
// order as in the large tiles, and the epilogue the same arithmetic, so the
// choice of tile never changes a result.  The same holds between the tiles
// of fp32 models.
//
// Measured (us per launch, back to back; large tiles -> this kernel): fp16
// 2000 x 512, K 2048: 20.3 -> 11.2; K 512: 8.7 -> 5.6 (in a call, on weights that
// are not in L2 yet, the two average 12.0); 1000 x 2048, K 512: 9.3 -> 6.3.
// fp32 (FMA kernel -> this one) 2132 x 768, K 256: 37 -> 12.4;
// 128 x 256, K 256: 34 -> 4.2; 8000 x 2048, K 512: 315 -> 138 (121 TFLOP/s).
//
// fp32: a 128-byte row is 32 values; lane group g = lane / 16 takes 16-byte
// chunk 4kk + g, so MFMA i of fragment kk multiplies K values 16kk + 4g + i.
// Even and odd K-steps have sums of their own, added at the end: chains of half
// the length (error of a call's scores against 64 bits, d 256, 2 layers: 1.0e-6
// with one chain, as with the FMA kernel, 7.4e-7 with two; 1% of the call).
//
// Epilogue: the accumulators are staged through LDS (row stride + 16 bytes:
// conflict-free both ways) and read back row-contiguous, four fp32 or eight
// 16-bit columns per lane.  Ordinary stores: the outputs of small calls are
// read back from L2 by the next launch.
#include "gemm_tile.h"

namespace upr {

namespace gemm_detail {

// Per operand type: the MFMA (kMT x kMT outputs, transposed: W first), how
// many 16-byte fragments of a 128-byte row a lane takes, and where its
// accumulator registers lie: quad q of an MFMA tile holds four consecutive
// columns from quad_col(q, lane) of row lane % kMT.
template <typename TA> struct Operand;
template <> struct Operand<f16> {
    typedef h8 frag;
    typedef f32x16 acc;
    static constexpr int kMT = 32, kFrags = 4, kQuads = 4;
    static __device__ __forceinline__ int quad_col(int q, int lane) { return 8 * q + 4 * (lane >> 5); }
    static __device__ __forceinline__ void mma(const frag& w, const frag& a, acc& c) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(w, a, c, 0, 0, 0);
    }
};
template <> struct Operand<float> {
    typedef f32x4 frag;
    typedef f32x4 acc;
    static constexpr int kMT = 16, kFrags = 2, kQuads = 1;
    static __device__ __forceinline__ int quad_col(int, int lane) { return 4 * (lane >> 4); }
    static __device__ __forceinline__ void mma(const frag& w, const frag& a, acc& c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], a[i], c, 0, 0, 0);
    }
};

// GELU of fp32 models.
__device__ __forceinline__ float gelu_tanh_f(float x) {
    // 0.5 x (1 + tanh(sqrt(2/pi) (x + 0.044715 x^3)))
    const float k0 = 0.7978845608028654f;
    const float y = k0 * (x + 0.044715f * x * x * x);
    return 0.5f * x * (1.0f + tanhf(y));
}

constexpr int kSmallThreads = 256;

// kB: block tile rows and columns; each of the four waves takes a quarter,
// kT x kT MFMA tiles.  kAhead: fragments are read one K-step ahead of their
// MFMAs (a second set of registers).
template <typename TA, typename TKV, int MODE, int kB>
__global__ __launch_bounds__(kSmallThreads, kB == 128 ? 2 : 1) void k_gemm_small(
    const TA* __restrict__ A, int64_t lda, const TA* __restrict__ W, int64_t M, int N, int K, Epilogue epi) {
    using Op = Operand<TA>;
    constexpr int kMT = Op::kMT, kT = kB / 2 / kMT;
    constexpr int kE = sizeof(TA), kRow = 128;      // bytes of a value, of an LDS row
    constexpr int kLoads = kB / 32;                 // 8-row loads per wave, operand and stage
    constexpr bool kAhead = kB < 128;
    constexpr int kStages = kB < 128 ? 4 : 2;
    constexpr int kLd = kB + 4;                     // row stride of the staged output (values)
    constexpr int kHalf = kB * kRow, kStage = 2 * kHalf;    // A rows, then W rows
    constexpr int kOut = 2 * kMT * kLd * 4;         // epilogue staging: 2 kMT rows per pass, in stage 0
    // separate arrays: the compiler can then tell that fragment reads of one
    // stage do not alias the loads in flight to the others
    constexpr int k4 = kStages == 4 ? kStage : 16;
    __shared__ __attribute__((aligned(16))) char s0[kOut > kStage ? kOut : kStage], s1[kStage], s2[k4], s3[k4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane % kMT, lgrp = lane / kMT;
    const int tiles_n = (N + kB - 1) / kB;
    const int t = xcd_tile(blockIdx.x, gridDim.x);
    const int64_t m0 = (int64_t)(t / tiles_n) * kB;
    const int n0 = (t % tiles_n) * kB;

    // rows past M (N) fall outside the descriptors and load as zeros
    const int64_t rows_a = M - m0 < kB ? M - m0 : kB;
    const int rows_b = N - n0 < kB ? N - n0 : kB;
    const __amdgpu_buffer_rsrc_t rsA = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(A + m0 * lda), (short)0, (int)(rows_a * lda * kE), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsB = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(W + (int64_t)n0 * K), (short)0, (int)((int64_t)rows_b * K * kE), 0x00020000);

    typename Op::acc acc[kT][kT];                   // [column tile][row tile]
    typename Op::acc acc_odd[kT][kT];               // fp32: the odd K-steps' sums
#pragma unroll
    for (int j = 0; j < kT; ++j)
#pragma unroll
        for (int i = 0; i < kT; ++i)
#pragma unroll
            for (int r = 0; r < 4 * Op::kQuads; ++r) acc[j][i][r] = acc_odd[j][i][r] = 0.f;
    // accumulators of an FFN down that carries the residual (Epilogue::acc_resid)
    if constexpr (MODE == EPI_RESID) {
        if (epi.acc_resid) {
            const float inv = 1.0f / epi.acc_scale;     // a power of two: exact
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                epi.resid + m0 * epi.ldr, (short)0, (int)(rows_a * epi.ldr * 4), 0x00020000);
#pragma unroll
            for (int j = 0; j < kT; ++j)
#pragma unroll
                for (int i = 0; i < kT; ++i)
#pragma unroll
                    for (int q = 0; q < Op::kQuads; ++q) {
                        const int col = n0 + (wn * kT + j) * kMT + Op::quad_col(q, lane);
                        const int row = (wm * kT + i) * kMT + lrow;
                        float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (col < N)                    // N is a multiple of 8
                            r = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(
                                                               rs, (unsigned)(row * epi.ldr + col) * 4u, 0, 0));
                        acc[j][i][4 * q + 0] = r.x * inv;
                        acc[j][i][4 * q + 1] = r.y * inv;
                        acc[j][i][4 * q + 2] = r.z * inv;
                        acc[j][i][4 * q + 3] = r.w * inv;
                    }
        }
    }

    // A load instruction fills 64 16-byte slots = 8 rows; load i of a wave
    // covers rows 8 (4i + wave) + lane / 8, slot s of row r holding chunk
    // s ^ (r / 2) % 8 (rows 32 apart share the key).
    const int lr = 8 * wave + (lane >> 3);
    const int ch = ((lane & 7) ^ ((lr >> 1) & 7)) << 4;
    const int voA = (int)(lr * lda * kE) + ch, voB = lr * K * kE + ch;
    const int stepA = (int)(32 * lda * kE), stepB = 32 * K * kE;
    auto issue = [&](char* dst, int step) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsA, (__attribute__((address_space(3))) void*)(dst + (4 * i + wave) * 8 * kRow), 16,
                voA + i * stepA + step * kRow, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rsB, (__attribute__((address_space(3))) void*)(dst + kHalf + (4 * i + wave) * 8 * kRow), 16,
                voB + i * stepB + step * kRow, 0, 0, 0);
    };
    // fragment kk of a row: chunk (64 / kMT) kk + lgrp
    int off[Op::kFrags];
#pragma unroll
    for (int kk = 0; kk < Op::kFrags; ++kk)
        off[kk] = lrow * kRow + ((((64 / kMT) * kk + lgrp) ^ ((lrow >> 1) & 7)) << 4);
    const int nk = K * kE / kRow;
    typename Op::frag fa[kAhead ? 2 : 1][Op::kFrags][kT], fb[kAhead ? 2 : 1][Op::kFrags][kT];
    // fragments of set `set`, of a K-step of parity `par`
    auto multiply = [&](auto set, auto par) __attribute__((always_inline)) {
        constexpr int X = decltype(set)::value;
        constexpr bool kOdd = sizeof(TA) == 4 && decltype(par)::value != 0;
#pragma unroll
        for (int kk = 0; kk < Op::kFrags; ++kk)
#pragma unroll
            for (int j = 0; j < kT; ++j)
#pragma unroll
                for (int i = 0; i < kT; ++i) Op::mma(fb[X][kk][j], fa[X][kk][i], kOdd ? acc_odd[j][i] : acc[j][i]);
    };
    auto kstep = [&](const char* cur, char* nxt, int step, auto par) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value, X = kAhead ? P : 0;
        // steps step+1 .. step+kStages-2 may stay in flight
        constexpr int kFly = (kStages - 2) * 2 * kLoads;
        static_assert(kFly < 64, "vmcnt field");
        __builtin_amdgcn_sched_barrier(0);          // the previous step's reads and MFMAs stay above
        if (step + kStages - 2 < nk)                // lgkmcnt(0): the last step's fragments are here
            __builtin_amdgcn_s_waitcnt(0x0070 | (kFly & 15) | ((kFly >> 4) << 14));
        else
            __builtin_amdgcn_s_waitcnt(0x0070);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if (step + kStages - 1 < nk) issue(nxt, step + kStages - 1);
#pragma unroll
        for (int kk = 0; kk < Op::kFrags; ++kk) {
#pragma unroll
            for (int i = 0; i < kT; ++i)
                fa[X][kk][i] = *reinterpret_cast<const typename Op::frag*>(cur + (wm * kT + i) * kMT * kRow + off[kk]);
#pragma unroll
            for (int j = 0; j < kT; ++j)
                fb[X][kk][j] =
                    *reinterpret_cast<const typename Op::frag*>(cur + kHalf + (wn * kT + j) * kMT * kRow + off[kk]);
        }
        if constexpr (kAhead) {
            __builtin_amdgcn_sched_barrier(0);      // the reads are issued before the MFMAs
            if (step > 0) multiply(std::integral_constant<int, 1 - X>{}, std::integral_constant<int, 1 - P>{});
        } else {
            multiply(std::integral_constant<int, X>{}, par);
        }
    };
    typedef std::integral_constant<int, 0> even;
    typedef std::integral_constant<int, 1> odd;
    issue(s0, 0);
    int kt = 0;
    if constexpr (kStages == 4) {
        if (nk > 1) issue(s1, 1);
        if (nk > 2) issue(s2, 2);
        for (; kt + 4 <= nk; kt += 4) {
            kstep(s0, s3, kt, even{});
            kstep(s1, s0, kt + 1, odd{});
            kstep(s2, s1, kt + 2, even{});
            kstep(s3, s2, kt + 3, odd{});
        }
        if (kt < nk) kstep(s0, s3, kt, even{});
        if (kt + 1 < nk) kstep(s1, s0, kt + 1, odd{});
        if (kt + 2 < nk) kstep(s2, s1, kt + 2, even{});
    } else {
        for (; kt + 2 <= nk; kt += 2) {
            kstep(s0, s1, kt, even{});
            kstep(s1, s0, kt + 1, odd{});
        }
        if (kt < nk) kstep(s0, s1, kt, even{});
    }
    if constexpr (kAhead) {
        if (nk & 1)
            multiply(even{}, even{});
        else
            multiply(odd{}, odd{});
    }
    if constexpr (sizeof(TA) == 4) {
#pragma unroll
        for (int j = 0; j < kT; ++j)
#pragma unroll
            for (int i = 0; i < kT; ++i) acc[j][i] += acc_odd[j][i];
    }

    // ---- epilogue.  Pass i stages row tile i of both wave rows: LDS row
    // kMT wm + lane % kMT.
    float* const sOut = reinterpret_cast<float*>(s0);
    constexpr int kPass = 2 * kMT;
    auto stage_out = [&](int i) __attribute__((always_inline)) {
        __syncthreads();                            // the fragment reads, or the previous pass's, are done
#pragma unroll
        for (int j = 0; j < kT; ++j)
#pragma unroll
            for (int q = 0; q < Op::kQuads; ++q)
                *reinterpret_cast<float4*>(sOut + (wm * kMT + lrow) * kLd + (wn * kT + j) * kMT +
                                           Op::quad_col(q, lane)) =
                    make_float4(acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]);
        __syncthreads();
    };
    // row of the block tile that staged row s of pass i holds
    auto out_row = [&](int s, int i) { return (s / kMT) * (kMT * kT) + kMT * i + s % kMT; };
    const float sc = epi.acc_scale;
    if constexpr (MODE == EPI_RESID) {
        constexpr int kC4 = kB / 4;                 // float4 per row
        const int c = tid % kC4, col = n0 + 4 * c;
        const bool col_ok = col < N;
        const float4 b4 = col_ok ? *reinterpret_cast<const float4*>(epi.bias + col) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int i = 0; i < kT; ++i) {
          stage_out(i);
#pragma unroll
          for (int sr = tid / kC4; sr < kPass; sr += kSmallThreads / kC4) {
            const int r = out_row(sr, i);
            if (r >= rows_a || !col_ok) continue;
            const float4 x = *reinterpret_cast<const float4*>(sOut + sr * kLd + 4 * c);
            float4* const dst = reinterpret_cast<float4*>(epi.resid + (m0 + r) * epi.ldr + col);
            float4 v = make_float4(fmaf(x.x, sc, b4.x), fmaf(x.y, sc, b4.y), fmaf(x.z, sc, b4.z), fmaf(x.w, sc, b4.w));
            if (!epi.acc_resid) {
                float4 g;
                if (epi.resid_src != nullptr) {     // bf16 token rows
                    const uint2 w = *reinterpret_cast<const uint2*>(
                        static_cast<const unsigned short*>(epi.resid_src) + (m0 + r) * epi.ldr + col);
                    g = make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
                                    __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
                } else {
                    g = *dst;
                }
                v = make_float4(g.x + v.x, g.y + v.y, g.z + v.z, g.w + v.w);
            }
            *dst = v;
          }
        }
    } else {
        constexpr bool kGelu = MODE == EPI_GELU || MODE == EPI_GELU_PERM;
        constexpr int kC8 = kB / 8;                 // eight columns per lane
        const int c = tid % kC8, col = n0 + 8 * c;
        const bool col_ok = col < N;
        // EPI_GELU_PERM: positions 8c .. 8c+7 of a row hold, within their
        // 16-column group, columns 4p .. 4p+3 and 8+4p .. 8+4p+3 (p = c % 2)
        const int c0 = MODE == EPI_GELU_PERM ? 16 * (c / 2) + 4 * (c & 1) : 8 * c;
        const int c1 = MODE == EPI_GELU_PERM ? c0 + 8 : c0 + 4;
        float bq[8], cq = sc;
        if (col_ok) {
            float cs = 1.0f;
            if constexpr (!kGelu) cs = col < (MODE == EPI_STORE ? epi.scale_cols : epi.d_model) ? epi.col_scale : 1.0f;
            cq = sc * cs;
#pragma unroll
            for (int e = 0; e < 8; ++e) bq[e] = epi.bias[n0 + (e < 4 ? c0 + e : c1 + e - 4)] * cs;
        }
        typedef std::conditional_t<kGelu, TA, TKV> TO;
        TO* obase = static_cast<TO*>(epi.out) + m0 * epi.ldo + col;
        int64_t ostride = epi.ldo;
        if constexpr (MODE == EPI_QKV_CACHE) {
            const int d = epi.d_model;
            if (col >= d) {                         // eight columns never straddle a head
                const int part = col >= 2 * d ? 2 : 1;
                const int cc = col - part * d;
                const int h = cc / epi.head_dim, e = cc - h * epi.head_dim;
                obase = static_cast<TO*>(part == 1 ? epi.cache_k : epi.cache_v) +
                        ((int64_t)h * epi.cache_cap + epi.row0 + m0) * epi.head_dim + e;
                ostride = epi.head_dim;
            }
        }
#pragma unroll
        for (int i = 0; i < kT; ++i) {
          stage_out(i);
#pragma unroll
          for (int sr = tid / kC8; sr < kPass; sr += kSmallThreads / kC8) {
            const int r = out_row(sr, i);
            if (r >= rows_a || !col_ok) continue;
            const float4 x = *reinterpret_cast<const float4*>(sOut + sr * kLd + c0);
            const float4 y = *reinterpret_cast<const float4*>(sOut + sr * kLd + c1);
            float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                v[e] = fmaf(v[e], cq, bq[e]);
                if constexpr (kGelu) v[e] = sizeof(TA) == 2 ? gelu_fast(v[e]) : gelu_tanh_f(v[e]);
            }
            TO* const op = obase + r * ostride;
            if constexpr (sizeof(TO) == 2) {
                constexpr bool kBf = !kGelu;
                *reinterpret_cast<u32x4*>(op) = u32x4{pack2<kBf>(v[0], v[1]), pack2<kBf>(v[2], v[3]),
                                                      pack2<kBf>(v[4], v[5]), pack2<kBf>(v[6], v[7])};
            } else {
                *reinterpret_cast<float4*>(op) = make_float4(v[0], v[1], v[2], v[3]);
                *reinterpret_cast<float4*>(op + 4) = make_float4(v[4], v[5], v[6], v[7]);
            }
          }
        }
    }
}

template <typename TA, typename TKV, int MODE>
hipError_t launch_small_mode(const TA* A, int64_t lda, const TA* W, int64_t M, int N, int K, const Epilogue& epi,
                             int block, hipStream_t s) {
    const int64_t tiles = ((M + block - 1) / block) * (int64_t)((N + block - 1) / block);
    constexpr int kB = sizeof(TA) == 2 ? 64 : 32;
    if (block == kB) {
        k_gemm_small<TA, TKV, MODE, kB><<<(unsigned)tiles, kSmallThreads, 0, s>>>(A, lda, W, M, N, K, epi);
        return hipGetLastError();
    }
    if constexpr (sizeof(TA) == 4) {
        if (block == 128) {
            k_gemm_small<TA, TKV, MODE, 128><<<(unsigned)tiles, kSmallThreads, 0, s>>>(A, lda, W, M, N, K, epi);
            return hipGetLastError();
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace gemm_detail

template <typename TA, typename TKV>
hipError_t launch_gemm_small(const TA* A, int64_t lda, const TA* W, int64_t M, int N, int K, const Epilogue& epi,
                             int block, hipStream_t s) {
    using namespace gemm_detail;
    if (M == 0) return hipSuccess;
    constexpr int kE = sizeof(TA);
    // whole 128-byte K-steps, 16-byte operand loads, eight output columns a lane
    if (K <= 0 || K * kE % 128 != 0 || lda * kE % 16 != 0 || N % 8 != 0) return hipErrorInvalidValue;
    switch (epi.mode) {
        case EPI_STORE:
            if (epi.ldo % 8 != 0 || epi.scale_cols % 8 != 0) return hipErrorInvalidValue;
            return launch_small_mode<TA, TKV, EPI_STORE>(A, lda, W, M, N, K, epi, block, s);
        case EPI_GELU:
            if (epi.ldo % 8 != 0) return hipErrorInvalidValue;
            return launch_small_mode<TA, TKV, EPI_GELU>(A, lda, W, M, N, K, epi, block, s);
        case EPI_RESID:
            if (epi.ldr % 4 != 0) return hipErrorInvalidValue;
            return launch_small_mode<TA, TKV, EPI_RESID>(A, lda, W, M, N, K, epi, block, s);
        case EPI_QKV_CACHE:
            if (epi.ldo % 8 != 0 || epi.head_dim % 8 != 0 || epi.d_model % 8 != 0) return hipErrorInvalidValue;
            return launch_small_mode<TA, TKV, EPI_QKV_CACHE>(A, lda, W, M, N, K, epi, block, s);
        case EPI_GELU_PERM:
            if constexpr (sizeof(TA) == 2) {
                if (epi.ldo % 16 != 0 || N % 16 != 0) return hipErrorInvalidValue;
                return launch_small_mode<TA, TKV, EPI_GELU_PERM>(A, lda, W, M, N, K, epi, block, s);
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_gemm_small<f16, bf16>(const f16*, int64_t, const f16*, int64_t, int, int, const Epilogue&,
                                                 int, hipStream_t);

// fp32 models: 32 x 32 tiles, whose time grows with their number, or 128 x 128
// ones, which cost less per output but run in rounds of one per compute unit.
// Per 32 x 32 outputs the large ones take 0.88 (K + 60) / (K + 100) of the small
// ones' time (the constants are the ends of a tile, in K values: per 1000 tiles
// of 32 x 32, K 64: 1.8 and 2.8 us; K 256: 4.4 and 5.5; K 2048: 30 and 35), so
// that they win where their rounds are full enough.  us, small / large: K 512,
// 2634 x 1536 (252 large tiles) 41 / 39, 3298 x 1536 (312) 50 / 66; K 256,
// 27456 x 256 (430) 43 / 38; K 2048, 8908 x 1024 (560) 320 / 371.  Over 150
// shapes of 60 to 1560 large tiles the choice costs at most 9% and 0.2% on
// average against the faster (large tiles from 504 up: 25% and 2.2%).
template <>
hipError_t launch_gemm<float, float>(const float* A, int64_t lda, const float* W, int64_t M, int N, int K,
                                     const Epilogue& epi, hipStream_t s) {
    if (epi.resid_src != nullptr) return hipErrorInvalidValue;      // fp32 residual rows only
    const int64_t cus = gemm_detail::device_cus();
    const int64_t tiles32 = ((M + 31) / 32) * (int64_t)((N + 31) / 32);
    const int64_t tiles128 = ((M + 127) / 128) * (int64_t)((N + 127) / 128);
    const int64_t rounds = (tiles128 + cus - 1) / cus;
    const bool large = 0.88 * (K + 60) * 16.0 * (double)(rounds * cus) <= (double)(K + 100) * (double)tiles32;
    return launch_gemm_small<float, float>(A, lda, W, M, N, K, epi, large ? 128 : 32, s);
}

}  // namespace upr
