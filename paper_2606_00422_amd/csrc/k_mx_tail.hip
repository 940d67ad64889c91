// The tail of a layer of the MXFP8 variant as one kernel, for calls of enough
// rows (mx_tail_tile) and d = 256 or 512:
//   g += o Wo^T + bo;  a = mx(LN2(g));  h = mx(gelu(a W1^T + b1));
//   g += h W2^T + b2;  then mx(LN) of the updated rows (the next layer's LN1),
//   the score head, or neither (action heads follow)
// with o, a and h as E4M3 codes and E8M0 block scales.  The sequence of
// launches it replaces (O projection with LN2, FFN up, FFN down, LN1 or the
// score head) moves the fp32 residual through HBM five times a layer and the
// hidden codes twice; it is left to smaller calls, with the same bits: both
// feed the matrix cores the same 64-value products in the same order and
// round, sum and encode in the same order.
//
// One workgroup = 128 rows (or 64, TM = 2) and whole rows of the output; eight
// waves, organised as the fp16 tail (k_ffn_fused.hip): operand rows resident
// in LDS, weights straight from L2 in fragment-major order (upr_model_create),
// hidden columns in chunks of 128, up phase and GELU of chunk c before the
// down phase of chunk c - 1.  What differs:
//  * A fragment is 32 rows x 64 codes, 2 KB: lane l takes the 16-byte pieces
//    l / 32 and 2 + l / 32 of row l % 32, and the E8M0 byte of block l / 32
//    (the operand layout of v_mfma_scale_f32_32x32x64).  The weights' scale
//    bytes are stored per lane, four fragments to a dword.
//  * A wave's 32 hidden columns of a chunk are one block: its maximum is 15
//    steps in registers and one exchange between the lane halves.
//  * Codes take half the LDS, so there are two chunk buffers and one barrier
//    per chunk.
//  * The FFN down accumulators start at zero (the sum r + (acc + b) of the
//    separate GEMM), so the residual after the O projection waits in HBM (the
//    register file holds one such tile).  Whole tiles, of 128 or 64 rows, keep
//    it, between launches too, in the order of the accumulators: every access
//    is 1 KB contiguous.
//  * The last step stages 32 updated rows at a time in LDS and treats them as
//    the row kernels do (row.h): one wave per row.
//
// Measured, 128000 rows x 512, F 2048 (1000 tiles): 485 us a layer; the four
// launches 750.  Of a tile's 120 us about 58 are the 16 chunks (3.7 us each:
// 2 us of MFMAs at the clock they run at; removing GELU, or weights that hit
// the first-level cache, would save 0.25 us each) and 60 the O projection and
// the two ends, which move 1.1 MB a tile: 5 TB/s over the chip, the rate of a
// large copy.  128-row tiles at d 512 spill 29 to 42 registers (120 to 172 bytes
// a lane), all but one to three of the reloads outside the chunk loop; 64-row
// tiles none.  Tried and slower or no faster: the two waves of a SIMD half a
// chunk apart with three chunk buffers (3.6 us a chunk, d 256 15% slower), the
// O projection's residual read a pass ahead (more spills).  At d 256 four of
// the eight waves have no output columns in the O projection and the FFN down.
#include "gemm_tile.h"
#include "row.h"

namespace upr {

namespace mx_tail_detail {

using namespace gemm_detail;

enum { kEndLn = 0, kEndScore = 1, kEndPlain = 2 };

constexpr int kFC = 128;              // hidden columns per chunk
constexpr int kMaxF = 8192;           // b1 is staged in LDS
constexpr int kRing = 4;              // weight fragments in flight per wave
constexpr int kDown = 4;              // W2 fragments of a chunk: 2 k-steps x 2 column tiles
static_assert(kMxTailMaxF == kMaxF);

template <int TM, int KD>
struct Lds {
    static constexpr int kRows = 32 * TM;
    static constexpr int kA = 0;                               // [KD / 128][kRows][128] codes
    static constexpr int kH = kA + kRows * KD;                 // [2][kRows][128] codes
    static constexpr int kS = kH + 2 * kRows * kFC;            // [KD / 128][kRows] scale dwords
    static constexpr int kHS = kS + KD / 128 * kRows * 4;      // [2][kRows] scale dwords
    static constexpr int kLnx = kHS + 2 * kRows * 4;           // [2][32][8] (mean, M2)
    static constexpr int kPar = kLnx + 2 * 32 * 8 * 8;         // [3][KD]: bo, LN2 gain, LN2 shift
    static constexpr int kB1 = kPar + 3 * KD * 4;              // [kMaxF]
    static constexpr int kMain = kB1 + kMaxF * 4;
    // the end: [2][32] updated rows, padded by 16 bytes
    static constexpr int kEndLd = KD + 4, kEnd = 2 * 32 * kEndLd * 4;
    static constexpr int kBytes = kMain > kEnd ? kMain : kEnd;
};

// acc += W x A over one 64-deep fragment pair; ow / oa: the scale bytes.
__device__ __forceinline__ void mfma_mx(f32x16& acc, const i32x8& b, int ow, unsigned sw, const i32x8& a, int oa,
                                        unsigned sa) {
#define UPR_MX_CASE(OW, OA) \
    case 4 * OW + OA: \
        acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(b, a, acc, 0, 0, OW, (int)sw, OA, (int)sa); \
        break;
    switch (4 * ow + oa) {
        UPR_MX_CASE(0, 0)
        UPR_MX_CASE(0, 2)
        UPR_MX_CASE(1, 0)
        UPR_MX_CASE(1, 2)
        UPR_MX_CASE(2, 0)
        UPR_MX_CASE(2, 2)
        UPR_MX_CASE(3, 0)
        UPR_MX_CASE(3, 2)
    }
#undef UPR_MX_CASE
}

// Workgroup barrier after this wave's LDS accesses.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xC07F);         // lgkmcnt(0)
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The larger of v in lanes l and l ^ 32.
__device__ __forceinline__ float half_max(float v) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Sixteen values of a lane, columns 8q + 4 (l / 32) + r of a 32-column block
// whose other half lane l ^ 32 holds, as MXFP8: *e the block exponent, result
// the codes of columns 16 (l / 32) .. + 15.
__device__ __forceinline__ u32x4 encode_block(const float (&v)[16], int* e) {
    float amax = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) amax = fmaxf(amax, fabsf(v[r]));
    *e = mx_block_exp(half_max(amax));
    const float inv = mx_inv_scale(*e);
    unsigned u[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        u[q] = mx_pack4(v[4 * q] * inv, v[4 * q + 1] * inv, v[4 * q + 2] * inv, v[4 * q + 3] * inv);
    const auto r02 = __builtin_amdgcn_permlane32_swap(u[0], u[2], false, false);
    const auto r13 = __builtin_amdgcn_permlane32_swap(u[1], u[3], false, false);
    return u32x4{r02[0], r02[1], r13[0], r13[1]};
}

template <int END, int TM, int KD>
__global__ __launch_bounds__(512, 1) void k_mx_tail(MxTail t, int64_t M, int F) {
    using L = Lds<TM, KD>;
    constexpr int kRows = 32 * TM, kUT = TM / 2;       // up-phase row tiles per wave
    constexpr int kUp = KD / 64, kG = (kUp + 3) / 4;   // fragments of a row of W1 or Wo, their scale dwords
    constexpr int kKB = KD / 128;
    constexpr int kStep = 1024, kMajor = 32;           // residual: bytes between a lane's runs of four columns
    static_assert(kUp % kRing == 0 && kDown % kRing == 0, "ring slots repeat every phase");
    __shared__ __attribute__((aligned(16))) char smem[L::kBytes];
    char* const sA = smem + L::kA;
    char* const sH = smem + L::kH;
    uint32_t* const sS = reinterpret_cast<uint32_t*>(smem + L::kS);
    char* const sHS = smem + L::kHS;
    float2* const sX = reinterpret_cast<float2*>(smem + L::kLnx);
    float* const sPar = reinterpret_cast<float*>(smem + L::kPar);
    float* const sB1 = reinterpret_cast<float*>(smem + L::kB1);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 31, lhalf = lane >> 5, key = (lrow >> 1) & 7;
    const int64_t m0 = (int64_t)xcd_tile(blockIdx.x, gridDim.x) * kRows;
    const int rows = (int)(M - m0 < kRows ? M - m0 : kRows);
    const int nch = F / kFC;
    // up phase: row tiles kUT um .., hidden columns 32 un ..; O projection and
    // down phase: output columns 64 wave .. + 63 (waves past d have none, and
    // read weights of another's)
    const int um = wave >> 2, un = wave & 3;
    const bool dn_on = KD == 512 || wave < KD / 64;
    const int wdn = wave & (KD / 64 - 1);

    // ---- parameters and the tile's rows of o and their scales into LDS (rows
    // past M read as zeros: codes 0, scales 2^-127)
    for (int i = tid; i < F / 4; i += 512)
        reinterpret_cast<float4*>(sB1)[i] = reinterpret_cast<const float4*>(t.b1)[i];
    if (tid < KD) {
        sPar[tid] = t.bo[tid];
        sPar[KD + tid] = t.ln2_g[tid];
        sPar[2 * KD + tid] = t.ln2_b[tid];
    }
    {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(t.codes + m0 * KD, (short)0, rows * KD, 0x00020000);
        const __amdgpu_buffer_rsrc_t rss =
            __builtin_amdgcn_make_buffer_rsrc(t.scales + m0 * (KD / 32), (short)0, rows * (KD / 32), 0x00020000);
        const int r8 = lane >> 3, slot = lane & 7;
#pragma unroll
        for (int ins = 0; ins < kRows / 8 * kKB / 8; ++ins) {
            const int n = ins * 8 + wave, kb = n / (kRows / 8), blk = n % (kRows / 8);
            const int row = blk * 8 + r8;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs, (__attribute__((address_space(3))) void*)(sA + (kb * kRows + blk * 8) * 128), 16,
                row * KD + kb * 128 + ((slot ^ ((row >> 1) & 7)) << 4), 0, 0, 0);
        }
        constexpr int kS = kKB * (kRows / 64);      // 64 dwords each
        if (wave < kS)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rss, (__attribute__((address_space(3))) void*)(sS + wave * 64), 4,
                (wave % (kRows / 64) * 64 + lane) * (KD / 32) + wave / (kRows / 64) * 4, 0, 0, 0);
        static_assert(kS <= 8);
    }

    // ---- weights: fragment `f` of a matrix is 2 KB at 2048 f (the lanes'
    // first pieces, then their second), scale dword `f` of every lane 256
    // bytes at 256 f
    const int base1 = t.w1_off, base2 = t.w2_off;       // from wo (one descriptor: the choice between
    const __amdgpu_buffer_rsrc_t rsW = __builtin_amdgcn_make_buffer_rsrc(      // W1 and W2 stays a scalar select)
        const_cast<uint8_t*>(t.wo), (short)0, base2 + F * KD, 0x00020000);
    const int lane16 = lane * 16;
    auto load_frag = [&](int at) __attribute__((always_inline)) -> i32x8 {
        const i32x4 lo = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rsW, lane16, at, 0));
        const i32x4 hi =
            __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(rsW, lane16 + 1024, at, 0));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto at_o = [&](int s) __attribute__((always_inline)) { return ((2 * wdn + (s & 1)) * kUp + (s >> 1)) * 2048; };
    auto at_1 = [&](int c, int s) __attribute__((always_inline)) { return base1 + ((4 * c + un) * kUp + s) * 2048; };
    auto at_2 = [&](int c, int q) __attribute__((always_inline)) {
        return base2 + ((2 * wdn + (q & 1)) * (F / 64) + 2 * c + (q >> 1)) * 2048;
    };
    // step s < kRing of block c >= 1: chunk c's W1, or the last chunk's W2
    auto load_first = [&](int c, int s) __attribute__((always_inline)) -> i32x8 {
        return load_frag(c < nch ? at_1(c, s) : at_2(nch - 1, s));
    };
    constexpr int kOSteps = 2 * kUp;
    i32x8 ring[kRing];
#pragma unroll
    for (int s = 0; s < kRing; ++s) ring[s] = load_frag(at_o(s));
    unsigned wos[2][kG];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < kG; ++g) wos[j][g] = t.wo_s[((2 * wdn + j) * kG + g) * 64 + lane];
    unsigned w1s[kG], w1n[kG], w2s = 0;
#pragma unroll
    for (int g = 0; g < kG; ++g) w1s[g] = t.w1_s[(un * kG + g) * 64 + lane];

    f32x16 acc[kTN][TM];
    auto clear_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kTN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;
    };
    clear_acc();
    // The accumulators' values are wanted here: keeps the compiler from moving
    // a phase's MFMAs (and with them every operand) past its end.
    auto pin_acc = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kTN; ++j)
#pragma unroll
            for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(acc[j][i]));
    };

    // pieces 2m + lhalf of this lane's (swizzled) 128-byte row
    int choff[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) choff[m] = lrow * 128 + (((2 * m + lhalf) ^ key) << 4);
    // (derived addresses stay within a phase instead of living across chunks)
    auto fresh_offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < 4; ++m) asm volatile("" : "+v"(choff[m]));
    };
    // rows 32 i .. of a 128-byte K-block at `base`, 64-deep half kk
    auto read_frag = [&](const char* base, int i, int kk) __attribute__((always_inline)) -> i32x8 {
        const i32x4 lo = *reinterpret_cast<const i32x4*>(base + i * 4096 + choff[2 * kk]);
        const i32x4 hi = *reinterpret_cast<const i32x4*>(base + i * 4096 + choff[2 * kk + 1]);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    __builtin_amdgcn_s_waitcnt(0x0F70);         // vmcnt(0): the resident rows have landed
    lds_barrier();

    // ---- O projection: acc = o Wo^T; operand fragments roll through three
    // registers sets two tiles ahead of their MFMAs
    if (dn_on) {
        constexpr int kQ = kUp * TM;
        auto frag = [&](int q) __attribute__((always_inline)) -> i32x8 {
            return read_frag(sA + (q / TM >> 1) * kRows * 128, q % TM, q / TM & 1);
        };
        i32x8 of[3];
        unsigned os[TM];
        of[0] = frag(0);
        of[1] = frag(1);
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int kk = q / TM, i = q % TM;
            if (q % (2 * TM) == 0) {
#pragma unroll
                for (int k = 0; k < TM; ++k) os[k] = sS[(kk >> 1) * kRows + k * 32 + lrow] >> (8 * lhalf);
            }
            if (q + 2 < kQ) of[(q + 2) % 3] = frag(q + 2);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                mfma_mx(acc[j][i], ring[(2 * kk + j) % kRing], kk & 3, wos[j][kk >> 2], of[q % 3], 2 * (kk & 1), os[i]);
            __builtin_amdgcn_s_setprio(0);
            if (i == TM - 1) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int sn = 2 * kk + j + kRing;
                    ring[sn % kRing] = sn < kOSteps ? load_frag(at_o(sn)) : load_frag(at_1(0, sn - kOSteps));
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        pin_acc();
    } else {
#pragma unroll
        for (int s = 0; s < kRing; ++s) ring[s] = load_frag(at_1(0, s));
    }

    // ---- its epilogue, in the MFMA layout (lane (row 32i + l % 32, half h) of
    // wave w holds columns 64w + 32j + 8q + 4h + (0..3) in acc[j][i][4q ..]):
    // g = r + (acc + bo), LayerNorm statistics per 64-column block as the
    // GEMM's staged epilogue sums them (EPI_RESID_LN_MX: the same pairs), and
    // LN2 as MXFP8 over o's codes and scales.
    const bool whole = rows == kRows;
    const __amdgpu_buffer_rsrc_t rsG =
        __builtin_amdgcn_make_buffer_rsrc(t.g + m0 * KD, (short)0, rows * KD * 4, 0x00020000);
    // byte offset of this lane's run (i, j, q) of the residual: accumulator
    // order in whole tiles, else rows
    const int colw = 64 * wave + 4 * lhalf;
    const int g0 = whole ? wave * 8 * kStep + lane16 : (lrow * KD + colw) * 4;
    const int gq = whole ? kStep : kMajor;
    auto g_off = [&](int i, int j, int q) __attribute__((always_inline)) {
        return g0 + i * 32 * KD * 4 + (4 * j + q) * gq;
    };
    auto load_g = [&](int i, float4 (&dst)[kTN][4]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kTN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                dst[j][q] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsG, g_off(i, j, q), 0, 0));
    };
    {
        const __amdgpu_buffer_rsrc_t rsT = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned short*>(static_cast<const unsigned short*>(t.resid_src)) + m0 * KD, (short)0,
            rows * KD * 2, 0x00020000);
        auto load_r = [&](int i, float4 (&dst)[kTN][4]) __attribute__((always_inline)) {
            if (t.resid_src == nullptr) {
                load_g(i, dst);
                return;
            }
            typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
#pragma unroll
            for (int j = 0; j < kTN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const u32x2 w = __builtin_bit_cast(
                        u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                                   rsT, ((i * 32 + lrow) * KD + colw + 32 * j + 8 * q) * 2, 0, 0));
                    dst[j][q] = make_float4(__uint_as_float(w.x << 16), __uint_as_float(w.x & 0xffff0000u),
                                            __uint_as_float(w.y << 16), __uint_as_float(w.y & 0xffff0000u));
                }
        };
        float4 o[kTN][4];
        if (dn_on) load_r(0, o);
        lds_barrier();              // every wave has read its last fragment of o
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            float mrow = 0.f, qrow = 0.f;
            if (dn_on) {
                if (i > 0) load_r(i, o);
                // sum over the wave's columns of the row
                auto tree = [&](const float (&v)[kTN][4]) __attribute__((always_inline)) {
                    float u[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) u[q] = v[0][q] + v[1][q];
                    const float v0 = u[0] + u[2], v1 = u[1] + u[3];
                    const float w = v0 + v1;
                    return w + __shfl_xor(w, 32, 64);
                };
                float s[kTN][4];
#pragma unroll
                for (int j = 0; j < kTN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 r = o[j][q];
                        const float4 b = *reinterpret_cast<const float4*>(sPar + colw + 32 * j + 8 * q);
                        const f32x16& a = acc[j][i];
                        o[j][q] = make_float4(r.x + (a[4 * q + 0] + b.x), r.y + (a[4 * q + 1] + b.y),
                                              r.z + (a[4 * q + 2] + b.z), r.w + (a[4 * q + 3] + b.w));
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o[j][q]), rsG,
                                                               g_off(i, j, q), 0, 0);
                        s[j][q] = (o[j][q].x + o[j][q].y) + (o[j][q].z + o[j][q].w);
                    }
                mrow = tree(s) / 64.f;
#pragma unroll
                for (int j = 0; j < kTN; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float u0 = o[j][q].x - mrow, u1 = o[j][q].y - mrow, u2 = o[j][q].z - mrow,
                                    u3 = o[j][q].w - mrow;
                        s[j][q] = fmaf(u0, u0, fmaf(u1, u1, fmaf(u2, u2, u3 * u3)));
                    }
                qrow = tree(s);
            }
            float2* const X = sX + (i & 1) * (32 * 8);
            if (lhalf == 0) X[lrow * 8 + wave] = make_float2(mrow, qrow);
            lds_barrier();
            const float4* const xr = reinterpret_cast<const float4*>(X + lrow * 8);
            float mean_w[8], m2_w[8];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 v = xr[k];
                mean_w[2 * k] = v.x; m2_w[2 * k] = v.y; mean_w[2 * k + 1] = v.z; m2_w[2 * k + 1] = v.w;
            }
            float tot = 0.f, sum = 0.f;
#pragma unroll
            for (int w = 0; w < KD / 64; ++w) {
                tot += 64.f;
                sum = fmaf(64.f, mean_w[w], sum);
            }
            const float mu = sum / tot;
            float M2 = 0.f;
#pragma unroll
            for (int w = 0; w < KD / 64; ++w) {
                const float dm = mean_w[w] - mu;
                M2 += fmaf(64.f * dm, dm, m2_w[w]);
            }
            const float rstd = 1.0f / sqrtf(M2 / tot + t.ln_eps);
            if (dn_on) {
                char* const rowp = sA + ((wave >> 1) * kRows + i * 32 + lrow) * 128;
                unsigned sc2 = 0;
#pragma unroll
                for (int j = 0; j < kTN; ++j) {
                    float y[16];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int col = colw + 32 * j + 8 * q;
                        const float4 g = *reinterpret_cast<const float4*>(sPar + KD + col);
                        const float4 b = *reinterpret_cast<const float4*>(sPar + 2 * KD + col);
                        const float4 h = o[j][q];
                        y[4 * q + 0] = keep_f32(fmaf((h.x - mu) * rstd, g.x, b.x));
                        y[4 * q + 1] = keep_f32(fmaf((h.y - mu) * rstd, g.y, b.y));
                        y[4 * q + 2] = keep_f32(fmaf((h.z - mu) * rstd, g.z, b.z));
                        y[4 * q + 3] = keep_f32(fmaf((h.w - mu) * rstd, g.w, b.w));
                    }
                    int e;
                    const u32x4 codes = encode_block(y, &e);
                    sc2 |= (unsigned)(e + 127) << (8 * j);
                    *reinterpret_cast<u32x4*>(rowp + (((4 * (wave & 1) + 2 * j + lhalf) ^ key) << 4)) = codes;
                }
                if (lhalf == 0)
                    reinterpret_cast<unsigned short*>(sS + (wave >> 1) * kRows + i * 32 + lrow)[wave & 1] =
                        (unsigned short)sc2;
            }
        }
        clear_acc();
        lds_barrier();              // LN2 is in LDS
    }

    // ---- up phase of chunk c: h = a W1c^T, GELU, MXFP8 into chunk buffer c % 2;
    // refill(s) reloads the ring slot that step s used.  The scales of chunk
    // c + 1's W1 and of W2's chunk c - 1 are loaded meanwhile.
    auto up_phase = [&](int c, auto&& refill) __attribute__((always_inline)) {
        fresh_offsets();
        constexpr int kQ = kUp * kUT;
        f32x16 hacc[kUT];
        unsigned as[kUT][kKB];
#pragma unroll
        for (int i = 0; i < kUT; ++i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) hacc[i][r] = 0.f;
#pragma unroll
            for (int k = 0; k < kKB; ++k)
                as[i][k] = sS[k * kRows + (um * kUT + i) * 32 + lrow] >> (8 * lhalf);
        }
        const int cn = c + 1 < nch ? c + 1 : c;
#pragma unroll
        for (int g = 0; g < kG; ++g) w1n[g] = t.w1_s[((4 * cn + un) * kG + g) * 64 + lane];
        w2s = t.w2_s[(wdn * nch + (c > 0 ? c - 1 : 0)) * 64 + lane];
        auto frag = [&](int q) __attribute__((always_inline)) -> i32x8 {
            const int s = q / kUT;
            return read_frag(sA + (s >> 1) * kRows * 128, um * kUT + q % kUT, s & 1);
        };
        i32x8 af[3];
        af[0] = frag(0);
        af[1] = frag(1);
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int s = q / kUT, i = q % kUT;
            if (q + 2 < kQ) af[(q + 2) % 3] = frag(q + 2);
            __builtin_amdgcn_s_setprio(1);
            mfma_mx(hacc[i], ring[s % kRing], s & 3, w1s[s >> 2], af[q % 3], 2 * (s & 1), as[i][s >> 1]);
            __builtin_amdgcn_s_setprio(0);
            if (i == kUT - 1) refill(s);
            __builtin_amdgcn_sched_barrier(0);
        }
        mfma_settled<20>();         // (a refill's choice of address may be a branch)
#pragma unroll
        for (int i = 0; i < kUT; ++i) asm volatile("" : "+v"(hacc[i]));
        char* const hb = sH + (c & 1) * kRows * kFC;
        char* const hs = sHS + (c & 1) * kRows * 4;
        float4 bq[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            bq[q] = *reinterpret_cast<const float4*>(sB1 + c * kFC + 32 * un + 8 * q + 4 * lhalf);
#pragma unroll
        for (int i = 0; i < kUT; ++i) {
            float v[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                v[4 * q + 0] = gelu_fast(hacc[i][4 * q + 0] + bq[q].x);
                v[4 * q + 1] = gelu_fast(hacc[i][4 * q + 1] + bq[q].y);
                v[4 * q + 2] = gelu_fast(hacc[i][4 * q + 2] + bq[q].z);
                v[4 * q + 3] = gelu_fast(hacc[i][4 * q + 3] + bq[q].w);
            }
            int e;
            const u32x4 codes = encode_block(v, &e);
            const int row = (um * kUT + i) * 32 + lrow;
            *reinterpret_cast<u32x4*>(hb + row * 128 + (((2 * un + lhalf) ^ key) << 4)) = codes;
            if (lhalf == 0) hs[row * 4 + un] = (char)(e + 127);
        }
#pragma unroll
        for (int g = 0; g < kG; ++g) w1s[g] = w1n[g];
        __builtin_amdgcn_sched_barrier(0);
    };
    // ---- down phase of chunk c: acc += h W2c^T
    auto down_phase = [&](int c, auto&& refill) __attribute__((always_inline)) {
        if (!dn_on) {
#pragma unroll
            for (int s = 0; s < kDown; ++s) refill(s);
            return;
        }
        fresh_offsets();
        constexpr int kQ = 2 * TM;
        const char* const hb = sH + (c & 1) * kRows * kFC;
        const uint32_t* const hs = reinterpret_cast<const uint32_t*>(sHS + (c & 1) * kRows * 4);
        unsigned os[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) os[i] = hs[i * 32 + lrow] >> (8 * lhalf);
        i32x8 hf[3];
        hf[0] = read_frag(hb, 0, 0);
        hf[1] = read_frag(hb, 1, 0);
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int kk = q / TM, i = q % TM;
            if (q + 2 < kQ) hf[(q + 2) % 3] = read_frag(hb, (q + 2) % TM, (q + 2) / TM);
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int j = 0; j < 2; ++j)
                mfma_mx(acc[j][i], ring[2 * kk + j], 2 * j + kk, w2s, hf[q % 3], 2 * kk, os[i]);
            __builtin_amdgcn_s_setprio(0);
            if (i == TM - 1) {
                refill(2 * kk);
                refill(2 * kk + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        pin_acc();
    };
    // Block 0 is chunk 0's up phase, block c chunk c's up and chunk c - 1's down
    // phase, block nch the last down phase.  The barrier that ends a block
    // comes after every wave's writes of chunk buffer c % 2, read in the next
    // block, and after its reads of the other buffer, written in the next.
    up_phase(0, [&](int s) __attribute__((always_inline)) {
        ring[s % kRing] = s + kRing < kUp ? load_frag(at_1(0, s + kRing)) : load_first(1, s + kRing - kUp);
    });
    lds_barrier();
    for (int c = 1; c < nch; ++c) {
        up_phase(c, [&](int s) __attribute__((always_inline)) {
            ring[s % kRing] = s + kRing < kUp ? load_frag(at_1(c, s + kRing)) : load_frag(at_2(c - 1, s + kRing - kUp));
        });
        down_phase(c - 1, [&](int s) __attribute__((always_inline)) { ring[s] = load_first(c + 1, s); });
        lds_barrier();
    }
    w2s = t.w2_s[(wdn * nch + nch - 1) * 64 + lane];
    down_phase(nch - 1, [](int) __attribute__((always_inline)) {});

    // ---- the end: g += acc + b2, 32 rows at a time through LDS (over
    // everything before it), one wave per row as the row kernels.  Two staging
    // buffers: the barrier of pass i comes after every wave's reads of pass
    // i - 1, whose buffer pass i + 1 overwrites.
    float4 b2[kTN][4], r[2][kTN][4];
    if (dn_on) {
        load_g(0, r[0]);
#pragma unroll
        for (int j = 0; j < kTN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) b2[j][q] = *reinterpret_cast<const float4*>(t.b2 + colw + 32 * j + 8 * q);
    }
    lds_barrier();                  // the last down phase has read its chunk buffer
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        float* const st = reinterpret_cast<float*>(smem) + (i & 1) * 32 * L::kEndLd;
        if (dn_on) {
            if (i + 1 < TM) load_g(i + 1, r[(i + 1) & 1]);
#pragma unroll
            for (int j = 0; j < kTN; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 x = r[i & 1][j][q], b = b2[j][q];
                    const f32x16& a = acc[j][i];
                    const float4 o = make_float4(x.x + (a[4 * q + 0] + b.x), x.y + (a[4 * q + 1] + b.y),
                                                 x.z + (a[4 * q + 2] + b.z), x.w + (a[4 * q + 3] + b.w));
                    if constexpr (END == kEndLn)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rsG, g_off(i, j, q), 0, 0);
                    *reinterpret_cast<float4*>(st + lrow * L::kEndLd + colw + 32 * j + 8 * q) = o;
                }
        }
        lds_barrier();
        const int row = i * 32 + 4 * wave;      // of the wave's four rows, the first
        float v[4][row_detail::kMaxPerLane];
#pragma unroll
        for (int k = 0; k < 4; ++k) row_detail::load_row<true>(st + (4 * wave + k) * L::kEndLd, KD, lane, v[k]);
        if constexpr (END == kEndPlain) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (row + k < rows) {
#pragma unroll
                    for (int j = 0; j < KD / 256; ++j)
                        *reinterpret_cast<float4*>(t.g + (m0 + row + k) * KD + j * 256 + 4 * lane) =
                            make_float4(v[k][4 * j], v[k][4 * j + 1], v[k][4 * j + 2], v[k][4 * j + 3]);
                }
        } else {
            float mu[4], rstd[4];
            row_detail::row_stats(v, KD, t.ln_eps, mu, rstd);
            if constexpr (END == kEndLn) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    row_detail::store_normed_mx(t.codes + (m0 + row + k) * KD, t.scales + (m0 + row + k) * (KD / 32),
                                                v[k], KD, lane, mu[k], rstd[k], t.ln_g, t.ln_b, row + k < rows);
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float s =
                        row_detail::score_row<true>(v[k], KD, lane, mu[k], rstd[k], t.ln_g, t.ln_b, t.score_w);
                    if (lane == 0 && row + k < rows) t.scores[m0 + row + k] = s + t.score_b[0];
                }
            }
        }
    }
}

template <int TM, int KD>
hipError_t launch_end(const MxTail& t, int64_t M, int F, hipStream_t s) {
    const unsigned grid = (unsigned)((M + 32 * TM - 1) / (32 * TM));
    if (t.scores != nullptr)
        k_mx_tail<kEndScore, TM, KD><<<grid, 512, 0, s>>>(t, M, F);
    else if (t.ln_g != nullptr)
        k_mx_tail<kEndLn, TM, KD><<<grid, 512, 0, s>>>(t, M, F);
    else
        k_mx_tail<kEndPlain, TM, KD><<<grid, 512, 0, s>>>(t, M, F);
    return hipGetLastError();
}

}  // namespace mx_tail_detail

bool mx_tail_supported(int d, int F) {
    return (d == 256 || d == 512) && F > 0 && F % mx_tail_detail::kFC == 0 && F <= kMxTailMaxF;
}

// us per layer of a ranking call over a short history, separate launches /
// 64-row tiles:
//   d 256: F 256: 500 rows 35 / 30; F 1024: 1300 44 / 38; F 2048: 2000 50 / 51, 3000 55 / 53
//   d 512: F 512: 700 48 / 51, 1500 50 / 46; F 1024: 3000 58 / 61, 4500 64 / 59; F 2048: 5500 79 / 81, 7000 88 / 82;
//          F 4096: 6000 109 / 113, 7000 119 / 116
// A tile takes about the same time however few of them run, more with F:
// 64-row tiles from a number of rows per compute unit that grows with F, 25 at
// most; 128-row tiles once 64-row tiles would need a second round (F = 4d, tail
// alone, 64-row / 128-row: d 256, 20000 rows 62 / 56; d 512, 20000 123 / 108).
int mx_tail_tile(int64_t M, int d, int F) {
    const int64_t cus = gemm_detail::device_cus();
    if (M > 64 * cus) return 128;
    const int64_t from = d == 256 ? std::max(2 * cus, cus * F / 256) : std::max(4 * cus, std::min(25 * cus, cus * F / 72));
    return M > from ? 64 : 0;
}

hipError_t launch_mx_tail(int tile, const MxTail& t, int64_t M, int d, int F, hipStream_t s) {
    using namespace mx_tail_detail;
    if (M == 0) return hipSuccess;
    if ((tile != 64 && tile != 128) || !mx_tail_supported(d, F) || !t.wo || t.w1_off < d * d || t.w2_off < t.w1_off + F * d)
        return hipErrorInvalidValue;
    if (d == 512) return tile == 128 ? launch_end<4, 512>(t, M, F, s) : launch_end<2, 512>(t, M, F, s);
    return tile == 128 ? launch_end<4, 256>(t, M, F, s) : launch_end<2, 256>(t, M, F, s);
}

}  // namespace upr
