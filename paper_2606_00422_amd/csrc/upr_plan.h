// Workspace plans of encode and rank, and the launchers they dispatch to.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "upr_internal.h"

namespace upr {

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// Query rows per work item of the MFMA attention (one workgroup handles this
// many history rows, in the causal encode pass, or candidates, in ranking,
// of one user for one head).
constexpr int kAttnTile = 128;
// (encode calls with few work items: a wave's walk over the keys is as long
// with 64-row items but carries half the queries)
constexpr int kSmallAttnTile = 64;
constexpr int64_t kSmallItems = 512;        // fewer 128-row items than this
constexpr int kRankAttnTile = 128;
constexpr int kSmallRankAttnTile = 64;      // ranking calls with few work items
constexpr int64_t kSmallRankItems = 512;    // fewer 128-candidate items than this
// Ranking calls whose candidates see long histories (on average at least
// kLongHistory rows each) take 256-candidate items, eight waves per
// workgroup: each K/V stage then serves twice the queries.
constexpr int kLongRankAttnTile = 256;
constexpr double kLongHistory = 4096.0;
constexpr int kF32AttnTile = 32;            // fp32 models, both passes

struct EncodePlan {
    int64_t row0 = 0, rows = 0;
    size_t off_g = 0, off_a = 0, off_q = 0, off_o = 0, off_h = 0, off_work = 0;
    int64_t work_items = 0;
    int attn_tile = kAttnTile;
    bool use_mfma_attn = false;
    size_t bytes = 0;
};

struct RankPlan {
    int64_t row0 = 0, rows = 0;
    size_t off_g = 0, off_a = 0, off_qkv = 0, off_o = 0, off_h = 0, off_work = 0;
    int64_t work_items = 0;
    int attn_tile = kRankAttnTile;
    bool use_mfma_attn = false;
    size_t bytes = 0;
};

inline bool bf16_storage(const upr_config& c) {
    return c.dtype == UPR_BF16 || c.dtype == UPR_BF16_MXFP8;
}
inline size_t dtype_bytes(const upr_config& c) { return bf16_storage(c) ? 2 : 4; }

// Number of MFMA attention work items over the rows of `offs`: one per
// (user, head, tile of up to `tile` rows).
inline int64_t attn_items(const upr_config& c, int U, const int32_t* offs, int tile) {
    int64_t items = 0;
    for (int u = 0; u < U; ++u) items += ((int64_t)offs[u + 1] - offs[u] + tile - 1) / tile;
    return items * c.n_heads;
}

// Whether the attention runs on the matrix cores, from a work list in the
// workspace.  bf16 models of head_dim 64 always do.  At head_dim 32, and for
// fp32 models, a one-wave-per-row kernel that needs no list stands in
//  * for histories whose keys pass the 2 GB a buffer descriptor spans here,
//  * for the fp8 variant's ranking pass (head_dim 32: the matrix-core kernel's
//    MXFP8 output covers whole 64-value heads), and
//  * where the list does not fit (`lists` false): a workspace that held these
//    calls before they had a list still does.  (bf16 encode at head_dim 64
//    then takes its larger items, whose list is half as long.)  `lists` is
//    also false for a cache off the 16-byte boundaries of the kernels' loads.
inline bool use_mfma_attn(const upr_config& c, bool rank, int U, const int32_t* hoffs, bool lists) {
    if (bf16_storage(c) && c.head_dim == 64) return true;
    if (!lists || (rank && c.dtype == UPR_BF16_MXFP8)) return false;
    const int64_t most = (int64_t{1} << 31) / (c.head_dim * (int64_t)dtype_bytes(c));
    for (int u = 0; u < U; ++u)
        if ((int64_t)hoffs[u + 1] - hoffs[u] >= most) return false;
    return true;
}

// Workspace of encode for the history rows of `hoffs` (host offsets): fp32
// residual stream, then LayerNorm output, queries, attention output and FFN
// hidden (model dtype), and the attention work list.
inline EncodePlan plan_encode(const upr_config& c, int U, const int32_t* hoffs, bool lists = true) {
    EncodePlan p;
    p.row0 = hoffs[0];
    p.rows = (int64_t)hoffs[U] - hoffs[0];
    if (p.rows <= 0) { p.rows = 0; return p; }
    const size_t es = dtype_bytes(c), R = (size_t)p.rows, d = c.d_model, F = c.d_ff;
    p.use_mfma_attn = use_mfma_attn(c, false, U, hoffs, lists);
    if (!bf16_storage(c))
        p.attn_tile = kF32AttnTile;
    else if (lists && attn_items(c, U, hoffs, kAttnTile) < kSmallItems)
        p.attn_tile = kSmallAttnTile;
    if (p.use_mfma_attn) p.work_items = attn_items(c, U, hoffs, p.attn_tile);
    size_t o = 0;
    p.off_g = o; o = align256(o + R * d * 4);
    p.off_a = o; o = align256(o + R * d * es);
    p.off_q = o; o = align256(o + R * d * es);
    p.off_o = o; o = align256(o + R * d * es);
    p.off_h = o; o = align256(o + R * F * es);
    p.off_work = o; o = align256(o + (size_t)p.work_items * 4 * sizeof(int32_t));
    p.bytes = o;
    return p;
}

// Workspace of rank for the candidate rows of `coffs` (host offsets):
// residual, LayerNorm output, fused q|k|v rows, attention output, FFN hidden
// (at least head_cols wide: the action heads' hidden layer reuses it), and
// the attention work list.  The fp8-projection variant keeps
// MXFP8 encodings in the LayerNorm-output and FFN-hidden buffers (codes,
// then scales at the next 256-byte boundary: rows x cols x 2 bytes hold
// both for rows x cols >= 256).
inline RankPlan plan_rank(const upr_config& c, int U, const int32_t* coffs, const int32_t* hoffs,
                          int head_cols = 0, bool lists = true) {
    RankPlan p;
    p.row0 = coffs[0];
    p.rows = (int64_t)coffs[U] - coffs[0];
    if (p.rows <= 0) { p.rows = 0; return p; }
    const size_t es = dtype_bytes(c), R = (size_t)p.rows, d = c.d_model, F = c.d_ff;
    p.use_mfma_attn = use_mfma_attn(c, true, U, hoffs, lists);
    if (p.use_mfma_attn && !bf16_storage(c)) {
        p.attn_tile = kF32AttnTile;
        p.work_items = attn_items(c, U, coffs, p.attn_tile);
    } else if (p.use_mfma_attn) {
        double seen = 0.0;                  // history rows seen, summed over candidates
        for (int u = 0; u < U; ++u)
            seen += (double)((int64_t)coffs[u + 1] - coffs[u]) * (double)((int64_t)hoffs[u + 1] - hoffs[u]);
        const int64_t long_items = attn_items(c, U, coffs, kLongRankAttnTile);
        if (seen >= kLongHistory * (double)p.rows && long_items >= kSmallRankItems) {
            p.attn_tile = kLongRankAttnTile;
            p.work_items = long_items;
        } else {
            p.work_items = attn_items(c, U, coffs, p.attn_tile);
            if (p.work_items < kSmallRankItems) {
                p.attn_tile = kSmallRankAttnTile;
                p.work_items = attn_items(c, U, coffs, p.attn_tile);
            }
        }
    }
    size_t o = 0;
    p.off_g = o; o = align256(o + R * d * 4);
    p.off_a = o; o = align256(o + R * d * es);
    p.off_qkv = o; o = align256(o + R * 3 * d * es);
    // (the fp8 variant's fallback attention, head_dim 32, writes fp32 here
    // before the MXFP8 encoder reads it)
    const size_t o_es = c.dtype == UPR_BF16_MXFP8 ? 4 : es;
    p.off_o = o; o = align256(o + R * d * o_es);
    p.off_h = o; o = align256(o + R * std::max<size_t>(F, (size_t)head_cols) * es);
    p.off_work = o; o = align256(o + (size_t)p.work_items * 4 * sizeof(int32_t));
    p.bytes = o;
    return p;
}

// Projection GEMM, out = A[M,K] W[N,K]^T + epilogue, on the tile that fills
// the device best: fp32 operands (fp32 models) or fp16 (bf16 models).
template <typename TA, typename TKV>
hipError_t launch_gemm(const TA* A, int64_t lda, const TA* W, int64_t M, int N, int K,
                       const Epilogue& epi, hipStream_t s);

// fp16 MFMA GEMM (K a multiple of 64, lda a multiple of 8) on 256-column
// tiles of 64 tm rows (tm = 1 to 4), or for the whole-row modes (tm = 0) on
// tiles of 128 or 32 rows.  (The MXFP8
// GEMM, launch_gemm_mx, is declared with the other launchers.)
hipError_t launch_gemm_mfma(int tm, const f16* A, int64_t lda, const f16* W, int64_t M, int N, int K,
                            const Epilogue& epi, hipStream_t s);

// Whether a residual update of M rows, [M, K] x [N, K]^T, is followed by a
// launch_block_layernorm instead of an EPI_RESID_LN / EPI_RESID_SCORE epilogue
// (same bits either way).
bool separate_layernorm(int64_t M, int N, int K);

// The same product on block x block tiles (k_gemm_small.hip; 64 for fp16, 32
// or 128 for fp32), modes EPI_STORE, EPI_GELU, EPI_GELU_PERM (fp16), EPI_RESID
// (acc_resid allowed) and EPI_QKV_CACHE.  A and W fp16 (K a multiple of 64) or
// fp32 (of 32).
template <typename TA, typename TKV>
hipError_t launch_gemm_small(const TA* A, int64_t lda, const TA* W, int64_t M, int N, int K,
                             const Epilogue& epi, int block, hipStream_t s);

// Fused layer tail (k_ffn_fused.hip) on the fp32 residual g:
//   g += O Wo^T + bo;  a = LN2(g);  g += gelu(a W1^T + b1) W2^T + b2
// then the LayerNorm (epi.mode EPI_RESID_LN) or the score head
// (EPI_RESID_SCORE).  O [M, d] fp16 attention output rows (leading dimension
// d); epa: the O projection's EPI_RESID_LN epilogue (Wo's scale, bo, LN2,
// the same residual; resid_src in the first layer), epi: the FFN down's
// (W2's scale, b2, the following LayerNorm or score head).  WoP [d, d],
// W1p [F, d] and W2p [d, F] in the fragment-major layout the model image
// builds; s1 = W1's scale.
bool ffn_fused_supported(int d, int F);
// Rows of the fused kernel's tiles in a call of M rows: 128, 64, or 0 when
// the call runs the unfused sequence on small tiles, which is faster for few
// rows.  The results are the same bits (same products in the same order).
int ffn_fused_tile(int64_t M, int d, int F);
hipError_t launch_ffn_fused(int tile, const f16* O, const f16* WoP, const Epilogue& epa, const f16* W1p,
                            const f16* W2p, const float* b1, float s1, int64_t M, int d, int F,
                            const Epilogue& epi, hipStream_t s);

// Fused layer tail of the MXFP8 variant (k_mx_tail.hip): the O projection of
// codes / scales ([M, d], [M, d / 32]), LN2, FFN, both residual updates, then
// LN of the updated rows over codes / scales (ln_g set), the score head (with
// ln_g, ln_b and `scores`) or neither.  wo, w1, w2 and their scale dwords in
// the fragment order the model image builds.  The residual g goes from one
// tail of a call to the next (same tile) in the tail's own order within the
// rows of a whole tile; a tail without ln_g and scores leaves it in rows.
struct MxTail {
    uint8_t* codes;
    uint8_t* scales;
    float* g;
    const void* resid_src;      // set: the first residual comes from these bf16 rows
    const uint8_t* wo;
    int w1_off, w2_off;         // bytes from wo to W1's and W2's fragments
    const uint32_t *wo_s, *w1_s, *w2_s;
    const float *bo, *ln2_g, *ln2_b, *b1, *b2;
    const float *ln_g, *ln_b;
    float ln_eps;
    const float *score_w, *score_b;
    float* scores;
};
constexpr int kMxTailMaxF = 8192;
bool mx_tail_supported(int d, int F);
// Rows of its tiles in a call of M rows: 128, 64, or 0 when the separate
// launches are faster.  The results are the same bits.
int mx_tail_tile(int64_t M, int d, int F);
hipError_t launch_mx_tail(int tile, const MxTail& t, int64_t M, int d, int F, hipStream_t s);

// Builds the list of `wl` (upr_internal.h) in a launch of its own.
hipError_t launch_attn_worklist(const WorkList& wl, hipStream_t s);

// MFMA ranking attention (bf16 q|k|v rows and cache, head_dim 64 or 32), fp16 output.
hipError_t launch_attn_rank(const bf16* qkv, f16* o, int64_t row0, int H, int D,
                            const int32_t* work, int64_t items,
                            int tile, const bf16* cache_k, const bf16* cache_v, int64_t cache_cap,
                            hipStream_t s);

// The same with the output as MXFP8 (codes [rows, H*64], one E8M0 scale byte
// per 32-value block [rows, H*2]), encoded from the normalised fp32 values:
// the fp8 projection variant's input of the O projection.
hipError_t launch_attn_rank_mx(const bf16* qkv, uint8_t* codes, uint8_t* scales, int64_t row0,
                               int H, int D, const int32_t* work,
                               int64_t items, int tile, const bf16* cache_k, const bf16* cache_v,
                               int64_t cache_cap, hipStream_t s);

// MFMA attention of fp32 models, ranking (q: q|k|v rows) or causal encode (q:
// query rows), fp32 output; the work list has kF32AttnTile-row items.
hipError_t launch_attn_f32(bool causal, const float* q, float* o, int64_t row0, int H, int D, const int32_t* work,
                           int64_t items, const float* cache_k, const float* cache_v, int64_t cache_cap,
                           hipStream_t s);

// MFMA causal encode attention (bf16 query rows and cache, head_dim 64 or 32),
// fp16 output.
hipError_t launch_attn_encode(const bf16* q, f16* o, int64_t row0, int H, int D,
                              const int32_t* work, int64_t items,
                              int tile, const bf16* cache_k, const bf16* cache_v,
                              int64_t cache_cap, hipStream_t s);

// Host MXFP8 encoding of x [rows, k] (k a multiple of 32): the weights of
// the fp8-projection variant, and upr_mx_quantize_host.
void mx_quantize_host(const float* x, int64_t rows, int k, uint8_t* codes, uint8_t* scales);

// Per-action heads: at most kMaxActions heads; utility weights by value.
constexpr int kMaxActions = 8;
struct HeadUtility {
    float u[kMaxActions];
};

// logit_c = w2_c . hid[:, c*Fh .. c*Fh+Fh) + b2_c, probs[r, c] = sigmoid(logit_c)
// (if probs), util[r] = sum_c u_c probs[r, c] (if util); hid rows of ldh
// elements, Fh a multiple of 8.
template <typename TA>
hipError_t launch_heads_out(const TA* hid, int64_t ldh, int64_t rows, int C, int Fh,
                            const float* w2, const float* b2, const HeadUtility& uw, float* probs,
                            float* util, hipStream_t s);

// Per-user top K by utility (one workgroup per user, at most
// kTopkMaxCandidates candidates per user: the caller checks).  A user whose
// device offsets leave [row_first, row_last] or that limit gets no entries.
constexpr int kTopkMaxCandidates = 16384;
hipError_t launch_topk(const float* util, const int32_t* coffs_dev, int U, int K,
                       int32_t* out_rows, float* out_util, int64_t row_first, int64_t row_last,
                       hipStream_t s);

}  // namespace upr
