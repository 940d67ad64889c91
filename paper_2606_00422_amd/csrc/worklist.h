// The work list of the matrix-core attention kernels (device code,
// header-only): built by a launch of its own, or by one block of the first
// LayerNorm's launch.
#pragma once

#include "upr_plan.h"

namespace upr {

constexpr int kSortMax = 2048;

// Work list: users ordered by history length (longest first, ties by index)
// when there are at most MAXU users, else in index order.  Items of user
// u (rank r) occupy H * start_r .. H * (start_r + tiles_u) - 1, item
// H*(start_r + j) + h being tile j of head h (tile tiles_u - 1 - j when
// `reverse`: the causal pass puts a user's costliest, last tiles first), so
// with H = 8 all tiles of one (user, head) share blockIdx % 8 and therefore
// one XCD's L2.  Tiles cover the rows of `coffs` (candidates, or the history
// itself for the causal pass).  An item is (first history row of its user,
// history length, first query row, head | query count << 16).
//
// The offsets are read from device memory, which the caller promises holds
// the host values the call validated.  The kernel checks that promise
// before it writes an item: `coffs` non-decreasing from row_first to
// row_last, `hoffs` non-decreasing within [0, cap], and the tile count equal
// to the one sized on the host.  If any check fails, every item is written
// empty (no queries), so the attention launches touch nothing outside the
// call's buffers (the call's outputs are then meaningless, as the contract
// says for inconsistent offsets).
template <int NT, int MAXU>
__device__ __forceinline__ void build_worklist(const WorkList& wl) {
    const int32_t* const __restrict__ coffs = wl.row_offsets;
    const int32_t* const __restrict__ hoffs = wl.hist_offsets;
    const int U = wl.U, H = wl.H, tile = wl.tile, reverse = wl.reverse;
    int4* const __restrict__ work = reinterpret_cast<int4*>(wl.work);
    const int64_t items = wl.items, row_first = wl.row_first, row_last = wl.row_last, cap = wl.cap;
    constexpr int kWaves = NT / 64;
    __shared__ int s_len[MAXU];
    __shared__ int s_user[MAXU];      // user at each rank
    __shared__ int s_scan[NT];          // inclusive scan of tiles over the chunk's ranks
    __shared__ int4 s_seg[NT];          // per rank of the chunk: history start and length, candidate start and count
    __shared__ long long s_wtot[kWaves];
    __shared__ int s_wsum[kWaves];
    __shared__ long long s_carry;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    {
        bool bad = false;
        long long tiles = 0;
        for (int u = tid; u < U; u += NT) {
            const int64_t c0 = coffs[u], c1 = coffs[u + 1], h0 = hoffs[u], h1 = hoffs[u + 1];
            bad |= c1 < c0 || h0 < 0 || h1 < h0 || h1 > cap;
            if (c1 >= c0) tiles += (c1 - c0 + tile - 1) / tile;
        }
        if (tid == 0) bad |= coffs[0] != row_first || coffs[U] != row_last;
        // the tile total: wave sums, then thread 0 adds the waves'
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) tiles += __shfl_xor(tiles, off, 64);
        if (lane == 0) s_wtot[wv] = tiles;
        __syncthreads();
        if (tid == 0) {
            long long t = 0;
            for (int w = 0; w < kWaves; ++w) t += s_wtot[w];
            bad |= t > (1ll << 40) || t * H != items;
        }
        if (__syncthreads_or(bad)) {
            for (int64_t i = tid; i < items; i += NT) work[i] = make_int4(0, 0, 0, 0);
            return;
        }
    }
    const bool sorted = U <= MAXU;
    if (sorted) {
        for (int u = tid; u < U; u += NT) s_len[u] = hoffs[u + 1] - hoffs[u];
        __syncthreads();
        for (int u = tid; u < U; u += NT) {
            const int nu = s_len[u];
            int rank = 0;
            for (int v = 0; v < U; ++v) {
                const int nv = s_len[v];
                rank += (nv > nu) || (nv == nu && v < u);
            }
            s_user[rank] = u;
        }
        __syncthreads();
    }
    if (tid == 0) s_carry = 0;
    __syncthreads();
    // Chunks of NT ranks: each thread reads its rank's segments once, the
    // tile counts are scanned (within waves by shuffles, then across the
    // sixteen wave totals), and each thread writes the H items of its tiles,
    // finding a tile's rank by binary search on the scan.
    for (int base = 0; base < U; base += NT) {
        const int r = base + tid;
        int t = 0;
        int4 seg = make_int4(0, 0, 0, 0);
        if (r < U) {
            const int u = sorted ? s_user[r] : r;
            const int c0 = coffs[u], h0 = hoffs[u];
            seg = make_int4(h0, hoffs[u + 1] - h0, c0, coffs[u + 1] - c0);
            t = (seg.w + tile - 1) / tile;
        }
        s_seg[tid] = seg;
        int v = t;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(v, off, 64);
            if (lane >= off) v += y;
        }
        if (lane == 63) s_wsum[wv] = v;
        __syncthreads();
        for (int w = 0; w < wv; ++w) v += s_wsum[w];
        s_scan[tid] = v;
        __syncthreads();
        const int total = s_scan[NT - 1];                 // tiles of this chunk
        const int nr = min(NT, U - base);             // ranks of this chunk
        for (int x = tid; x < total; x += NT) {
            int lo = 0, hi = nr - 1;                    // smallest rank with s_scan > x
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (s_scan[mid] > x) hi = mid; else lo = mid + 1;
            }
            const int4 sg = s_seg[lo];
            const int tr = s_scan[lo] - (lo > 0 ? s_scan[lo - 1] : 0);
            const int j = x - (s_scan[lo] - tr);
            const int tt = reverse ? tr - 1 - j : j;
            const int cnt = min(tile, sg.w - tt * tile);
            const long long idx0 = (long long)H * (s_carry + x);
            for (int hh = 0; hh < H; ++hh)
                if (idx0 + hh < items) work[idx0 + hh] = make_int4(sg.x, sg.y, sg.z + tt * tile, hh | (cnt << 16));
        }
        __syncthreads();
        if (tid == 0) s_carry += total;
        __syncthreads();
    }
}

}  // namespace upr
