// Alg. 2, last steps (App. B.1): the chunks to attend to, as rows.  Block function: the tail of the selection's workgroup, or a launch
// of its own where the lists don't fit beside it.
#ifndef XKV_EXPAND_BLOCK_H
#define XKV_EXPAND_BLOCK_H

#include "xkv_common.h"

namespace xkv {

// Union of the k_ch selected chunks (sel, in LDS: ascending, no repeats) with the o static outliers of this (sequence, KV head)
// (ascending, no repeats), expanded to token rows in ascending order.  rows gets (k_ch + o) * c entries, of which the first
// counts[row] are real (only the context's last chunk can be short, and it can only be the last of the union); the rest is
// filled with row 0 and ignored by the attention kernel.  lds: expand_lds_words(k_ch, o) words.  All `threads` threads of the
// workgroup take part; sel may be written up to this call (it begins with a barrier).
inline size_t expand_lds_words(int k_ch, int o) { return (size_t)k_ch + 4 * (size_t)o + 1; }
__device__ __forceinline__ void expand_block(const int32_t *sel, int k_ch, const ExpandArgs &e, int row, int32_t *lds, int threads)
{
    const int o = e.o, c = e.c, n_c = e.n_c, cap = (k_ch + o) * c, tid = threadIdx.x;
    int32_t *ou_s = lds, *lb_s = ou_s + o, *dup_s = lb_s + o, *n_merged = dup_s + o, *merged = n_merged + 1;  // [k_ch + o]
    auto clampc = [&](int v) { return v < 0 ? 0 : (v >= n_c ? n_c - 1 : v); };
    for (int b = tid; b < o; b += threads) ou_s[b] = clampc(e.outliers[(size_t)row * o + b]);
    __syncthreads();
    // both lists are ascending without repeats: an element's place in the union is its own index plus the number of
    // elements of the other list in front of it (outliers that are also selected chunks are dropped)
    for (int b = tid; b < o; b += threads) {
        int lo = 0, hi = k_ch;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (sel[mid] < ou_s[b]) lo = mid + 1; else hi = mid;
        }
        lb_s[b] = lo;
        dup_s[b] = (lo < k_ch && sel[lo] == ou_s[b]) ? 1 : 0;
    }
    __syncthreads();
    for (int a = tid; a < k_ch; a += threads) {
        const int mine = sel[a];
        int before = 0;
        for (int b = 0; b < o; ++b) before += (!dup_s[b] && ou_s[b] < mine) ? 1 : 0;
        merged[a + before] = mine;
    }
    for (int b = tid; b < o; b += threads) {
        if (!dup_s[b]) {
            int before = 0;
            for (int b2 = 0; b2 < b; ++b2) before += dup_s[b2] ? 0 : 1;
            merged[lb_s[b] + before] = ou_s[b];
        }
    }
    if (tid == 0) {
        int n = k_ch;
        for (int b = 0; b < o; ++b) n += dup_s[b] ? 0 : 1;
        *n_merged = n;
    }
    __syncthreads();
    const int n = *n_merged;
    int total = n * c;
    if (n > 0 && merged[n - 1] == n_c - 1) total -= n_c * c - e.L;  // the short last chunk
    int32_t *out = e.rows + (size_t)row * cap;
    for (int i = tid; i < cap; i += threads) out[i] = i < total ? merged[i / c] * c + i % c : 0;
    if (tid == 0) e.counts[row] = total;
}

}  // namespace xkv
#endif
