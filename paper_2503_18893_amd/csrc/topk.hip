// Per-row ArgTopK by radix select on the monotone 32-bit image of the fp32 scores
// (App. B.1 Alg. 2, top-k step, applied per token).  Bit-exact and deterministic.
//
// A row of L scores is split into chunks; one workgroup owns one (row, chunk).  Four passes resolve the
// 32-bit key of the k-th largest element 8 bits at a time.  A pass histograms, per chunk, the current
// digit of the keys that still match the resolved prefix, keeps the chunk's histogram and adds it to the
// row's histogram with integer atomics (order-independent, so the result is deterministic).  Launch
// boundaries are the only synchronisation: every workgroup of the next launch reads the row histogram
// (1 KiB), finds the bin holding the k-th element, refines the prefix, and counts from its own chunk's
// stored histogram how many of its keys are thereby known to lie above the threshold.  The last launch
// knows the threshold key T and how many keys equal to T are still needed (ties go to the smaller token
// id), sums the counts of the chunks before its own and writes the selected ids in ascending order with
// wavefront ballots.
#include <cmath>
#include <type_traits>

#include "xkv_common.h"
#include "expand_block.h"
#include "row_select.h"

namespace xkv {

// scratch arrays (uint32 words), carved by launch_topk
struct TopkScratch {
    uint32_t *hist;      // [rows][chunks][4][256] per-chunk digit histograms (level 3: suffix sums)
    uint32_t *state;     // [rows][8]  (prefix, k_rem) after each level
    uint32_t *row_hist;  // [rows][4][256] per-row digit histograms (zeroed by topk_init_kernel)
    uint32_t *chunk_gt;  // [rows][chunks] keys of the chunk above the threshold by levels 0..2
};

__global__ void topk_init_kernel(uint32_t *row_hist, int words)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;  // every level of every row
    if (i < words) row_hist[i] = 0;
}

// Inclusive suffix sum over the 256 bins held one per thread.  All 256 threads take part.
__device__ __forceinline__ uint32_t suffix_sum_256(uint32_t c, uint32_t *sh /* >= 4 words */)
{
    const int lane = lane_id(), w = wave_id();
    uint32_t s = c;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t nb = __shfl_down(s, off, kWave);
        if (lane + off < kWave) s += nb;
    }
    __syncthreads();  // sh may still be read by a previous use
    if (lane == 0) sh[w] = s;
    __syncthreads();
    for (int ww = w + 1; ww < 4; ++ww) s += sh[ww];
    return s;
}

// From the row histogram of `level`: the bin b with (#keys in bins above b) < k_rem <= (#keys in bins >= b).
__device__ __forceinline__ void resolve_level(const uint32_t *__restrict__ row_hist_level, uint32_t k_rem,
                                              uint32_t *sh /* >= 8 words */, uint32_t &digit, uint32_t &k_rem_out)
{
    const uint32_t c = row_hist_level[threadIdx.x];
    const uint32_t incl = suffix_sum_256(c, sh), above = incl - c;
    if (above < k_rem && k_rem <= incl) {
        sh[4] = threadIdx.x;
        sh[5] = k_rem - above;
    }
    __syncthreads();
    digit = sh[4];
    k_rem_out = sh[5];
}

template <int LEVEL>
__global__ __launch_bounds__(256) void topk_hist_kernel(const float *__restrict__ S, TopkScratch ws, int L, int k,
                                                        int chunks, int chunk)
{
    __shared__ uint32_t sh_hist[kTopkBins];
    __shared__ uint32_t sh_misc[8];
    const int row = blockIdx.y, c = blockIdx.x;
    uint32_t *row_hist = ws.row_hist + (size_t)row * kTopkLevels * kTopkBins;
    uint32_t *my_hist = ws.hist + ((size_t)row * chunks + c) * kTopkLevels * kTopkBins;
    uint32_t prefix = 0, k_rem = (uint32_t)k;
    if constexpr (LEVEL > 0) {
        if constexpr (LEVEL > 1) {
            prefix = ws.state[(size_t)row * kStateWords + 2 * (LEVEL - 2)];
            k_rem = ws.state[(size_t)row * kStateWords + 2 * (LEVEL - 2) + 1];
        }
        uint32_t digit, k_new;
        resolve_level(row_hist + (LEVEL - 1) * kTopkBins, k_rem, sh_misc, digit, k_new);
        prefix = (prefix << 8) | digit;
        k_rem = k_new;
        if (c == 0 && threadIdx.x == 0) {
            ws.state[(size_t)row * kStateWords + 2 * (LEVEL - 1)] = prefix;
            ws.state[(size_t)row * kStateWords + 2 * (LEVEL - 1) + 1] = k_rem;
        }
        // keys of this chunk that matched the old prefix and have a larger digit lie above the threshold
        const uint32_t mine = my_hist[(LEVEL - 1) * kTopkBins + threadIdx.x];
        const uint32_t incl = suffix_sum_256(threadIdx.x > digit ? mine : 0u, sh_misc);
        if (threadIdx.x == 0) {
            uint32_t *cg = ws.chunk_gt + (size_t)row * chunks + c;
            *cg = (LEVEL == 1 ? 0u : *cg) + incl;
        }
    }
    sh_hist[threadIdx.x] = 0;
    __syncthreads();
    const float *Srow = S + (size_t)row * L;
    const int lane = lane_id();
    const int base = c * chunk;
    for (int i0 = 0; i0 < chunk; i0 += 1024) {  // chunk is a multiple of 256: every trip count is uniform
        float val[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // four independent coalesced loads in flight
            const int t = base + i0 + u * 256 + (int)threadIdx.x;
            val[u] = (i0 + u * 256 < chunk && t < L) ? Srow[t] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (i0 + u * 256 >= chunk) break;
            const int t = base + i0 + u * 256 + (int)threadIdx.x;
            const uint32_t key = order_key(val[u]);
            bool active = t < L;
            if constexpr (LEVEL > 0) active = active && ((key >> (32 - 8 * LEVEL)) == prefix);
            const uint32_t digit = (key >> (24 - 8 * LEVEL)) & 0xFFu;
            // scores cluster in few bins at the top levels: add the leader's bin once per wavefront
            const uint64_t m = __ballot(active);
            if (m != 0) {
                const int first = __ffsll((unsigned long long)m) - 1;
                const uint32_t d0 = __shfl(digit, first, kWave);
                const uint64_t same = __ballot(active && digit == d0);
                if (lane == first) atomicAdd(&sh_hist[d0], (uint32_t)__popcll(same));
                if (active && digit != d0) atomicAdd(&sh_hist[digit], 1u);
            }
        }
    }
    __syncthreads();
    const uint32_t cnt = sh_hist[threadIdx.x];
    if (cnt != 0) atomicAdd(&row_hist[LEVEL * kTopkBins + threadIdx.x], cnt);
    if constexpr (LEVEL < 3) {
        my_hist[LEVEL * kTopkBins + threadIdx.x] = cnt;
    } else {
        // last level: keep the suffix sums, so that "keys above digit d" is one load for the writer
        my_hist[LEVEL * kTopkBins + threadIdx.x] = suffix_sum_256(cnt, sh_misc);
    }
}

__global__ __launch_bounds__(256) void topk_write_kernel(const float *__restrict__ S, TopkScratch ws,
                                                         int32_t *__restrict__ idx_out, int L, int k, int chunks,
                                                         int chunk)
{
    __shared__ uint32_t sh_misc[8];
    __shared__ uint32_t sh_red[2][4];
    __shared__ uint32_t sh_cnt[2][4];
    const int row = blockIdx.y, c = blockIdx.x;
    const uint32_t *row_hist = ws.row_hist + (size_t)row * kTopkLevels * kTopkBins;
    const uint32_t *hist_row = ws.hist + (size_t)row * chunks * kTopkLevels * kTopkBins;
    const uint32_t prefix = ws.state[(size_t)row * kStateWords + 4];
    const uint32_t k_rem = ws.state[(size_t)row * kStateWords + 5];
    uint32_t digit, need_eq;
    resolve_level(row_hist + 3 * kTopkBins, k_rem, sh_misc, digit, need_eq);
    const uint32_t T = (prefix << 8) | digit;  // key of the k-th largest element

    // selected keys of the chunks before this one: above T (levels 0..2 counted earlier, level 3 from the
    // stored suffix sums) and equal to T
    const int lane = lane_id(), w = wave_id();
    uint32_t gt = 0, eq = 0;
    for (int ch = threadIdx.x; ch < c; ch += 256) {
        const uint32_t *h3 = hist_row + ((size_t)ch * kTopkLevels + 3) * kTopkBins;
        const uint32_t ge = h3[digit], above = digit < 255u ? h3[digit + 1] : 0u;
        gt += ws.chunk_gt[(size_t)row * chunks + ch] + above;
        eq += ge - above;
    }
    for (int off = 32; off > 0; off >>= 1) {
        gt += __shfl_xor(gt, off, kWave);
        eq += __shfl_xor(eq, off, kWave);
    }
    if (lane == 0) {
        sh_red[0][w] = gt;
        sh_red[1][w] = eq;
    }
    __syncthreads();
    const uint32_t gt_before = sh_red[0][0] + sh_red[0][1] + sh_red[0][2] + sh_red[0][3];
    const uint32_t eq_before = sh_red[1][0] + sh_red[1][1] + sh_red[1][2] + sh_red[1][3];

    // each wavefront owns a contiguous quarter of the chunk; first count, then write in order
    const float *Srow = S + (size_t)row * L;
    const int sub = chunk / 4;
    const int begin = c * chunk + w * sub;
    uint32_t my_gt = 0, my_eq = 0;
    for (int i0 = 0; i0 < sub; i0 += 4 * kWave) {  // sub is a multiple of 64
        float val[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = begin + i0 + u * kWave + lane;
            val[u] = (i0 + u * kWave < sub && t < L) ? Srow[t] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = begin + i0 + u * kWave + lane;
            const bool in = i0 + u * kWave < sub && t < L;
            const uint32_t key = order_key(val[u]);
            my_gt += (uint32_t)__popcll(__ballot(in && key > T));
            my_eq += (uint32_t)__popcll(__ballot(in && key == T));
        }
    }
    if (lane == 0) {
        sh_cnt[0][w] = my_gt;
        sh_cnt[1][w] = my_eq;
    }
    __syncthreads();
    uint32_t gt_run = gt_before, eq_run = eq_before;
    for (int ww = 0; ww < w; ++ww) {
        gt_run += sh_cnt[0][ww];
        eq_run += sh_cnt[1][ww];
    }
    int32_t *out = idx_out + (size_t)row * k;
    for (int i0 = 0; i0 < sub; i0 += 4 * kWave) {
        float val[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = begin + i0 + u * kWave + lane;
            val[u] = (i0 + u * kWave < sub && t < L) ? Srow[t] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = begin + i0 + u * kWave + lane;
            const bool in = i0 + u * kWave < sub && t < L;
            const uint32_t key = order_key(val[u]);
            const bool is_gt = in && key > T, is_eq = in && key == T;
            const uint64_t mg = __ballot(is_gt), me = __ballot(is_eq);
            const uint32_t gt_me = gt_run + lanes_below(mg), eq_me = eq_run + lanes_below(me);
            if (is_gt || (is_eq && eq_me < need_eq)) {
                const uint32_t pos = gt_me + (eq_me < need_eq ? eq_me : need_eq);
                if (pos < (uint32_t)k) out[pos] = t;
            }
            gt_run += (uint32_t)__popcll(mg);
            eq_run += (uint32_t)__popcll(me);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Rows of up to 65536 scores: the whole selection in one launch.  One workgroup of 16 wavefronts owns a row
// and keeps its keys in registers (NV per thread; wavefront w holds the contiguous segment
// [w 64 NV, (w+1) 64 NV), element j of a lane is w 64 NV + 64 j + lane), so the row is read from memory once
// and nothing but the ids is written.  The four 8-bit radix passes histogram into LDS counters that are
// replicated per lane pair ([bin][lane/2], two 16-bit halves per word: a lane position sees at most
// 16 NV <= 1024 keys), so the clustered top digits cost no serialised atomics; the replicas are summed, the
// first wavefront finds the bin of the k-th key, and the pass repeats on the next digit.  The ordered write
// counts the keys to take with ballots, from the registers: where all keys equal to the threshold are taken and the ids fit,
// they are collected in LDS and leave as whole lines; otherwise as in topk_write_kernel, stored one by one.  expand.rows: the ids
// are chunks and go on to the rows that they stand for (expand_block.h; a launch of its own took 5 to 7 us).
// ------------------------------------------------------------------------------------------
constexpr int kRowStage = 16384;  // most ids staged in LDS

template <int NV, bool EXPAND>
__global__ __launch_bounds__(kRowThreads) void topk_row_kernel(const float *__restrict__ S, int32_t *__restrict__ idx_out, int L, int k,
                                                               ExpandArgs expand)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t hist[];  // [kTopkBins * 32]; at the end the ids, where they fit
    __shared__ uint32_t bins[kTopkBins];
    __shared__ uint32_t sh[3 + 2 * kRowWaves];
    const int row = blockIdx.x, tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const float *Srow = S + (size_t)row * L;
    const int base = w * 64 * NV + lane;

    uint32_t key[NV];
    const bool whole = (w + 1) * 64 * NV <= L;  // this wavefront's segment lies within the row
    if (whole) {  // (one lane offset for all loads: the clamped form below spends four vector instructions on each)
        const float *Sw = Srow + w * 64 * NV;
#pragma unroll
        for (int j = 0; j < NV; ++j) key[j] = __float_as_uint(Sw[64 * j + lane]);
    } else {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int t = base + 64 * j;
            key[j] = __float_as_uint(Srow[t < L ? t : L - 1]);
            if (j % 8 == 7) __builtin_amdgcn_sched_barrier(0);  // bounds the address registers alive at once
        }
    }
    // Positions beyond the row get key 0, below every real key (those are clamped to >= 1; only one NaN pattern
    // maps to 0): they can then be histogrammed and compared like the rest and are never selected, k <= L.
    // (Each phase recomputes its positions from an opaque copy of `base`; otherwise the compiler keeps all NV of
    // them in registers from the loads to the final write.)
    int base_v = base;
    asm volatile("" : "+v"(base_v));
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const uint32_t kk = order_key(__uint_as_float(key[j]));
        key[j] = kk > 1u ? kk : 1u;
    }
    if (!whole) {
#pragma unroll
        for (int j = 0; j < NV; ++j) key[j] = base_v + 64 * j < L ? key[j] : 0u;
    }

    // Levels 0..2 histogram into `hist`.  While many keys still match the prefix the counters are replicated per
    // lane pair ([bin][lane/2], two 16-bit halves per word); once at most 4096 match (known exactly from the
    // previous level's bin count) a plain 256-word histogram is cheaper to clear and to sum.  Level 3 histograms
    // per wavefront ([wavefront][bin]), so that each wavefront can read off afterwards how many of its own keys
    // lie above / at the threshold without another pass over its registers.
    uint32_t prefix = 0, k_rem = (uint32_t)k, n_match = (uint32_t)L;
    uint32_t above24 = 0;  // level 3: keys of this wavefront whose upper 24 bits are already above the prefix
#pragma unroll
    for (int level = 0; level < kTopkLevels; ++level) {
        const bool per_wave = level == 3;
        const bool direct = !per_wave && level > 0 && n_match <= 4096u;  // uniform over the workgroup
        if (per_wave) {
            for (int i = tid; i < kRowWaves * kTopkBins; i += kRowThreads) hist[i] = 0;
        } else if (direct) {
            if (tid < kTopkBins) hist[tid] = 0;
        } else {
            for (int i = tid; i < kTopkBins * 32; i += kRowThreads) hist[i] = 0;
        }
        __syncthreads();
        const uint32_t inc = (per_wave || direct) ? 1u : 1u << (16 * (lane & 1));
        const uint32_t slot0 = per_wave ? (uint32_t)w * kTopkBins : direct ? 0u : (uint32_t)(lane >> 1);
        const uint32_t dmul = (per_wave || direct) ? 1u : 32u;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const uint32_t upper = level == 0 ? 0u : key[j] >> (32 - 8 * level);
            const bool match = level == 0 || upper == prefix;
            const uint32_t digit = (key[j] >> (24 - 8 * level)) & 0xFFu;
            if (match) atomicAdd(&hist[digit * dmul + slot0], inc);
            if (level == 3) {
                above24 += (uint32_t)__popcll(__ballot(upper > prefix));
                asm volatile("" : "+s"(above24));
            }
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        if (per_wave) {
            if (tid < kTopkBins) {
                uint32_t sum = 0;
#pragma unroll
                for (int ww = 0; ww < kRowWaves; ++ww) sum += hist[ww * kTopkBins + tid];
                bins[tid] = sum;
            }
        } else if (direct) {
            if (tid < kTopkBins) bins[tid] = hist[tid];
        } else {  // sum the replicas: four threads per bin, eight words each
            const int bin = tid >> 2, part = tid & 3;
            uint32_t sum = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint32_t v = hist[bin * 32 + part * 8 + i];
                sum += (v & 0xFFFFu) + (v >> 16);
            }
            sum += __shfl_xor(sum, 1, kWave);
            sum += __shfl_xor(sum, 2, kWave);
            if (part == 0) bins[bin] = sum;
        }
        __syncthreads();
        if (w == 0) {  // the bin b with (#keys in bins above b) < k_rem <= (#keys in bins >= b)
            uint32_t c[4], tot = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                c[i] = bins[4 * lane + i];
                tot += c[i];
            }
            uint32_t sfx = tot;  // keys in the bins of this lane and of all higher lanes
#pragma unroll
            for (int off = 1; off < kWave; off <<= 1) {
                const uint32_t nb = __shfl_down(sfx, off, kWave);
                if (lane + off < kWave) sfx += nb;
            }
            uint32_t above = sfx - tot;
#pragma unroll
            for (int i = 3; i >= 0; --i) {
                const uint32_t incl = above + c[i];
                if (above < k_rem && k_rem <= incl) {
                    sh[0] = (uint32_t)(4 * lane + i);
                    sh[1] = k_rem - above;
                    sh[2] = c[i];
                }
                above = incl;
            }
        }
        __syncthreads();
        prefix = (prefix << 8) | sh[0];
        k_rem = sh[1];
        n_match = sh[2];
    }
    const uint32_t T = prefix, need_eq = k_rem;  // key of the k-th largest; how many keys equal to it are taken

    // keys above / equal to T in this wavefront's segment: those above in the upper 24 bits were counted during
    // the last pass, the rest sit in the wavefront's own level-3 histogram (lane l sums bins 4l .. 4l+3)
    uint32_t my_gt, my_eq;
    {
        const uint32_t d3 = T & 0xFFu;
        uint32_t g = 0, e = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t bin = 4 * lane + i, c = hist[w * kTopkBins + bin];
            g += bin > d3 ? c : 0u;
            e += bin == d3 ? c : 0u;
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            g += __shfl_xor(g, off, kWave);
            e += __shfl_xor(e, off, kWave);
        }
        my_gt = above24 + g;
        my_eq = e;
    }
    if (lane == 0) {
        sh[3 + w] = my_gt;
        sh[3 + kRowWaves + w] = my_eq;
    }
    __syncthreads();
    uint32_t gt_run = 0, eq_run = 0, eq_all = 0;
#pragma unroll
    for (int ww = 0; ww < kRowWaves; ++ww) {
        gt_run += ww < w ? sh[3 + ww] : 0u;
        eq_run += ww < w ? sh[3 + kRowWaves + ww] : 0u;
        eq_all += sh[3 + kRowWaves + ww];
    }
    int32_t *out = idx_out + (size_t)row * k;
    // The comparisons are redone rather than kept: 2 NV lane masks would not fit the scalar registers.  The empty
    // statement hides from the compiler that Tw is T.
    uint32_t Tw = T;
    int base_w = base;
    asm volatile("" : "+v"(Tw), "+v"(base_w));
    if (need_eq == eq_all && k <= kRowStage) {
        // Every key equal to the threshold is taken (usually there is one), so what counts is which keys reach it.  The ids
        // meet in LDS and leave as whole lines: a store of this loop has a lane or four that write.
        uint32_t run = (uint32_t)__builtin_amdgcn_readfirstlane((int)(gt_run + eq_run));
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const bool take = key[j] >= Tw;
            const uint64_t m = __ballot(take);
            const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, run));
            if (take) hist[pos] = (uint32_t)(base_w + 64 * j);  // (k of them, exactly)
            run += (uint32_t)__popcll(m);
            asm volatile("" : "+s"(run));
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (EXPAND) {
            expand_block((const int32_t *)hist, k, expand, row, (int32_t *)hist + k, kRowThreads);
        } else {
            __syncthreads();
            for (int i = tid; i < k; i += kRowThreads) out[i] = (int32_t)hist[i];
        }
        return;
    }
    if (my_eq == 0) {
        // no key of this segment equals the threshold (the usual case): only the keys above it matter.  (128 rows,
        // 20000 of 65536 ids: 27.1 us; with all wavefronts in the loop below 28.7)
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const bool is_gt = key[j] > Tw;
            const uint64_t mg = __ballot(is_gt);
            if (is_gt) {
                const uint32_t pos = gt_run + lanes_below(mg) + (eq_run < need_eq ? eq_run : need_eq);
                if (pos < (uint32_t)k) out[pos] = base_w + 64 * j;
            }
            gt_run += (uint32_t)__popcll(mg);
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int t = base_w + 64 * j;
            const bool is_gt = key[j] > Tw, is_eq = key[j] == Tw;
            const uint64_t mg = __ballot(is_gt), me = __ballot(is_eq);
            const uint32_t gt_me = gt_run + lanes_below(mg), eq_me = eq_run + lanes_below(me);
            if (is_gt || (is_eq && eq_me < need_eq)) {
                const uint32_t pos = gt_me + (eq_me < need_eq ? eq_me : need_eq);
                if (pos < (uint32_t)k) out[pos] = t;
            }
            gt_run += (uint32_t)__popcll(mg);
            eq_run += (uint32_t)__popcll(me);
            if (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (EXPAND) {  // (ids written by this workgroup; ties, or too many for LDS)
        __syncthreads();
        for (int i = tid; i < k; i += kRowThreads) hist[i] = (uint32_t)out[i];
        expand_block((const int32_t *)hist, k, expand, row, (int32_t *)hist + k, kRowThreads);
    }
}

// ------------------------------------------------------------------------------------------
// Long rows (kRowFloor to kRowMost scores, budgets that leave the lists below room): one launch that starts from a guess.  The
// histogram of kRowSamples scores, 16 in a row at 256 places, over slices of their range gives a value that the k largest and
// a margin reach.  Every wavefront compacts those of its scores that do into a list of its own in LDS, and the exact selection works
// on these lists, ten scores a lane at most, on 11-bit digits of the keys' distance from the guess.  The selected ids set bits
// of a bitmap, which is read off in order.  Where many scores are equal to the guess, the lists take those above it and a second bitmap
// the equal ones, of which the lowest ids fill up the budget.  The guess only decides how much is left to do: where fewer than k
// scores or more than the lists hold reach it (samples that miss what the row has), radix passes over the whole row follow.
// The time is the instructions per score of four wavefronts per SIMD (a microsecond for two and a half of them at 65536 scores; a
// workgroup reads such a row in three) and, in all that runs once, the fetching of the code: loops are kept rolled.  Scores
// 1024 apart belong to one thread, so that neighbours, which are alike, spread over all lists.
// Against the row in registers, 8 rows, k a sixteenth: 16384 scores 10.1 -> 10.2 us, 20480, twice the registers, 14.5 -> 10.6 (the lists'
// length decides: k 3000 of 32768 14.6 -> 13.5, rectified 14.6 -> 16.2, hence half of it at most up to 32768 scores), 32768 14.5 -> 12.3,
// 40001 22.9 -> 14.1, 65536 22.4 -> 18.1; against the five launches 32 rows of 131072, k 1024, 38.6 -> 20.5, 128 rows 110 -> 21.
// 8 rows of 32768 equal scores 42 -> 11.9, five different values 19.9 -> 13.1; ninth powers of normal numbers, whose range has to be sliced
// again, 14.7 -> 19.9, 65536 of them 21.4 -> 24.1; radix passes 67 and 91.  Of 131072 scores, where the five launches use more compute units
// than 8 rows have here, equal ones 27 -> 30, rising ones 24 -> 27, normal ones 27 -> 20.
// ------------------------------------------------------------------------------------------
constexpr int kRowFloor = 16 * kRowThreads + 1, kRowMost = 131072, kRowSamples = 4096;
constexpr int kRowExpect = 8192;  // scores that may be expected to reach the guess
constexpr float kRowSigmas = 4.5f;  // margin in standard deviations of the samples' rank

template <int CTRL> __device__ __forceinline__ uint32_t max_step(uint32_t x)
{
    const uint32_t y = __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
    return x > y ? x : y;
}
__device__ __forceinline__ uint32_t wave_max_dpp(uint32_t x)  // the same in every lane
{
    x = max_step<0x111>(x);
    x = max_step<0x112>(x);
    x = max_step<0x114>(x);
    x = max_step<0x118>(x);
    x = max_step<0x142>(x);
    x = max_step<0x143>(x);
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}
template <int CTRL> __device__ __forceinline__ float max_step(float x)
{
    return fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(x), __float_as_uint(x), CTRL, 0xF, 0xF, false)));
}
__device__ __forceinline__ float wave_max_dpp(float x)
{
    x = max_step<0x111>(x);
    x = max_step<0x112>(x);
    x = max_step<0x114>(x);
    x = max_step<0x118>(x);
    x = max_step<0x142>(x);
    x = max_step<0x143>(x);
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), 63));
}
__device__ __forceinline__ float float_of_key(uint32_t key) { return __uint_as_float((int)key < 0 ? key ^ 0x80000000u : ~key); }

// LDS of the guess: bitmap, bins, lists, bitmap of the scores that equal the guess
constexpr int kRowListWords = 2 * kRowWaves * kRowList, kRowMapWords = kRowMost / 32;
constexpr int kRowWords = kRowListWords + kRowBins + kRowMapWords;  // ... without the last

// Bounds (as floats' bits) from the samples: at least r_lo and, where that can be had, at most r_max of them reach lo_bits; about r_hi
// hi_bits.  Slices of the samples' range; where the one that holds the r_lo-th largest has too many (few large scores
// stretch the range) or many that may be equal, slices of that one, and so on.  True: the samples in it are all equal, and lo_bits is
// what they are.  bins: zero before and after.
constexpr int kRowSlicings = 5;
constexpr uint32_t kRowEqual = 384;  // samples in a slice that call for a closer look (equal scores add up in one counter; a slicing takes 0.7 us)
__device__ __forceinline__ bool guess_bounds(const float (&x)[4], uint32_t r_lo, uint32_t r_hi, uint32_t r_max, uint32_t *bins, RowShared &sh,
                                             uint32_t &lo_bits, uint32_t &hi_bits)
{
    static_assert(kRowSamples == 4 * kRowThreads && kRowBins == 2 * kRowThreads, "four samples and two bins per thread");
    const int w = wave_id(), tid = threadIdx.x;
    uint32_t bin[4], in = 15u, above_all = 0;  // slices of this thread's samples, which are in the one at hand; samples of all threads above it
    if (tid < 2) sh.pick[tid][0] = tid == 0 ? 0u : kRowBins - 1;
    // one slicing of the samples `in`: finds the slices of the r_lo-th and, where it is in it, the r_hi-th largest; true: that will do
    auto slice = [&](float mn, float range, int level) __attribute__((always_inline)) {
        __syncthreads();
        const uint32_t c0 = bins[2 * tid], c1 = bins[2 * tid + 1];
        bins[2 * tid] = 0;
        bins[2 * tid + 1] = 0;
        const uint32_t above = sum_above(c0 + c1, sh.wave[level & 1]);
        auto pick = [&](int which, uint32_t r) __attribute__((always_inline)) {
            if (above < r && r <= above + c1 + c0) {
                const bool odd = r <= above + c1;
                sh.pick[which][0] = 2 * tid + (odd ? 1 : 0);
                sh.pick[which][1] = above + (odd ? 0u : c1);
                sh.pick[which][2] = odd ? c1 : c0;
            }
        };
        const bool hi_in = level == 0 || r_hi > above_all;
        pick(0, r_lo - above_all);
        if (hi_in) pick(1, r_hi - above_all);
        __syncthreads();
        const uint32_t b_lo = sh.pick[0][0], in_bin = sh.pick[0][2];
        const float width = range * (1.0f / kRowBins);
        // (a thousandth of a slice lower: an edge rounded up, by 2^-12 at most, would leave out scores that the slice has)
        lo_bits = __float_as_uint(fmaf((float)b_lo - 0.001f, width, mn));
        if (hi_in) hi_bits = __float_as_uint(fmaf((float)sh.pick[1][0] + 1.0f, width, mn));
        above_all += sh.pick[0][1];
        if (above_all + in_bin <= r_max && in_bin <= kRowEqual) return true;
#pragma unroll
        for (int u = 0; u < 4; ++u) in &= ~((bin[u] == b_lo ? 0u : 1u) << u);
        return false;
    };
    // (scores that are not finite count as the nearest end of the others' range; NaN as the lower end)
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (fabsf(x[u]) < INFINITY) {
            mn = fminf(mn, x[u]);
            mx = fmaxf(mx, x[u]);
        }
    mn = -wave_max_dpp(-mn);
    mx = wave_max_dpp(mx);
    if (lane_id() == 0) {
        sh.lo[w] = __float_as_uint(mn);
        sh.hi[w] = __float_as_uint(mx);
    }
    __syncthreads();
#pragma unroll
    for (int ww = 0; ww < kRowWaves; ++ww) {
        mn = fminf(mn, __uint_as_float(sh.lo[ww]));
        mx = fmaxf(mx, __uint_as_float(sh.hi[ww]));
    }
    float range = mx - mn, scale = range > 0.0f && range < INFINITY ? (float)kRowBins / range : 0.0f;
    auto bin_of = [&](float v) __attribute__((always_inline)) {
        return (uint32_t)fminf(fmaxf((v - mn) * scale, 0.0f), (float)(kRowBins - 1));
    };
    if (__builtin_expect(range == 0.0f, 0)) {  // (zeros of both signs are looked at below)
        hi_bits = __float_as_uint(mx + 0.0f);
        __syncthreads();
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bin[u] = bin_of(x[u]);
            atomicAdd(&bins[bin[u]], 1u);
        }
        if (__builtin_expect(slice(mn, range, 0), 1)) return false;
    }
    for (int level = 1; level < kRowSlicings; ++level) {
        uint32_t kmn = 0, kmx = 0;  // keys, the lower one turned over: zero where there is none
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if ((in >> u & 1u) && fabsf(x[u]) < INFINITY) {
                const uint32_t key = order_key(x[u]);
                kmn = kmn > ~key ? kmn : ~key;
                kmx = kmx > key ? kmx : key;
            }
        kmn = wave_max_dpp(kmn);
        kmx = wave_max_dpp(kmx);
        if (lane_id() == 0) {
            sh.lo[w] = kmn;
            sh.hi[w] = kmx;
        }
        __syncthreads();
#pragma unroll
        for (int ww = 0; ww < kRowWaves; ++ww) {
            kmn = kmn > sh.lo[ww] ? kmn : sh.lo[ww];
            kmx = kmx > sh.hi[ww] ? kmx : sh.hi[ww];
        }
        kmn = (uint32_t)__builtin_amdgcn_readfirstlane((int)~kmn);
        kmx = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmx);
        mn = float_of_key(kmn);
        if (kmn == kmx) {
            lo_bits = __float_as_uint(mn);
            return true;
        }
        range = float_of_key(kmx) - mn;
        scale = range > 0.0f && range < INFINITY ? (float)kRowBins / range : 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            bin[u] = range == 0.0f ? (__float_as_uint(x[u]) == 0u ? 1u : 0u) : bin_of(x[u]);  // (zeros of both signs)
            if (in >> u & 1u) atomicAdd(&bins[bin[u]], 1u);
        }
        if (slice(mn, range, level)) return false;
    }
    return false;
}

// Calls f(bits, id, real) for every score of the row in groups of 8 x 1024, thread tid taking scores tid, tid + 1024, ..; the next two
// groups are in flight.  (Beyond the row `real` is false; it is a constant in all groups but the last.)
template <typename F> __device__ __forceinline__ void for_scores(const float *__restrict__ Srow, int L, F f)
{
    constexpr int U = 8, GROUP = U * kRowThreads;
    const int tid = threadIdx.x;
    uint32_t v[2][U];
    auto fetch = [&](int t0, uint32_t (&x)[U]) __attribute__((always_inline)) {  // (always requested: the waits count requests)
        if (t0 + GROUP <= L) {
#pragma unroll
            for (int j = 0; j < U; ++j) x[j] = __float_as_uint((Srow + t0 + kRowThreads * j)[(uint32_t)tid]);
        } else {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const int t = t0 + kRowThreads * j + tid;
                x[j] = __float_as_uint(Srow[(uint32_t)(t < L ? t : L - 1)]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    fetch(0, v[0]);
    fetch(GROUP, v[1]);
    for (int t0 = 0; t0 < L; t0 += 2 * GROUP) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int g0 = t0 + GROUP * h;
            if (g0 + GROUP <= L) {
#pragma unroll
                for (int j = 0; j < U; ++j) f(v[h][j], g0 + kRowThreads * j + tid, std::true_type());
            } else if (g0 < L) {
#pragma unroll
                for (int j = 0; j < U; ++j) f(v[h][j], g0 + kRowThreads * j + tid, g0 + kRowThreads * j + tid < L);
            }
            fetch(g0 + 2 * GROUP, v[h]);
        }
    }
}

// The same selection by four radix passes over the row: where the guess did not help.  Sets the bits of the
// selected ids in map (`words`, cleared here).  hist: kTopkBins * 32 words.
__device__ __forceinline__ void select_by_radix(const float *__restrict__ Srow, int L, uint32_t k, uint32_t *hist, uint32_t *map, int words,
                                                RowShared &sh)
{
    const int tid = threadIdx.x, lane = lane_id();
    uint32_t prefix = 0, k_rem = k, in_bin = 0;
    __syncthreads();
    for (int i = tid; i < kTopkBins * 32; i += kRowThreads) hist[i] = 0;
    for (int i = tid; i < words; i += kRowThreads) map[i] = 0;
    for (int level = 0; level < kTopkLevels; ++level) {
        __syncthreads();
        // (counters replicated 32 times: scores cluster in few bins at the top levels)
        for_scores(Srow, L, [&](uint32_t bits, int, auto real) __attribute__((always_inline)) {
            const uint32_t key = order_key(__uint_as_float(bits));
            if (real && (level == 0 || key >> (32 - 8 * level) == prefix)) atomicAdd(&hist[(key >> (24 - 8 * level) & 0xFFu) * 32 + (lane & 31)], 1u);
        });
        __syncthreads();
        uint32_t sum = 0;  // four threads per bin, eight counters each
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int at = (tid >> 2) * 32 + (tid & 3) * 8 + ((i + (tid >> 2)) & 7);
            sum += hist[at];
            hist[at] = 0;
        }
        sum += __builtin_amdgcn_update_dpp(0u, sum, 0xB1, 0xF, 0xF, true);
        sum += __builtin_amdgcn_update_dpp(0u, sum, 0x4E, 0xF, 0xF, true);
        const uint32_t c = (tid & 3) == 0 ? sum : 0u, above = sum_above(c, sh.wave[level & 1]);
        if (above < k_rem && k_rem <= above + c) {
            sh.pick[level & 1][0] = tid >> 2;
            sh.pick[level & 1][1] = k_rem - above;
            sh.pick[level & 1][2] = c;
        }
        __syncthreads();
        prefix = prefix << 8 | sh.pick[level & 1][0];
        k_rem = sh.pick[level & 1][1];
        in_bin = sh.pick[level & 1][2];
        if (in_bin == k_rem && level < kTopkLevels - 1) {  // everything from here up
            prefix <<= 24 - 8 * level;
            break;
        }
    }
    const bool ties = in_bin != k_rem;
    uint32_t *eq = hist;
    if (ties) {
        for (int i = tid; i < words; i += kRowThreads) eq[i] = 0;  // (hist is read)
        __syncthreads();
    }
    for_scores(Srow, L, [&](uint32_t bits, int t, auto real) __attribute__((always_inline)) {
        const uint32_t key = order_key(__uint_as_float(bits));
        // 64 neighbouring scores per wavefront: their bits are two words of the map
        const uint64_t m = __ballot(real && (ties ? key > prefix : key >= prefix)), e = ties ? __ballot(real && key == prefix) : 0;
        if (lane < 2 && real) {
            map[(t >> 5) + lane] = (uint32_t)(m >> (32 * lane));
            if (ties) eq[(t >> 5) + lane] = (uint32_t)(e >> (32 * lane));
        }
    });
    __syncthreads();
    if (ties) lowest_bits(eq, map, words, k_rem, sh);
    __syncthreads();
}

// r_lo, r_hi, r_max: ranks among the samples, see guess_bounds.  expand as above.
__global__ __launch_bounds__(kRowThreads) void topk_long_kernel(const float *__restrict__ S, int32_t *__restrict__ idx_out, int L, int k,
                                                               uint32_t r_lo, uint32_t r_hi, uint32_t r_max, ExpandArgs expand)
{
    // bitmap, bins, lists (counters of the radix passes; at the end, with `expand`, the ids and what their union needs), equals
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    __shared__ RowShared sh;
    const int row = blockIdx.x, tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const float *Srow = S + (size_t)row * L;
    const int words = (L + 63) / 64 * 2;
    uint32_t *map = smem, *bins = smem + kRowMapWords, *lists = bins + kRowBins;
    bool done;
    {
        float sample[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            sample[u] = Srow[(uint32_t)(16 * w + 4 * u + (lane >> 4)) * (uint32_t)(L - 16) / 255u + (lane & 15)];
        bins[2 * tid] = 0;
        bins[2 * tid + 1] = 0;
        for (int i = tid; i < words; i += kRowThreads) map[i] = 0;
        uint32_t *eq = lists + kRowListWords;
        if (tid < 2) eq[words - 2 + tid] = 0;  // (all others are written)
        uint32_t lo_bits, hi_bits;
        const bool equal = guess_bounds(sample, r_lo, r_hi, r_max, bins, sh, lo_bits, hi_bits);  // (the same for all threads)
        lo_bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo_bits);
        // Scores that reach the bound.  Their bits as signed numbers are in order above zero; below a negative bound lie exactly
        // the larger unsigned numbers: turned over, they are in the same order.
        const uint32_t flip = (int)lo_bits < 0 ? 0x7FFFFFFFu : 0u;
        const int bound = (int)(lo_bits ^ flip);
        uint32_t *list = lists + w * 2 * kRowList, count = 0;  // scores, then ids: one store of two words; counted on where it is full
        auto compact = [&](bool take, uint32_t bits, int t) __attribute__((always_inline)) {
            const uint64_t m = __ballot(take);
            if (equal && m == 0) return;  // (few are taken then)
            const uint32_t pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, count));
            const uint32_t at = pos < kRowList ? pos : kRowList - 1;  // (a list that overflows is not used)
            if (take) {
                list[at] = bits;
                list[at + kRowList] = (uint32_t)t;
            }
            count += (uint32_t)__popcll(m);
        };
        const uint32_t lo_key = order_key(__uint_as_float(lo_bits)), hi_key = order_key(__uint_as_float(hi_bits));
        if (!equal) {
            for_scores(Srow, L, [&](uint32_t bits, int t, auto real) __attribute__((always_inline)) {
                compact(real && (int)(bits ^ flip) >= bound, bits, t);
            });
            done = select_from_lists(lists, count, k, lo_key, hi_key, bins, map, words, sh);
        } else {
            // many scores are equal to the bound: those go to a bitmap, the lists take what is above
            for_scores(Srow, L, [&](uint32_t bits, int t, auto real) __attribute__((always_inline)) {
                compact(real && (int)(bits ^ flip) > bound, bits, t);
                const uint64_t e = __ballot(real && bits == lo_bits);
                if (lane < 2 && real) eq[(t >> 5) + lane] = (uint32_t)(e >> (32 * lane));  // (64 neighbours per wavefront)
            });
            if (lane == 0) sh.wave[2][w] = count;
            __syncthreads();
            uint32_t n = 0, most = 0;
#pragma unroll
            for (int ww = 0; ww < kRowWaves; ++ww) {
                n += sh.wave[2][ww];
                most = sh.wave[2][ww] > most ? sh.wave[2][ww] : most;
            }
            if (most > kRowList) {
                done = false;
            } else if (n >= (uint32_t)k) {
                done = select_from_lists(lists, count, k, lo_key, hi_key, bins, map, words, sh);
            } else {  // all of those, and the lowest ids of the equal ones
                for (uint32_t i = lane; i < count; i += 64) atomicOr(&map[list[kRowList + i] >> 5], 1u << (list[kRowList + i] & 31));
                __syncthreads();
                lowest_bits(eq, map, words, (uint32_t)k - n, sh);
#pragma unroll
                for (int ww = 0; ww < kRowWaves; ++ww) n += sh.wave[0][ww];
                done = n >= (uint32_t)k;
                __syncthreads();
            }
        }
    }
    if (!done) select_by_radix(Srow, L, k, lists, map, words, sh);
    if (expand.rows) {
        int32_t *ids = (int32_t *)bins;
        write_map(map, words, k, sh, ids);
        expand_block(ids, k, expand, row, ids + k, kRowThreads);
    } else {
        write_map(map, words, k, sh, idx_out + (size_t)row * k);
    }
}

// Ranks among the samples for a row's guess (0: none).  Margin: kRowSigmas standard deviations of the number of samples that the k
// largest scores have, and an eighth of k for scores that come in clusters.
static uint32_t row_guess(int L, int k, uint32_t *r_hi, uint32_t *r_max)
{
    *r_hi = *r_max = 0;
    if (L < kRowFloor || L > kRowMost) return 0;
    const double share = (double)k / L, mean = share * kRowSamples, dev = kRowSigmas * std::sqrt(mean * (1.0 - share)) + mean / 8 + 4.0;
    const double reach = (mean + 2 * dev) * L / kRowSamples;
    if ((reach < L ? reach : L) > (L <= kRowThreads * 32 ? kRowExpect / 2 : kRowExpect)) return 0;
    *r_max = (uint32_t)((double)kRowExpect * kRowSamples / L);
    *r_hi = mean > dev ? (uint32_t)(mean - dev) : 0u;
    return (uint32_t)(mean + dev) + 1u;
}

bool topk_row_shape_ok(const xkv_shape &s)
{
    uint32_t r_hi, r_max;
    return s.L <= kRowThreads * 64 || row_guess(s.L, s.k, &r_hi, &r_max) > 0;
}

// Whether the rows of the chunks fit `most` words of LDS behind `before`; then *ex is set and *words is raised to what they need.
static bool with_expansion(const xkv_shape &s, const ExpandArgs *expand, bool *expanded, size_t before, size_t most, ExpandArgs *ex, size_t *words)
{
    if (!expand) return false;
    const size_t need = before + s.k + expand_lds_words(s.k, expand->o);
    if (need > most) return false;
    *ex = *expand;
    *expanded = true;
    if (*words < need) *words = need;
    return true;
}

template <int NV>
static hipError_t launch_topk_row_t(const xkv_shape &s, const Plan &p, const float *S, int32_t *idx, const ExpandArgs *expand,
                                    bool *expanded, hipStream_t st)
{
    size_t words = s.k <= kRowStage && s.k > kTopkBins * 32 ? s.k : kTopkBins * 32;
    ExpandArgs ex{};
    static DynamicLdsOnce attr, attr_expand;  // (two kernels: rows of a few thousand scores take 8.0 us, 8.3 with the expansion in the code)
    if (with_expansion(s, expand, expanded, 0, kRowStage, &ex, &words)) {
        const hipError_t e = attr_expand.ensure((const void *)topk_row_kernel<NV, true>, (size_t)kRowStage * 4);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((topk_row_kernel<NV, true>), dim3(p.rows), dim3(kRowThreads), 4 * words, st, S, idx, s.L, s.k, ex);
    } else {
        const hipError_t e = attr.ensure((const void *)topk_row_kernel<NV, false>, (size_t)kRowStage * 4);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((topk_row_kernel<NV, false>), dim3(p.rows), dim3(kRowThreads), 4 * words, st, S, idx, s.L, s.k, ex);
    }
    return hipGetLastError();
}

static hipError_t launch_topk_long(const xkv_shape &s, const Plan &p, const float *S, int32_t *idx, uint32_t r_lo, uint32_t r_hi,
                                   uint32_t r_max, const ExpandArgs *expand, bool *expanded, hipStream_t st)
{
    static DynamicLdsOnce attr;
    size_t words = kRowWords + kRowMapWords;
    const hipError_t e = attr.ensure((const void *)topk_long_kernel, words * 4);
    if (e != hipSuccess) return e;
    ExpandArgs ex{};
    with_expansion(s, expand, expanded, kRowMapWords, kRowWords, &ex, &words);
    hipLaunchKernelGGL(topk_long_kernel, dim3(p.rows), dim3(kRowThreads), 4 * words, st, S, idx, s.L, s.k, r_lo, r_hi, r_max, ex);
    return hipGetLastError();
}

hipError_t launch_topk_init(const Plan &p, uint32_t *state, hipStream_t st)
{
    const int words = p.rows * kTopkLevels * kTopkBins;
    hipLaunchKernelGGL(topk_init_kernel, dim3((words + 255) / 256), dim3(256), 0, st, topk_row_hist(p, state), words);
    return hipGetLastError();
}

hipError_t launch_topk(const xkv_shape &s, const Plan &p, const float *S, int32_t *idx, uint32_t *hist,
                       uint32_t *state, bool level0_done, hipStream_t st, const ExpandArgs *expand, bool *expanded)
{
    if (expanded) *expanded = false;
    if (p.topk_row) {
        uint32_t r_hi, r_max;
        const uint32_t r_lo = row_guess(s.L, s.k, &r_hi, &r_max);
        if (r_lo > 0) return launch_topk_long(s, p, S, idx, r_lo, r_hi, r_max, expand, expanded, st);
        const int per_thread = (s.L + kRowThreads - 1) / kRowThreads;
        if (per_thread <= 8) return launch_topk_row_t<8>(s, p, S, idx, expand, expanded, st);
        if (per_thread <= 16) return launch_topk_row_t<16>(s, p, S, idx, expand, expanded, st);
        if (per_thread <= 32) return launch_topk_row_t<32>(s, p, S, idx, expand, expanded, st);
        return launch_topk_row_t<64>(s, p, S, idx, expand, expanded, st);
    }
    TopkScratch ws;
    ws.hist = hist;
    ws.state = state;
    ws.row_hist = topk_row_hist(p, state);
    ws.chunk_gt = ws.row_hist + (size_t)p.rows * kTopkLevels * kTopkBins;
    dim3 grid(p.topk_chunks, p.rows), block(256);
    if (!level0_done) {
        hipError_t e = launch_topk_init(p, state, st);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(topk_hist_kernel<0>, grid, block, 0, st, S, ws, s.L, s.k, p.topk_chunks, p.topk_chunk);
    }
    hipLaunchKernelGGL(topk_hist_kernel<1>, grid, block, 0, st, S, ws, s.L, s.k, p.topk_chunks, p.topk_chunk);
    hipLaunchKernelGGL(topk_hist_kernel<2>, grid, block, 0, st, S, ws, s.L, s.k, p.topk_chunks, p.topk_chunk);
    hipLaunchKernelGGL(topk_hist_kernel<3>, grid, block, 0, st, S, ws, s.L, s.k, p.topk_chunks, p.topk_chunk);
    hipLaunchKernelGGL(topk_write_kernel, grid, block, 0, st, S, ws, idx, s.L, s.k, p.topk_chunks, p.topk_chunk);
    return hipGetLastError();
}

}  // namespace xkv
