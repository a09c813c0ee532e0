// Exact selection of the k largest of a row's scores by one workgroup of kRowThreads threads, from lists in LDS (block functions).
#ifndef XKV_ROW_SELECT_H
#define XKV_ROW_SELECT_H

#include "xkv_common.h"

namespace xkv {

constexpr int kRowWaves = 16, kRowThreads = kRowWaves * 64;
constexpr int kRowBins = 2048;
constexpr int kRowRounds = 10, kRowList = 64 * kRowRounds;  // entries of a wavefront's list

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Inclusive sum over the lanes below and this one.
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t scan_step(uint32_t x)
{
    return x + __builtin_amdgcn_update_dpp(0u, x, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
    x = scan_step<0x111, 0xF>(x);  // within rows of 16: from 1, 2, 4 and 8 lanes below
    x = scan_step<0x112, 0xF>(x);
    x = scan_step<0x114, 0xF>(x);
    x = scan_step<0x118, 0xF>(x);
    x = scan_step<0x142, 0xA>(x);  // row 0's total to row 1, row 2's to row 3, then that of both to the upper half
    return scan_step<0x143, 0xC>(x);
}
struct RowShared {
    uint32_t wave[3][kRowWaves], pick[2][4];
    uint32_t lo[kRowWaves], hi[kRowWaves];
};
// Sum over the threads above this one of `mine`; *all: over all threads.  part: kRowWaves words that nobody reads any more.
// One barrier.
__device__ __forceinline__ uint32_t sum_above(uint32_t mine, uint32_t *part)
{
    const uint32_t s = wave_scan(mine), all = (uint32_t)__builtin_amdgcn_readlane((int)s, 63);
    const int w = wave_id();
    if (lane_id() == 0) part[w] = all;
    __syncthreads();
    uint32_t above = all - s;
#pragma unroll
    for (int ww = 1; ww < kRowWaves; ++ww) above += ww > w ? part[ww] : 0u;
    return above;
}
__device__ __forceinline__ uint32_t sum_below(uint32_t mine, uint32_t *part)
{
    const uint32_t s = wave_scan(mine);
    const int w = wave_id();
    if (lane_id() == 63) part[w] = s;
    __syncthreads();
    uint32_t below = s - mine;
#pragma unroll
    for (int ww = 0; ww < kRowWaves - 1; ++ww) below += ww < w ? part[ww] : 0u;
    return below;
}

// Set bits of map[0 .. words) in ascending order to out; at most `k` are set.  One barrier; whoever set the bits has passed one.
__device__ __forceinline__ void write_map(const uint32_t *map, int words, uint32_t k, RowShared &sh, int32_t *out)
{
    const int per = (words + kRowThreads - 1) / kRowThreads, first = (int)threadIdx.x * per;
    uint32_t n = 0;
    for (int i = 0; i < per; ++i) n += first + i < words ? (uint32_t)__popc(map[first + i]) : 0u;
    uint32_t pos = sum_below(n, sh.wave[2]);
    for (int i = 0; i < per; ++i) {
        uint32_t m = first + i < words ? map[first + i] : 0u;
        while (m != 0) {
            if (pos < k) out[pos] = 32 * (first + i) + __ffs((int)m) - 1;
            ++pos;
            m &= m - 1;
        }
    }
}

// Adds the k_rem lowest set bits of eq to map.  One barrier; the bits have been set before one.
__device__ __forceinline__ void lowest_bits(const uint32_t *eq, uint32_t *map, int words, uint32_t k_rem, RowShared &sh)
{
    const int per = (words + kRowThreads - 1) / kRowThreads, first = (int)threadIdx.x * per;
    uint32_t n = 0;
    for (int i = 0; i < per; ++i) n += first + i < words ? (uint32_t)__popc(eq[first + i]) : 0u;
    uint32_t before = sum_below(n, sh.wave[0]);
    for (int i = 0; i < per && first + i < words; ++i) {
        uint32_t m = eq[first + i], take = 0;
        for (; m != 0 && before < k_rem; ++before) {
            take |= m & -m;
            m &= m - 1;
        }
        map[first + i] |= take;
    }
}

// The k largest by (key, lower id first) of the scores in the wavefronts' lists (the scores' bits, then their ids; `count` in this
// wavefront's), all of whose keys are >= lo; hi: a key that few exceed (any value is right).  Sets the bits of their ids in map
// (zero before; `words` of them) and returns true, or false where there are fewer than k or a list was too short.
// bins: zero.
__device__ __forceinline__ bool select_from_lists(uint32_t *lists, uint32_t count, uint32_t k, uint32_t lo, uint32_t hi, uint32_t *bins,
                                                  uint32_t *map, int words, RowShared &sh)
{
    const int lane = lane_id(), w = wave_id(), tid = threadIdx.x;
    if (lane == 0) sh.wave[2][w] = count;
    const uint32_t mine = count < kRowList ? count : kRowList;
    const uint32_t *list = lists + w * 2 * kRowList + lane;
    uint32_t d[kRowRounds], id[kRowRounds];  // distances from lo
#pragma unroll
    for (int j = 0; j < kRowRounds; ++j) {
        d[j] = id[j] = 0;
        if ((uint32_t)(64 * j) < mine) {  // (the same in the wavefront)
            d[j] = order_key(__uint_as_float(list[64 * j])) - lo;
            id[j] = list[64 * j + kRowList];
        }
    }
    auto real = [&](int j) __attribute__((always_inline)) { return (uint32_t)(64 * j + lane) < mine; };
    // undecided: distances in [base, base + 2^width), of which k_rem are taken, and everything above is
    uint32_t base = 0, k_rem = k, in_bin = 0;
    int width = 32, shift = 32 - __clz((int)((hi > lo ? hi - lo : 0u) | 1u)) - 11;
    shift = shift < 0 ? 0 : shift;
    for (int level = 0;; ++level) {
        // (where the bins don't span the interval, the last one takes the rest of it)
#pragma unroll
        for (int j = 0; j < kRowRounds; ++j) {
            if ((uint32_t)(64 * j) >= mine) break;
            const uint32_t x = d[j] - base, bin = x >> shift;
            if (real(j) && d[j] >= base && (width == 32 || x >> width == 0u)) atomicAdd(&bins[bin < kRowBins ? bin : kRowBins - 1], 1u);
        }
        __syncthreads();
        if (level == 0) {
            uint32_t n = 0, most = 0;
#pragma unroll
            for (int ww = 0; ww < kRowWaves; ++ww) {
                n += sh.wave[2][ww];
                most = sh.wave[2][ww] > most ? sh.wave[2][ww] : most;
            }
            if (n < k || most > kRowList) return false;
        }
        const uint32_t c0 = bins[2 * tid], c1 = bins[2 * tid + 1];
        bins[2 * tid] = 0;
        bins[2 * tid + 1] = 0;
        const uint32_t above = sum_above(c0 + c1, sh.wave[level & 1]);
        uint32_t *pick = sh.pick[level & 1];
        if (above < k_rem && k_rem <= above + c1 + c0) {
            const bool odd = k_rem <= above + c1;
            pick[0] = 2 * tid + (odd ? 1 : 0);
            pick[1] = k_rem - above - (odd ? 0u : c1);
            pick[2] = odd ? c1 : c0;
        }
        __syncthreads();
        const uint32_t bin = pick[0];
        k_rem = pick[1];
        in_bin = pick[2];
        base += bin << shift;
        const bool rest = shift + 11 < width && bin == kRowBins - 1;
        if (!rest) width = shift;
        if (in_bin == k_rem || width == 0) break;  // all of them are taken, or they are equal
        shift = width > 11 ? width - 11 : 0;
    }
    const bool ties = in_bin != k_rem;  // distances above base are taken, and the k_rem lowest ids of those equal to it
#pragma unroll
    for (int j = 0; j < kRowRounds; ++j) {
        if ((uint32_t)(64 * j) >= mine) break;
        if (real(j) && (ties ? d[j] > base : d[j] >= base)) atomicOr(&map[id[j] >> 5], 1u << (id[j] & 31));
    }
    if (ties) {
        uint32_t *eq = lists;  // (all entries are in registers)
        __syncthreads();
        for (int i = tid; i < words; i += kRowThreads) eq[i] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kRowRounds; ++j)
            if (real(j) && d[j] == base) atomicOr(&eq[id[j] >> 5], 1u << (id[j] & 31));
        __syncthreads();
        lowest_bits(eq, map, words, k_rem, sh);
    }
    __syncthreads();
    return true;
}

}  // namespace xkv
#endif
