// 4-bit and 3-bit round-to-nearest quantisation of rows of the token basis A (App. "Integrate with Quantization": a
// plain RTN quantiser on the compressed cache, 25.6x at 4 bits and 32x at 3 bits; the formats below are what the two
// published ratios imply -- one extra bit per element of side information = two 16-bit numbers per group of 32).
//
// 3-bit row layout: one 16-byte piece per group of 32 ranks -- 96 bits of codes (little-endian over three words),
// then the word (step, lo) of two bf16 -- so r/2 bytes per row.  The 96 bits are four units of 24 bits, unit u for
// ranks 8u..8u+7 of the group; inside a unit the even ranks sit in the low 12 bits (rank 8u+2i at bits [3i, 3i+3))
// and the odd ranks in the high 12 (rank 8u+2i+1 at bits [12+3i, 12+3i+3)), so that moving the high half up to bit
// 16 gives the same "two adjacent ranks 16 bits apart" word as the 4-bit format.  step = bf16((max - lo) / 7).
//
// 4-bit row layout, r a multiple of 32:  r/8 32-bit words of codes (word j holds ranks 8j..8j+7: rank 8j+2i in bits
// [4i, 4i+4), rank 8j+2i+1 in bits [16+4i, 16+4i+4), so two adjacent ranks are one shift and one mask away from a
// packed pair of 16-bit numbers), then r/32 pairs (step, lo) of bf16: 5r/8 bytes, then zero bytes up to the next
// multiple of 16 (none when r is a multiple of 128), so that every row and every group is 16-byte aligned.
//   lo = min of the group, step = bf16((max - lo) / 15) (1 if that is 0), code = clip(rint((x - lo) * (1 / step)), 0, 15),
// each a single fp32 operation (the same sequence as the CPU oracle: the codes agree bit for bit);  x^ = step * code + lo.
#include "xkv_common.h"

namespace xkv {

typedef __attribute__((ext_vector_type(4))) uint32_t q_u32x4_t;

constexpr long long kQuantFar = 160 * 1024 * 1024;  // bytes
constexpr int kQuantCached = 2048 * 1024, kQuantSmall = 416 * 1024;  // pieces of 16 bytes

template <int CTRL> __device__ __forceinline__ uint32_t quad_perm(uint32_t x)  // lane exchange within groups of four
{
    return __builtin_amdgcn_update_dpp(0u, x, CTRL, 0xF, 0xF, true);
}
// (fminf / fmaxf would first turn signalling NaN into quiet ones, an instruction per operand)
__device__ __forceinline__ float min3(float a, float b, float c)
{
    float d;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ float max3(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// (lo, hi) of a group -> its step and the reciprocal.  The two quotients take a product and a correction each: with y the rounded
// reciprocal of b, q = a y and r = a - b q (exact), q + r y is the rounded a / b; a reciprocal one unit off is corrected the same way
// unless all 24 bits of b are ones, and a step has 8 (Markstein, IBM J. Res. Dev. 34, 1990).  Outside the range where r is exact the
// ordinary division is used.
template <int BITS> __device__ __forceinline__ void group_scale(float lo, float hi, float &step, float &inv)
{
    constexpr float kQmax = (float)((1 << BITS) - 1), kQinv = 1.0f / kQmax;
    constexpr uint32_t kSmall = 0x20000000u, kLarge = 0x5F000000u;  // 2^-63, 2^63
    const float range = hi - lo;
    float q = range * kQinv;
    q = fmaf(fmaf(-kQmax, q, range), kQinv, q);
    if (__float_as_uint(range) - kSmall > kLarge - kSmall && range != 0.0f) q = range / kQmax;
    step = bf16_to_f32(f32_to_bf16(q));
    step = step > 0.0f ? step : 1.0f;
    inv = __builtin_amdgcn_rcpf(step);
    inv = fmaf(fmaf(-step, inv, 1.0f), inv, inv);
    if (__float_as_uint(step) - kSmall > kLarge - kSmall) inv = 1.0f / step;
}

// Eight ranks (four words of two) -> their codes: even ranks in the low half, odd ranks in the high half (16 bits up for 4-bit codes, 12
// for 3-bit codes).
template <int BITS> __device__ __forceinline__ uint32_t eight_codes(const float (&x)[8], float lo, float inv)
{
    constexpr float kQmax = (float)((1 << BITS) - 1);
    float c[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) c[e] = __builtin_amdgcn_fmed3f(rintf((x[e] - lo) * inv), 0.0f, kQmax);
    uint32_t word = 0;
    if constexpr (BITS == 4) {
#pragma unroll
        for (int h = 0; h < 4; ++h) {  // byte h: ranks 4 (h % 2) + h / 2 and two further
            const int e = 4 * (h & 1) + (h >> 1);
            word = __builtin_amdgcn_cvt_pk_u8_f32(fmaf(c[e + 2], 16.0f, c[e]), h, word);
        }
    } else {
        // (a half of four codes is a number below 4096: exact in single precision)
        const float even = fmaf(fmaf(c[6], 8.0f, c[4]), 64.0f, fmaf(c[2], 8.0f, c[0]));
        const float odd = fmaf(fmaf(c[7], 8.0f, c[5]), 64.0f, fmaf(c[3], 8.0f, c[1]));
        word = (uint32_t)fmaf(odd, 4096.0f, even);
    }
    return word;
}

__device__ __forceinline__ void unpack8(const q_u32x4_t &raw, float (&x)[8])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[2 * e] = __uint_as_float(raw[e] << 16);
        x[2 * e + 1] = __uint_as_float(raw[e] & 0xFFFF0000u);
    }
}

__device__ __forceinline__ uint32_t group_params(float step, float lo)
{
    return (__float_as_uint(step) >> 16) | __float_as_uint(lo);  // (both have empty low halves)
}

// Large calls: a lane per group of 32 ranks, four 16-byte pieces, so that what a group needs is done once.  A workgroup takes whole rows,
// as many as 256 groups make, collects the quantised rows in LDS and writes them as one run of 16-byte pieces; with rows longer
// than that (STAGED false) every lane stores its own.
// What bounds it: the stream, then about 75 vector instructions per piece; 140 with a lane per piece, where the two took the same time.
// 50001 rows of 512 in 4 bits 13.5 us (67 MB; reading and writing as many bytes alone 11.5), a lane per piece 16.6; 3 bits 12.4 and
// 15.9; 262144 rows 60.4 and 68.6, in 3 bits 56.0 and 67.8; 20000 rows of 640 7.6 and 9.7.  STREAM: calls of more than 2^21 pieces (32
// MiB), whose rows are hardly in the caches.  Others ask for a group's four pieces per lane, which share lines, so through the
// cache: 20000 rows of 640 8.4 us the other way; 262144 rows of 512 this way 63.6, non-temporal 80.
// far: more than 160 MiB of packed rows, which do not stay in the last level either, pass by the caches too: 1048576 rows of 512 in 4 bits
// 247 -> 237 us (a lane per piece 239), 524288 the same either way, 300000 66 -> 69; in 3 bits 600000 rows of 768 206 -> 198, 550000 of 512 (134 MiB)
// 113 -> 120.
template <int BITS, bool STAGED, bool STREAM>
__global__ __launch_bounds__(256) void quantize_groups_kernel(const bf16_t *__restrict__ X, unsigned char *__restrict__ out, long long groups, int r, int far)
{
    __shared__ q_u32x4_t pieces[STREAM ? 1024 : STAGED ? 512 : 1];
    unsigned char *stage = reinterpret_cast<unsigned char *>(pieces);  // STAGED
    const uint32_t gpr = (uint32_t)r >> 5, most = STAGED ? 256 / gpr * gpr : 256;  // groups per row, of this workgroup
    const long long first = (long long)blockIdx.x * most, row0 = first / gpr;
    const uint32_t g0 = STAGED ? 0u : (uint32_t)(first - row0 * gpr);
    const uint32_t left = groups - first < most ? (uint32_t)(groups - first) : most;
    const uint32_t pitch = (uint32_t)quant_row_bytes(r, BITS);
    unsigned char *og = out + row0 * (long long)pitch;
    auto put = [&](uint32_t o, auto v) __attribute__((always_inline)) {
        if constexpr (STAGED)
            *reinterpret_cast<decltype(v) *>(stage + o) = v;
        else
            *reinterpret_cast<decltype(v) *>(og + o) = v;
    };
    const uint32_t i = threadIdx.x;
    const q_u32x4_t *src = reinterpret_cast<const q_u32x4_t *>(X) + 4 * first;
    q_u32x4_t raw[4];
    if constexpr (STREAM) {
        // the rows come in as they lie, 16 bytes a lane and past the caches, and change hands in LDS: piece p of group g in place 4 g +
        // (p ^ (g / 4 % 4)), which neither side finds on a busy bank
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t p = 256 * u + i;
            raw[u] = __builtin_nontemporal_load(src + (p < 4 * left ? p : 0u));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t p = 256 * u + i, g = p >> 2;
            pieces[4 * g + ((p & 3) ^ ((g >> 2) & 3))] = raw[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) raw[u] = pieces[4 * i + (u ^ ((i >> 2) & 3))];
        if constexpr (STAGED) __syncthreads();  // (the same room for what leaves)
    } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) raw[u] = src[4 * (i < left ? i : 0u) + u];
    }
    if (i < left) {
        float lo, hi;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float x[8];
            unpack8(raw[u], x);
            lo = u == 0 ? min3(x[0], x[1], x[1]) : min3(lo, x[0], x[1]);
            hi = u == 0 ? max3(x[0], x[1], x[1]) : max3(hi, x[0], x[1]);
#pragma unroll
            for (int e = 2; e < 8; e += 2) lo = min3(lo, x[e], x[e + 1]), hi = max3(hi, x[e], x[e + 1]);
        }
        float step, inv;
        group_scale<BITS>(lo, hi, step, inv);
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float x[8];
            unpack8(raw[u], x);
            w[u] = eight_codes<BITS>(x, lo, inv);
        }
        const uint32_t row = (g0 + i) / gpr, g = g0 + i - row * gpr, at = row * pitch, par = group_params(step, lo);
        if constexpr (BITS == 3) {  // four units of 24 bits, then the parameters
            put(at + 16 * g, q_u32x4_t{w[0] | (w[1] << 24), (w[1] >> 8) | (w[2] << 16), (w[2] >> 16) | (w[3] << 8), par});
        } else {
            put(at + 16 * g, q_u32x4_t{w[0], w[1], w[2], w[3]});
            put(at + ((uint32_t)r >> 1) + 4 * g, par);
            if (g == 0)  // the row's padding
                for (uint32_t o = ((uint32_t)r >> 1) + ((uint32_t)r >> 3); o < pitch; o += 4) put(at + o, 0u);
        }
    }
    if constexpr (STAGED) {
        __syncthreads();
        const uint32_t n16 = left / gpr * pitch / 16;
        q_u32x4_t *to = reinterpret_cast<q_u32x4_t *>(og);
        if (STREAM && far)
            for (uint32_t j = threadIdx.x; j < n16; j += 256) __builtin_nontemporal_store(reinterpret_cast<const q_u32x4_t *>(stage)[j], to + j);
        else
            for (uint32_t j = threadIdx.x; j < n16; j += 256) to[j] = reinterpret_cast<const q_u32x4_t *>(stage)[j];
    }
}

// Small calls: a lane per 16-byte piece (8 ranks); the four lanes of a group share min and max through two exchanges, and every lane
// stores its own word.
template <int BITS>
__global__ __launch_bounds__(256) void quantize_pieces_kernel(const bf16_t *__restrict__ X, unsigned char *__restrict__ out, long long pieces, int r)
{
    const uint32_t ppr = (uint32_t)r >> 3;  // pieces per row
    const long long first = (long long)blockIdx.x * 256, row0 = first / ppr;
    const uint32_t pc0 = (uint32_t)(first - row0 * ppr);
    const uint32_t left = pieces - first < 256 ? (uint32_t)(pieces - first) : 256u;
    const uint32_t pitch = (uint32_t)quant_row_bytes(r, BITS);
    // pieces is a multiple of 4 (r % 32 == 0), so a group's four lanes are all inside or all outside
    const uint32_t i = threadIdx.x, lrow = (pc0 + i) / ppr;
    const q_u32x4_t raw = reinterpret_cast<const q_u32x4_t *>(X)[first + (i < left ? i : left - 1)];  // (may still be in the caches)
    unsigned char *og = out + row0 * (long long)pitch;
    uint32_t pc = pc0 + i - lrow * ppr, orow = lrow * pitch;
    asm volatile("" : "+v"(pc), "+v"(orow));  // (while the piece is on its way, not before the store)
    __builtin_amdgcn_sched_barrier(0);
    float x[8];
    unpack8(raw, x);
    const float mn = min3(min3(x[0], x[1], x[2]), min3(x[3], x[4], x[5]), min3(x[6], x[7], x[7]));
    const float mx = max3(max3(x[0], x[1], x[2]), max3(x[3], x[4], x[5]), max3(x[6], x[7], x[7]));
    // the group's other three lanes: 1 0 3 2, 2 3 0 1, 3 2 1 0
    const float mn1 = __uint_as_float(quad_perm<0xB1>(__float_as_uint(mn))), mx1 = __uint_as_float(quad_perm<0xB1>(__float_as_uint(mx)));
    const float lo0 = min3(mn, mn1, mn1), hi0 = max3(mx, mx1, mx1);
    const float mn2 = __uint_as_float(quad_perm<0x4E>(__float_as_uint(lo0))), mx2 = __uint_as_float(quad_perm<0x4E>(__float_as_uint(hi0)));
    const float lo = min3(lo0, mn2, mn2), hi = max3(hi0, mx2, mx2);  // bf16 values
    float step, inv;
    group_scale<BITS>(lo, hi, step, inv);
    const uint32_t word = eight_codes<BITS>(x, lo, inv), par = group_params(step, lo);
    if constexpr (BITS == 3) {
        // the group's four 24-bit units into three words; the group's first lane writes the 16-byte piece
        const uint32_t u1 = quad_perm<0x55>(word), u2 = quad_perm<0xAA>(word), u3 = quad_perm<0xFF>(word);
        if (i < left && (pc & 3) == 0)
            *reinterpret_cast<q_u32x4_t *>(og + (orow + 4 * pc)) = q_u32x4_t{word | (u1 << 24), (u1 >> 8) | (u2 << 16), (u2 >> 16) | (u3 << 8), par};
    } else if (i < left) {
        *reinterpret_cast<uint32_t *>(og + (orow + 4 * pc)) = word;
        if ((pc & 3) == 0) *reinterpret_cast<uint32_t *>(og + (orow + ((uint32_t)r >> 1) + pc)) = par;
        if (pc == 0)  // the row's padding
            for (uint32_t o = ((uint32_t)r >> 1) + ((uint32_t)r >> 3); o < pitch; o += 4) *reinterpret_cast<uint32_t *>(og + (orow + o)) = 0u;
    }
}

hipError_t launch_quantize_rows(const void *X, long long rows, int r, int bits, void *out, hipStream_t st)
{
    const long long groups = rows * (long long)(r >> 5), pieces = 4 * groups;
    if (groups == 0) return hipSuccess;
    // A small call is one round of loads: its pieces are spread over four times as many lanes, which is the faster where the rows come from
    // memory (a lane per group then waits for four requests of parts of lines) and the slower where they are in the caches.  The line is where
    // the sums of both are the same.  Lane per piece / per group, us, rows of 512 in 4 bits: 4200 in the caches 2.87 / 2.96, from
    // memory 3.5 / 4.0; 5700 3.14 / 3.07 and 3.89 / 4.29; 6700 (418 K pieces) 3.40 / 3.11 and 4.14 / 4.42; 8200 3.64 / 3.28 and 4.56 / 4.66;
    // 9000 3.85 / 3.53 and 5.35 / 5.04.
    const bool small = pieces <= kQuantSmall, staged = (r >> 5) <= 256;
    const long long most = small ? 256 : staged ? 256 / (r >> 5) * (r >> 5) : 256, blocks = ((small ? pieces : groups) + most - 1) / most;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    auto launch_with = [&](auto kernel, auto... args) { hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const bf16_t *)X, (unsigned char *)out, args...); };
    auto launch = [&](auto kernel) { launch_with(kernel, groups, r, (int)(rows * (long long)quant_row_bytes(r, bits) > kQuantFar)); };
    if (small)
        bits == 3 ? launch_with(quantize_pieces_kernel<3>, pieces, r) : launch_with(quantize_pieces_kernel<4>, pieces, r);
    else if (pieces <= kQuantCached)
        if (bits == 3)
            staged ? launch(quantize_groups_kernel<3, true, false>) : launch(quantize_groups_kernel<3, false, false>);
        else
            staged ? launch(quantize_groups_kernel<4, true, false>) : launch(quantize_groups_kernel<4, false, false>);
    else if (bits == 3)
        staged ? launch(quantize_groups_kernel<3, true, true>) : launch(quantize_groups_kernel<3, false, true>);
    else
        staged ? launch(quantize_groups_kernel<4, true, true>) : launch(quantize_groups_kernel<4, false, true>);
    return hipGetLastError();
}

}  // namespace xkv
