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

constexpr int kQuantPieces = 4;         // 16-byte pieces per thread (1 where the call is small)
constexpr int kQuantSmall = 1536 * 1024;  // pieces

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

// One lane per 16-byte piece (8 ranks); the four lanes of a group share min and max through two exchanges.  A
// workgroup takes whole rows, as many as 256 U pieces hold, collects the quantised rows in LDS and writes them as
// one run of 16-byte pieces; with rows longer than that (STAGED false) every lane stores its own word.
// The row stream and the vector ALU take about the same time, so: a thread of a large call has kQuantPieces requests in flight; rows and
// offsets are 32-bit numbers from the workgroup's first row (a 64-bit division per piece took longer than the
// quantisation), exchanges are lane permutations on the ALU, clamping is one median, two codes meet in a multiply-add before they
// become a byte.  The two quotients take a product and a correction each: with y the rounded reciprocal of b, q = a y and
// r = a - b q (exact), q + r y is the rounded a / b; a reciprocal one unit off is corrected the same way unless all
// 24 bits of b are ones, and a step has 8 (Markstein, IBM J. Res. Dev. 34, 1990).  Outside the range where r is exact the
// ordinary division is used.  50001 rows of 512: 17.6 -> 15.2 us (67 MB; reading and writing as many bytes alone 11.5; with a
// store of a word per lane and one for the parameters 16.3: rows of 320 bytes leave most lines in parts).
template <int BITS, bool STAGED, int U>
__global__ __launch_bounds__(256) void quantize_rows_kernel(const bf16_t *__restrict__ X, unsigned char *__restrict__ out,
                                                            long long pieces, int r)
{
    constexpr int kBlock = 256 * U;  // pieces of a workgroup: kBlock / (r / 8) rows of at most 5 r / 8 + 12 bytes
    __shared__ __attribute__((aligned(16))) unsigned char stage[STAGED ? 8 * kBlock : 16];
    constexpr float kQmax = (float)((1 << BITS) - 1), kQinv = 1.0f / kQmax;
    constexpr uint32_t kSmall = 0x20000000u, kLarge = 0x5F000000u;  // 2^-63, 2^63
    const uint32_t ppr = (uint32_t)r >> 3;  // pieces per row
    const uint32_t most = STAGED ? kBlock / ppr * ppr : kBlock;  // pieces of this workgroup
    const long long first = (long long)blockIdx.x * most, row0 = first / ppr;
    const uint32_t pc0 = STAGED ? 0u : (uint32_t)(first - row0 * ppr);
    const uint32_t left = pieces - first < most ? (uint32_t)(pieces - first) : most;
    const uint32_t pitch = BITS == 3 ? (uint32_t)r >> 1 : (uint32_t)quant_row_bytes(r);
    const q_u32x4_t *Xb = reinterpret_cast<const q_u32x4_t *>(X) + first;
    unsigned char *og = out + row0 * (long long)pitch;
    auto put = [&](uint32_t o, auto v) __attribute__((always_inline)) {
        if constexpr (STAGED)
            *reinterpret_cast<decltype(v) *>(stage + o) = v;
        else
            *reinterpret_cast<decltype(v) *>(og + o) = v;
    };
    // pieces is a multiple of 4 (r % 32 == 0), so a group's four lanes are all inside or all outside
    q_u32x4_t raw[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = u * 256 + threadIdx.x;
        const q_u32x4_t *src = Xb + (i < left ? i : left - 1);
        raw[u] = U == 1 ? *src : __builtin_nontemporal_load(src);  // (a small call's rows may still be in the caches)
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint32_t i = u * 256 + threadIdx.x, lrow = (pc0 + i) / ppr, pc = pc0 + i - lrow * ppr;
        const bool in = i < left;
        float x[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[2 * e] = __uint_as_float(raw[u][e] << 16);
            x[2 * e + 1] = __uint_as_float(raw[u][e] & 0xFFFF0000u);
        }
        float mn = min3(min3(x[0], x[1], x[2]), min3(x[3], x[4], x[5]), min3(x[6], x[7], x[7]));
        float mx = max3(max3(x[0], x[1], x[2]), max3(x[3], x[4], x[5]), max3(x[6], x[7], x[7]));
        // the group's other three lanes: 1 0 3 2, 2 3 0 1, 3 2 1 0
        const float mn1 = __uint_as_float(quad_perm<0xB1>(__float_as_uint(mn))), mx1 = __uint_as_float(quad_perm<0xB1>(__float_as_uint(mx)));
        const float lo0 = min3(mn, mn1, mn1), hi0 = max3(mx, mx1, mx1);
        const float mn2 = __uint_as_float(quad_perm<0x4E>(__float_as_uint(lo0))), mx2 = __uint_as_float(quad_perm<0x4E>(__float_as_uint(hi0)));
        const float lo = min3(lo0, mn2, mn2), hi = max3(hi0, mx2, mx2);  // bf16 values
        const float range = hi - lo;
        float q = range * kQinv;
        q = fmaf(fmaf(-kQmax, q, range), kQinv, q);
        if (__float_as_uint(range) - kSmall > kLarge - kSmall && range != 0.0f) q = range / kQmax;
        float step = bf16_to_f32(f32_to_bf16(q));
        step = step > 0.0f ? step : 1.0f;
        float inv = __builtin_amdgcn_rcpf(step);
        inv = fmaf(fmaf(-step, inv, 1.0f), inv, inv);
        if (__float_as_uint(step) - kSmall > kLarge - kSmall) inv = 1.0f / step;
        float c[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) c[e] = __builtin_amdgcn_fmed3f(rintf((x[e] - lo) * inv), 0.0f, kQmax);
        // even ranks in the low half, odd ranks in the high half (16 bits up for 4-bit codes, 12 for 3-bit codes)
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
        const uint32_t par = (__float_as_uint(step) >> 16) | __float_as_uint(lo);  // (both have empty low halves)
        const uint32_t orow = lrow * pitch;
        if constexpr (BITS == 3) {
            // the group's four 24-bit units into three words; the group's first lane writes the 16-byte piece
            const uint32_t u1 = quad_perm<0x55>(word), u2 = quad_perm<0xAA>(word), u3 = quad_perm<0xFF>(word);
            q_u32x4_t piece;
            piece[0] = word | (u1 << 24);
            piece[1] = (u1 >> 8) | (u2 << 16);
            piece[2] = (u2 >> 16) | (u3 << 8);
            piece[3] = par;
            if (in && (pc & 3) == 0) put(orow + 4 * pc, piece);
        } else if (in) {
            put(orow + 4 * pc, word);
            if ((pc & 3) == 0) put(orow + ((uint32_t)r >> 1) + pc, par);
            if (pc == 0)  // the row's padding
                for (uint32_t o = ((uint32_t)r >> 1) + ((uint32_t)r >> 3); o < pitch; o += 4) put(orow + o, 0u);
        }
    }
    if constexpr (STAGED) {
        __syncthreads();
        const uint32_t n16 = left / ppr * pitch / 16;
        for (uint32_t i = threadIdx.x; i < n16; i += 256)
            reinterpret_cast<q_u32x4_t *>(og)[i] = reinterpret_cast<const q_u32x4_t *>(stage)[i];
    }
}

hipError_t launch_quantize_rows(const void *X, long long rows, int r, int bits, void *out, hipStream_t st)
{
    const int ppr = r >> 3;
    const long long pieces = rows * (long long)ppr;
    if (pieces == 0) return hipSuccess;
    // A small call is one round of loads and stores: its pieces are spread over as many workgroups as there are, and stored as they
    // come (two calls, their landmarks and selection, us: 4100 rows of 512, four pieces a thread 26.8, one 25.3; 12000 of 768 28.2
    // and 27.0; 20000 of 640 37.0 with four and 39.4 with one and 64-bit row numbers).
    const bool small = pieces <= kQuantSmall;
    const int block = 256 * (small ? 1 : kQuantPieces);
    const bool staged = !small && ppr <= block;
    const long long most = staged ? block / ppr * ppr : block, blocks = (pieces + most - 1) / most;
    if (blocks > 0x7FFFFFFFLL) return hipErrorInvalidValue;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const bf16_t *)X, (unsigned char *)out, pieces, r);
    };
    if (bits == 3)
        small ? launch(quantize_rows_kernel<3, false, 1>)
              : staged ? launch(quantize_rows_kernel<3, true, kQuantPieces>) : launch(quantize_rows_kernel<3, false, kQuantPieces>);
    else
        small ? launch(quantize_rows_kernel<4, false, 1>)
              : staged ? launch(quantize_rows_kernel<4, true, kQuantPieces>) : launch(quantize_rows_kernel<4, false, kQuantPieces>);
    return hipGetLastError();
}

}  // namespace xkv
