// Dense reconstruction X^_l = A B_l for all L tokens (Sec. 3.2), written head-major
// [batch][H_kv][L][d_h].  Builds the uncompressed cache the dense baseline reads.
#include "xkv_common.h"

namespace xkv {

// 64 x 64 output tile per workgroup, 4 x 4 outputs per thread, rank walked 16 at a time via LDS.
template <typename T>
__global__ __launch_bounds__(256) void reconstruct_kernel(const T *__restrict__ A,  // [batch][L][r]
                                                          const T *__restrict__ B,  // [batch][G][r][d]
                                                          T *__restrict__ X,        // [batch][H_kv][L][d_h]
                                                          int G, int layer, int L, int r, int H_kv, int d_h)
{
    __shared__ float sA[16][64 + 1];
    __shared__ float sB[16][64 + 1];
    const int b = blockIdx.z, d = H_kv * d_h;
    const int t0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
    const int tx = threadIdx.x % 16, ty = threadIdx.x / 16;
    const T *Ab = A + (size_t)b * L * r;
    const T *Bb = B + ((size_t)b * G + layer) * r * d;
    float acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = 0.0f;

    for (int i0 = 0; i0 < r; i0 += 16) {
        for (int e = threadIdx.x; e < 64 * 16; e += 256) {
            const int tt = e / 16, ii = e % 16;  // A tile: consecutive threads read along the rank
            const int t = t0 + tt, i = i0 + ii;
            sA[ii][tt] = (t < L && i < r) ? to_f32(Ab[(size_t)t * r + i]) : 0.0f;
            const int i2 = e / 64, cc = e % 64;  // B tile: consecutive threads read along the columns
            const int ib = i0 + i2, c = c0 + cc;
            sB[i2][cc] = (ib < r && c < d) ? to_f32(Bb[(size_t)ib * d + c]) : 0.0f;
        }
        __syncthreads();
#pragma unroll
        for (int ii = 0; ii < 16; ++ii) {
            float av[4], bv[4];
#pragma unroll
            for (int a = 0; a < 4; ++a) av[a] = sA[ii][ty * 4 + a];
#pragma unroll
            for (int c = 0; c < 4; ++c) bv[c] = sB[ii][tx * 4 + c];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[a][c] = fmaf(av[a], bv[c], acc[a][c]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int t = t0 + ty * 4 + a;
        if (t >= L) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int col = c0 + tx * 4 + c;
            if (col >= d) continue;
            const int g = col / d_h, j = col % d_h;
            X[(((size_t)b * H_kv + g) * L + t) * d_h + j] = from_f32<T>(acc[a][c]);
        }
    }
}

// ==========================================================================================
// bf16 matrix-core path (d_h = 128, rank a multiple of 16) on v_mfma_f32_32x32x16_bf16.  A workgroup of 4 wavefronts owns
// 128 tokens x 256 dims (two KV heads); a wavefront takes all of its tokens and 64 of the dims, so that a step of 16 ranks
// is 4 + 2 operand reads from LDS for 8 products.  The rank is walked in slabs of 32 that go global -> LDS directly, three
// stages, two slabs ahead; 72 KiB, so that two workgroups share a compute unit and one multiplies while the other
// starts or writes its result.
//  - A slab [128 tokens][4 pieces of 8 ranks]: piece p of token t in place p ^ (t / 4 % 4);
//  - B slab [32 ranks][32 pieces of 8 dims]: piece p of rank i in place p ^ 4 (i % 4), row by row as it lies in memory; the
//    products want the ranks contiguous per lane, which the transposing LDS read does (ds_read_b64_tr_b16);
//  - result rounded to bf16 once, staged in LDS, written as whole 128 B lines.
// All three without bank conflicts in what the LDS serves at a time.  Token tiles, counted over all sequences, go to the dies
// in turn, the column tiles of a token tile to the same die (its rows of A are read once from memory).  (With every
// sequence beginning at the first die 16 of 256 tokens kept two of the eight busy: 23.4 us, now 14.6; 64 of 100 tokens,
// rank 128, 33.5 us, now 8.0.)
// What bounds it: the copies into LDS (24 KiB per slab and workgroup, 403 MB from L2 at 8.5 TB/s) before the products:
// 47 us at L = 32768, r = 512, H_kv = 8 (34 GFLOP, 0.73 PFLOP/s; the products alone are 14 us, memory 18 us).  Eight wavefronts
// of 32 tokens x 128 dims, every wavefront reading all of B_l's fragments for its 32 tokens and B_l transposed by 2 B
// stores, took 64 us, bound by LDS and by A read once per head.
// ==========================================================================================
typedef __attribute__((ext_vector_type(8))) __bf16 rc_bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short rc_s16x4_t;
typedef __attribute__((ext_vector_type(8))) short rc_s16x8_t;
typedef __attribute__((ext_vector_type(16))) float rc_f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t rc_u32x4_t;
typedef __attribute__((address_space(3))) rc_s16x4_t rc_lds_s16x4_t;

constexpr int kRcThreads = 256, kRcTok = 128, kRcDims = 256, kRcSlab = 32, kRcStages = 3;
constexpr int kRcLdsA = kRcTok * kRcSlab * 2, kRcLdsB = kRcSlab * kRcDims * 2, kRcStage = kRcLdsA + kRcLdsB;
constexpr int kRcLds = kRcStages * kRcStage;
static_assert(kRcLds >= kRcTok * kRcDims * 2, "the result is staged where the slabs were");

__global__ __launch_bounds__(kRcThreads, 2) void reconstruct_mfma_kernel(const bf16_t *__restrict__ A,
                                                                        const bf16_t *__restrict__ B,
                                                                        bf16_t *__restrict__ X, int G, int layer,
                                                                        int L, int r, int H_kv, int col_tiles,
                                                                        int tok_tiles, int batch)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char rc_smem[];
    const int d = H_kv * 128, grp = (int)(blockIdx.x >> 3) / col_tiles, col_tile = (int)(blockIdx.x >> 3) - grp * col_tiles;
    const int tile = (int)(blockIdx.x & 7) + 8 * grp, b = __builtin_amdgcn_readfirstlane(tile / tok_tiles);
    if (b >= batch) return;  // (the grid counts token tiles in eights)
    const int t0 = (tile - b * tok_tiles) * kRcTok, c0 = col_tile * kRcDims;
    const int lane = lane_id(), w = wave_id(), n = lane & 31, hf = lane >> 5;
    const unsigned char *Ab = reinterpret_cast<const unsigned char *>(A + (size_t)b * L * r);
    const unsigned char *Bb = reinterpret_cast<const unsigned char *>(B + ((size_t)b * G + layer) * (size_t)r * d);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)rc_smem;

    // copies of a slab: a wavefront brings 32 tokens of A (2 instructions of 16 rows x 4 pieces) and 8 ranks of B
    // (4 instructions of 2 rows x 32 pieces).  Tokens, ranks and columns beyond the matrix: the last ones again (their
    // results are not stored, the ranks not multiplied).
    const unsigned char *ap[2];
    int apc[2], bcol[4], brow[4];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int t = 32 * w + 16 * j + (lane >> 2);
        ap[j] = Ab + (size_t)(t0 + t < L ? t0 + t : L - 1) * r * 2;
        apc[j] = (lane & 3) ^ ((t >> 2) & 3);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        brow[j] = 8 * w + 2 * j + (lane >> 5);
        const int c = c0 + 8 * ((lane & 31) ^ ((brow[j] & 3) << 2));
        bcol[j] = (c < d ? c : d - 8) * 2;
    }
    auto issue = [&](int s) __attribute__((always_inline)) {
        const uint32_t st = lds0 + (uint32_t)(s % kRcStages) * kRcStage;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int at = kRcSlab * s + 8 * apc[j];
            copy16_global_to_lds(ap[j] + (at < r ? at : r - 8) * 2, __builtin_amdgcn_readfirstlane(st + (2 * w + j) * 1024));
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = kRcSlab * s + brow[j];
            copy16_global_to_lds(Bb + (size_t)(i < r ? i : r - 1) * d * 2 + bcol[j],
                                    __builtin_amdgcn_readfirstlane(st + kRcLdsA + (4 * w + j) * 1024));
        }
    };

    // operand reads: A, row = token n of block tt, piece 2 f + hf; B, transposed, lanes of 16: 16 dims, ranks
    // 16 f + 8 hf + 4 h .. + 3 (lane / 4 % 4 the rank, lane % 4 the four dims it asks for)
    const int a_at = n * 64, ax = (n >> 2) & 3;
    const int b_row = 8 * hf + ((lane >> 2) & 3), b_c4 = 64 * w + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);  // first of four dims
    int b_at[2];
#pragma unroll
    for (int dd = 0; dd < 2; ++dd)  // (the rank modulo 4, which the place depends on, is the same in all four reads)
        b_at[dd] = b_row * 512 + ((((b_c4 + 32 * dd) >> 3) ^ ((b_row & 3) << 2)) << 4) + ((b_c4 & 4) << 1);

    rc_f32x16_t acc[4][2];
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int dd = 0; dd < 2; ++dd)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[tt][dd][v] = 0.0f;

    auto step = [&](const unsigned char *st, int f) __attribute__((always_inline)) {
        rc_bf16x8_t af[4], bf[2];
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
            af[tt] = *reinterpret_cast<const rc_bf16x8_t *>(st + tt * 2048 + a_at + (((2 * f + hf) ^ ax) << 4));
#pragma unroll
        for (int dd = 0; dd < 2; ++dd) {
            const unsigned char *q = st + kRcLdsA + f * 8192 + b_at[dd];
            const rc_s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rc_lds_s16x4_t *)q);
            const rc_s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rc_lds_s16x4_t *)(q + 2048));
            bf[dd] = __builtin_bit_cast(rc_bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
            for (int dd = 0; dd < 2; ++dd)
                acc[tt][dd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[dd], af[tt], acc[tt][dd], 0, 0, 0);  // rows dims, columns tokens
    };

    const int n_slabs = (r + kRcSlab - 1) / kRcSlab;
    issue(0);
    if (n_slabs > 1) issue(1);
    for (int s = 0; s < n_slabs; ++s) {
        if (s + 1 < n_slabs)
            XKV_WAIT_VMCNT(6);  // slab s is there, slab s + 1 may be on its way
        else
            XKV_WAIT_VMCNT(0);
        lds_barrier();  // ... for every wavefront, and nobody reads slab s - 1 any more
        if (s + 2 < n_slabs) issue(s + 2);
        const unsigned char *st = rc_smem + (s % kRcStages) * kRcStage;
        step(st, 0);
        if (kRcSlab * s + 16 < r) step(st, 1);
    }

    // lane (token n, hf) holds dims 32 dd + 8 (v / 4) + 4 hf + v % 4.  Round once, stage [128 tokens][8 pieces of 8 dims] per
    // wavefront, piece p of token t in place p ^ (t / 2 % 8), store whole lines
    lds_barrier();
    unsigned char *ot = rc_smem + w * (kRcTok * 128);
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int dd = 0; dd < 2; ++dd)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                uint2 pk;
                pk.x = (uint32_t)f32_to_bf16(acc[tt][dd][4 * q4 + 0]) | ((uint32_t)f32_to_bf16(acc[tt][dd][4 * q4 + 1]) << 16);
                pk.y = (uint32_t)f32_to_bf16(acc[tt][dd][4 * q4 + 2]) | ((uint32_t)f32_to_bf16(acc[tt][dd][4 * q4 + 3]) << 16);
                *reinterpret_cast<uint2 *>(ot + (32 * tt + n) * 128 + (((4 * dd + q4) ^ ((n >> 1) & 7)) << 4) + 8 * hf) = pk;
            }
    const int col = c0 + 64 * w;  // first dim of this wavefront
    if (col >= d) return;         // (an odd number of KV heads)
    bf16_t *Xg = X + (((size_t)b * H_kv + (col >> 7)) * L + t0) * 128 + (col & 64);
#pragma unroll 4
    for (int j = 0; j < 16; ++j) {
        const int t = 8 * j + (lane >> 3), pc = lane & 7;
        const rc_u32x4_t val = *reinterpret_cast<const rc_u32x4_t *>(ot + t * 128 + ((pc ^ ((t >> 1) & 7)) << 4));
        if (t0 + t < L) *reinterpret_cast<rc_u32x4_t *>(Xg + (size_t)t * 128 + 8 * pc) = val;
    }
}

static bool reconstruct_mfma_ok(const xkv_shape &s, int r, const void *A, const void *B, const void *X)
{
    return s.dtype == XKV_BF16 && s.d_h == 128 && r % 16 == 0 && r >= 16 &&
           ((((uintptr_t)A | (uintptr_t)B | (uintptr_t)X)) & 15u) == 0;
}

hipError_t launch_reconstruct(const xkv_shape &s, int layer, const void *A, const void *B, int r, void *X,
                              hipStream_t st)
{
    if (reconstruct_mfma_ok(s, r, A, B, X)) {
        static DynamicLdsOnce attr;
        if (hipError_t e0 = attr.ensure((const void *)reconstruct_mfma_kernel, kRcLds); e0 != hipSuccess) return e0;
        const int tok_tiles = (s.L + kRcTok - 1) / kRcTok, col_tiles = (s.H_kv * 128 + kRcDims - 1) / kRcDims;
        const long long tiles = ((long long)tok_tiles * s.batch + 7) / 8 * 8 * col_tiles;
        hipLaunchKernelGGL(reconstruct_mfma_kernel, dim3((unsigned)tiles), dim3(kRcThreads), kRcLds, st, (const bf16_t *)A,
                           (const bf16_t *)B, (bf16_t *)X, s.G, layer, s.L, r, s.H_kv, col_tiles, tok_tiles, s.batch);
        return hipGetLastError();
    }
    const int d = s.H_kv * s.d_h;
    dim3 grid((d + 63) / 64, (s.L + 63) / 64, s.batch), block(256);
    if (s.dtype == XKV_F32)
        hipLaunchKernelGGL(reconstruct_kernel<float>, grid, block, 0, st, (const float *)A, (const float *)B,
                           (float *)X, s.G, layer, s.L, r, s.H_kv, s.d_h);
    else
        hipLaunchKernelGGL(reconstruct_kernel<bf16_t>, grid, block, 0, st, (const bf16_t *)A, (const bf16_t *)B,
                           (bf16_t *)X, s.G, layer, s.L, r, s.H_kv, s.d_h);
    return hipGetLastError();
}

}  // namespace xkv
