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
// Takes the calls that reconstruct_kept_kernel does not (reconstruct_keeps_factor).  What bounds it: the copies into LDS (24 KiB per slab and workgroup, at ranks
// 512 403 MB from L2 at 8.5 TB/s) before the products: 47 us there at L = 32768, H_kv = 8 (34 GFLOP, 0.73 PFLOP/s).  Eight wavefronts
// of 32 tokens x 128 dims, every wavefront reading all of B_l's fragments for its 32 tokens and B_l transposed by 2 B
// stores, took 64 us, bound by LDS and by A read once per head.
// ==========================================================================================
typedef __attribute__((ext_vector_type(8))) __bf16 rc_bf16x8_t;
typedef __attribute__((ext_vector_type(4))) short rc_s16x4_t;
typedef __attribute__((ext_vector_type(8))) short rc_s16x8_t;
typedef __attribute__((ext_vector_type(16))) float rc_f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t rc_u32x4_t;
typedef __attribute__((ext_vector_type(2))) __bf16 rc_bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float rc_f32x2_t;
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

// ==========================================================================================
// Multiples of 128 ranks up to 768, few or long sequences: the factor B_l stays in registers.  A wavefront holds 64 dims of all ranks as operands (256
// registers at 512 ranks) and walks a run of tokens, 32 at a time; four wavefronts, 256 dims, share the rows of A, which go global -> LDS
// directly, whole rows.  Four tiles are live: the one that is multiplied, the next (landed, so that its first operands are read ahead of
// the barrier) and two on their way; above 512 ranks, where the LDS holds three, one.  An operand read of A feeds two
// products, and nothing of B_l is read again: 1 + 4 KiB of LDS traffic per token and 256 dims at 512 ranks instead of 12.
//  - A tile [32 tokens][r / 8 pieces of 8 ranks]: piece p of token t in place p ^ (t % 16);
//  - B_l passes through the same room once, in slabs laid out as above, with the first tiles of A behind it;
//  - the result of a tile is rounded and stored while the next one is multiplied, where there are registers for two tiles of sums or a
//    second workgroup on the compute unit (ranks up to 256), which multiplies meanwhile.
// The runs of a sequence cover its tokens evenly, one workgroup (or two) per compute unit; each die takes a contiguous part of the list
// (sequence, run, 256 dims), so that rows of A and B_l are read once into its L2 (64 x 512 tokens of two heads 24.2 -> 15.7 us).
// What bounds it: the matrix cores at the clock that they run at under load, then the stores.  L = 32768, H_kv = 8, ranks 512: 37 us (0.93
// PFLOP/s; 47 before), of which start and B_l take 5; all numbers zero 30 us, without stores 35; four sequences 131 us (201; 1.05
// PFLOP/s, a large library product 1.25).  Ranks 128: 17.7 us (22.1), 256 22 (30), 384 30 (39), 640 49 (56), 768 54 (64); 64 tokens of
// ranks 512 6.1 (12.4).  Many short sequences: see reconstruct_keeps_factor.
// ==========================================================================================
constexpr int kRkTok = 32;
constexpr int rk_stages(int nf) { return nf <= 32 ? 4 : 3; }
constexpr bool rk_pair(int nf) { return nf <= 16; }  // two workgroups per compute unit

// All but the youngest `left` copies have landed.  (left: even, known once the loop around it is unrolled)
// (Any access more behind them, a register stored to scratch memory for instance, makes this wait longer, never too short.)
__device__ __forceinline__ void wait_copies(int left)
{
    switch (left) {
#define XKV_W(n) case n: XKV_WAIT_VMCNT(n); break;
    XKV_W(2) XKV_W(4) XKV_W(6) XKV_W(8) XKV_W(10) XKV_W(12) XKV_W(14) XKV_W(16) XKV_W(18) XKV_W(20) XKV_W(22) XKV_W(24) XKV_W(26) XKV_W(28) XKV_W(30) XKV_W(32)
#undef XKV_W
    default: XKV_WAIT_VMCNT(0);
    }
}

template <int NF> constexpr int rk_lds() { return rk_stages(NF) * kRkTok * NF * 32 + 4 * 4096; }

template <int NF>  // steps of 16 ranks
__global__ __launch_bounds__(256, rk_pair(NF) ? 2 : 1) void reconstruct_kept_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ B,
                                                                                 bf16_t *__restrict__ X, int G, int layer, int L, int H_kv,
                                                                                 int col_groups, int runs, int run_tiles, int total_runs, int per_die)
{
    constexpr bool AT_ONCE = NF <= 16 || NF > 32;  // registers are short; with two workgroups on a compute unit the other one multiplies meanwhile
    constexpr int r = NF * 16, NP = r / 8, NC = NP / 8, kTile = kRkTok * r * 2, kPutAt = AT_ONCE ? 0 : 8, RING = AT_ONCE ? 4 : 8, STAGES = rk_stages(NF);  // pieces of a row, copies per tile and wavefront
    extern __shared__ __attribute__((aligned(16))) unsigned char rc_smem[];
    const int unit = (int)(blockIdx.x & 7) * per_die + (int)(blockIdx.x >> 3), run_id = unit / col_groups, cg = unit - run_id * col_groups;
    if ((int)(blockIdx.x >> 3) >= per_die || run_id >= total_runs) return;
    const int b = __builtin_amdgcn_readfirstlane(run_id / runs), t_begin = (run_id - b * runs) * run_tiles * kRkTok, c0 = cg * kRcDims, d = H_kv * 128;
    const int left = (L - t_begin + kRkTok - 1) / kRkTok, nt = left < run_tiles ? left : run_tiles;
    const int lane = lane_id(), w = wave_id(), n = lane & 31, hf = lane >> 5;
    const unsigned char *Ab = reinterpret_cast<const unsigned char *>(A + (size_t)b * L * r);
    const unsigned char *Bb = reinterpret_cast<const unsigned char *>(B + ((size_t)b * G + layer) * (size_t)r * d);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)rc_smem;

    // ---- copies of a tile, NC per wavefront.  Rows beyond the sequence: the last one again
    auto copy = [&](int tile, int j) __attribute__((always_inline)) {
        int l = lane;
        if constexpr (NF > 32) asm volatile("" : "+v"(l));  // (computed each time: no registers for NC rows and bytes)
        const int e = 64 * (w * NC + j) + l, t = e / NP, row = t_begin + tile * kRkTok + t;
        copy16_global_to_lds(Ab + ((size_t)(row < L ? row : L - 1) * (r * 2) + 16 * ((e - t * NP) ^ (t & 15))),
                             __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(tile % STAGES) * kTile + (uint32_t)(w * NC + j) * 1024));
    };

    // ---- B_l into registers: slabs of 32 ranks, [rank][32 pieces of 8 dims], piece p of rank i in place p ^ 4 (i % 4), through RS places of
    // which the first tiles of A take over the last's
    rc_bf16x8_t bf[NF][2];
    {
        constexpr int NS = NF / 2, RS = STAGES * NF / 16;
        const int b_row = 8 * hf + ((lane >> 2) & 3), b_c4 = 64 * w + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        auto slab = [&](int sl) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {  // two ranks per copy
                const int i = 8 * w + 2 * j + hf, c = c0 + 8 * (n ^ ((i & 3) << 2));
                copy16_global_to_lds(Bb + (size_t)(32 * sl + i) * d * 2 + (c < d ? c : d - 8) * 2,
                                     __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(sl % RS) * 16384 + (uint32_t)(4 * w + j) * 1024));
            }
        };
        // (all these tiles also where the run is shorter: rows of the next run, not used)
        // step s: slab s - 1 is done with, and its place is filled: by slab s - 1 + RS, or by the tiles of A whose room is free
        auto tiles_after = [](int s) constexpr {
            int tile = 0;
            for (; tile < STAGES - 1; ++tile)
                for (int p = tile * kTile / 16384; p < RS && p * 16384 < (tile + 1) * kTile; ++p)
                    if (p + RS * ((NS - 1 - p) / RS) >= s) return tile;
            return tile;
        };
#pragma unroll
        for (int sl = 0; sl < RS; ++sl) slab(sl);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            // younger than slab s: the slabs and tiles that the steps before asked for
            const int last = s == 0 ? RS - 1 : s - 2 + RS < NS - 1 ? s - 2 + RS : NS - 1, tiles = s == 0 ? 0 : tiles_after(s - 1);
            wait_copies(4 * (last - s) + NC * tiles);
            lds_barrier();
            if (s > 0 && s - 1 + RS < NS) slab(s - 1 + RS);
            if (s > 0)
#pragma unroll
                for (int tile = tiles_after(s - 1); tile < tiles_after(s); ++tile)
#pragma unroll
                    for (int j = 0; j < NC; ++j) copy(tile, j);
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int dd = 0; dd < 2; ++dd) {
                    const unsigned char *q = rc_smem + (s % RS) * 16384 + f * 8192 + b_row * 512 + ((((b_c4 + 32 * dd) >> 3) ^ ((b_row & 3) << 2)) << 4) + ((b_c4 & 4) << 1);
                    const rc_s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rc_lds_s16x4_t *)q);
                    const rc_s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rc_lds_s16x4_t *)(q + 2048));
                    bf[2 * s + f][dd] = __builtin_bit_cast(rc_bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
        }
        lds_barrier();
#pragma unroll
        for (int tile = tiles_after(NS - 1); tile < STAGES - 1; ++tile)
#pragma unroll
            for (int j = 0; j < NC; ++j) copy(tile, j);
    }

    // operand of step f of the tile in `st`: ranks 16 f + 8 hf .. of token n.  The place differs from 2 f + hf in its low four bits
    const unsigned char *arow = rc_smem + n * (r * 2);
    const int ax = hf ^ (n & 15);
    auto a_frag = [&](const unsigned char *st, int f) __attribute__((always_inline)) {
        return *reinterpret_cast<const rc_bf16x8_t *>(st + ((f >> 3) << 8) + (((2 * f & 15) ^ ax) << 4));
    };
    const bool stores = c0 + 64 * w < d;  // (an odd number of KV heads)
    bf16_t *Xw = X + (((size_t)b * H_kv + (stores ? (c0 + 64 * w) >> 7 : 0)) * L + t_begin) * 128 + 64 * (w & 1);

    rc_bf16x8_t ring[RING];
    // A finished tile leaves through a wavefront-private image of 32 tokens x 8 pieces of 8 dims, piece p of token t in place p ^ (t % 8), so
    // that the stores write whole lines.  Lane (token n, hf) holds dims 32 dd + 8 (v / 4) + 4 hf + v % 4; the halves trade, so that each
    // lane has 8 dims in a row.  Step q of eight: four pieces in, four lines out.
    unsigned char *img = rc_smem + STAGES * kTile + w * 4096;
    auto put = [&](bf16_t *Xt, const rc_f32x16_t (&done)[2], int q, int rows) __attribute__((always_inline)) {
        if (q < 4) {
            const int dd = q >> 1, v0 = 8 * (q & 1);
            uint32_t pk[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const rc_bf16x2_t two = __builtin_convertvector((rc_f32x2_t{done[dd][v0 + 2 * u], done[dd][v0 + 2 * u + 1]}), rc_bf16x2_t);
                pk[u] = __builtin_bit_cast(uint32_t, two);
            }
            const auto x = __builtin_amdgcn_permlane32_swap(pk[0], pk[2], false, false), y = __builtin_amdgcn_permlane32_swap(pk[1], pk[3], false, false);
            *reinterpret_cast<rc_u32x4_t *>(img + n * 128 + (((2 * q + hf) ^ (n & 7)) << 4)) = rc_u32x4_t{x[0], y[0], x[1], y[1]};
        } else {
            const int t = 8 * (q - 4) + (lane >> 3), pc = lane & 7;
            const rc_u32x4_t val = *reinterpret_cast<const rc_u32x4_t *>(img + t * 128 + ((pc ^ (t & 7)) << 4));
            if (t < rows) *reinterpret_cast<rc_u32x4_t *>(Xt + t * 128 + 8 * pc) = val;
        }
    };
    // tile i: products into `now`; meanwhile the result of the tile before it, `last`, is rounded and stored
    auto body = [&](int i, rc_f32x16_t (&now)[2], const rc_f32x16_t (&last)[2]) __attribute__((always_inline)) {
        const unsigned char *st = arow + (i % STAGES) * kTile, *next = arow + ((i + 1) % STAGES) * kTile;
        bf16_t *Xt = Xw + (long long)(i - 1) * (kRkTok * 128);
        const int rows = i > 0 && stores ? L - t_begin - (i - 1) * kRkTok : 0;
#pragma unroll
        for (int dd = 0; dd < 2; ++dd)
#pragma unroll
            for (int v = 0; v < 16; ++v) now[dd][v] = 0.0f;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const rc_bf16x8_t a = ring[f % RING];
#pragma unroll
            for (int dd = 0; dd < 2; ++dd) now[dd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[f][dd], a, now[dd], 0, 0, 0);  // rows dims, columns tokens
            ring[f % RING] = f + RING < NF ? a_frag(st, f + RING) : a_frag(next, f + RING - NF);
            if ((!AT_ONCE && f < 4) || (f >= kPutAt && f < kPutAt + 4)) put(Xt, last, f < kPutAt ? f : f - kPutAt + 4, rows);
            constexpr int C0 = STAGES == 4 ? NF / 2 : 4;
            if (f >= C0 && f < C0 + NF / 2 && (f - C0) % 4 == 0 && i + STAGES - 1 < nt) {
                copy(i + STAGES - 1, (f - C0) / 2);
                copy(i + STAGES - 1, (f - C0) / 2 + 1);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (AT_ONCE) {
#pragma unroll
            for (int q = 0; q < 4; ++q) put(Xt, now, q, 0);
        }
    };
    // A barrier before each tile: tile i + 1 has landed for every wavefront, and nobody reads tile i - 1 any more, in whose room tile i + 3
    // goes.  The copies are the last vector-memory operations of a body: all but those of tile i + 2 are waited for.  (The operands
    // of tile i that are being read meanwhile need no wait here: those of tile i - 1 came back before them.)
    auto meet = [&](int i) __attribute__((always_inline)) {
        if (i + 2 < nt && STAGES == 4)
            XKV_WAIT_VMCNT(NC);
        else
            XKV_WAIT_VMCNT(0);
        asm volatile("" : : : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" : : : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    rc_f32x16_t acc[2][2];
#pragma unroll
    for (int dd = 0; dd < 2; ++dd)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[1][dd][v] = 0.0f;
    meet(0);
#pragma unroll
    for (int f = 0; f < RING; ++f) ring[f] = a_frag(arow, f);
    for (int i = 0;;) {  // (two tiles a round: which sums are meant is known at compile time)
        body(i, acc[0], acc[1]);
        if (++i == nt) {
            bf16_t *Xt = Xw + (long long)(nt - 1) * (kRkTok * 128);
#pragma unroll
            for (int q = AT_ONCE ? 4 : 0; q < 8; ++q) put(Xt, acc[0], q, stores ? L - t_begin - (nt - 1) * kRkTok : 0);
            break;
        }
        meet(i);
        body(i, acc[1], acc[0]);
        if (++i == nt) {
            bf16_t *Xt = Xw + (long long)(nt - 1) * (kRkTok * 128);
#pragma unroll
            for (int q = AT_ONCE ? 4 : 0; q < 8; ++q) put(Xt, acc[1], q, stores ? L - t_begin - (nt - 1) * kRkTok : 0);
            break;
        }
        meet(i);
    }
}

// How many runs a sequence is cut into: whole rounds of the chip, of which the one is taken that is done first; a workgroup's start, B_l
// from memory into registers, counts as `start` tiles.
static void reconstruct_cut(int tiles, long long groups, int slots, int start, int *runs, int *run_tiles)
{
    const long long first = (groups + slots - 1) / slots;
    long long best = 0;
    for (long long rounds = first; rounds < first + 4; ++rounds) {
        long long n = slots * rounds / groups;
        n = n < 1 ? 1 : n > tiles ? tiles : n;
        const int per = (int)((tiles + n - 1) / n), used = (tiles + per - 1) / per;
        const long long time = (groups * used + slots - 1) / slots * (per + start);
        if (best > 0 && time >= best) continue;
        best = time;
        *runs = used;
        *run_tiles = per;
    }
}

// Whether B_l in registers pays (r = 128, 256 .. 768).  With two workgroups on a compute unit, ranks up to 256, one multiplies while the
// other starts, and it does, but for factors that have one slab tile of 128 tokens each (more than 96, so that little of it is padding)
// and fill the chip with slab workgroups once: B_l kept / slabs, us, ranks 256, 64 sequences x 8 KV heads x 128 tokens 12.2 / 12.0, 128 of them
// 20.0 / 18.8, with 97 tokens 19.3 / 17.9, 129 x 4 x 128 16.5 / 14.8; but 56 x 8 x 128, 128 x 8 x 96 and x 129 the same or less, 130 x 8 x 97
// 22.4 / 22.2; ranks 128, 128 x 8 x 128 14.7 / 14.2, 112 of them 0.99.  Above, nothing goes on beside a workgroup's start, and many short
// sequences are mostly starts, each with a factor of its own from memory; the slabs' copies are bound by the same bytes there, but
// go on beside products.  Both times in tiles of 32 tokens x 256 dims (0.35 us per 128 ranks), fitted to 2250 shapes: the slower kernel is
// taken by 12 % at most, 0.14 % on average.  B_l kept / slabs, us, ranks 768: 64 sequences x 8 KV heads x 128 tokens 27.2 / 21.4, 128 of
// them 60 / 45, 300 x 1 x 384 77 / 67, 128 x 2 x 200 21.9 / 25.8, 33 x 2 x 1000 21 / 37, 33 x 8 x 384 38 / 33; ranks 384: 200 x 8 x 128 59
// / 46, 300 x 1 x 96 18.0 / 16.9, 33 x 2 x 1000 13.7 / 22.2.
bool reconstruct_keeps_factor(const xkv_shape &s, int r)
{
    if (r % 128 != 0 || r > 768) return false;
    const int col_groups = (s.H_kv * 128 + kRcDims - 1) / kRcDims, tiles = (s.L + kRkTok - 1) / kRkTok, tok_tiles = (s.L + kRcTok - 1) / kRcTok;
    const long long groups = (long long)s.batch * col_groups;
    if (r <= 256) return tok_tiles > 1 || tiles < kRcTok / kRkTok || groups < (r == 256 ? 256 : 480) || groups > 512;
    int runs = 1, run_tiles = tiles;
    reconstruct_cut(tiles, groups, 256, 4, &runs, &run_tiles);
    // (rounds of the chip: the last one is done earlier where it is not full)
    auto rounds = [](long long n) { return 0.75 * (double)((n + 255) / 256) + 0.25 * (double)n / 256; };
    const double factors = (double)s.batch * s.H_kv;  // read once, or by the token tiles on every die
    const double kept = 3.85 * rounds(groups * runs) + (double)((groups * runs + 255) / 256) * run_tiles + factors / 123;
    const double products = 7.0 * rounds(groups * tok_tiles);
    const double bytes = factors * std::min(tok_tiles, 8) / 132 + (double)s.batch * s.L * (1.0 + 128.0 * s.H_kv / r) / 9500;
    return kept <= std::max(products, bytes) + 1900.0 / r;
}

template <int NF>
static hipError_t launch_reconstruct_kept(const xkv_shape &s, int layer, const bf16_t *A, const bf16_t *B, bf16_t *X, hipStream_t st)
{
    static DynamicLdsOnce attr;
    if (hipError_t e = attr.ensure((const void *)reconstruct_kept_kernel<NF>, rk_lds<NF>()); e != hipSuccess) return e;
    const int col_groups = (s.H_kv * 128 + kRcDims - 1) / kRcDims, tiles = (s.L + kRkTok - 1) / kRkTok;
    int runs = 1, run_tiles = tiles;
    reconstruct_cut(tiles, (long long)s.batch * col_groups, rk_pair(NF) ? 512 : 256, 4, &runs, &run_tiles);
    const int total = runs * s.batch;
    const int per_die = (int)(((long long)total * col_groups + 7) / 8);
    const long long grid = 8LL * per_die;
    hipLaunchKernelGGL(reconstruct_kept_kernel<NF>, dim3((unsigned)grid), dim3(256), rk_lds<NF>(), st, A, B, X, s.G, layer, s.L, s.H_kv,
                       col_groups, runs, run_tiles, total, per_die);
    return hipGetLastError();
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
        const bf16_t *Ab = (const bf16_t *)A, *Bb = (const bf16_t *)B;
        if (reconstruct_keeps_factor(s, r)) switch (r / 128) {
            case 1: return launch_reconstruct_kept<8>(s, layer, Ab, Bb, (bf16_t *)X, st);
            case 2: return launch_reconstruct_kept<16>(s, layer, Ab, Bb, (bf16_t *)X, st);
            case 3: return launch_reconstruct_kept<24>(s, layer, Ab, Bb, (bf16_t *)X, st);
            case 4: return launch_reconstruct_kept<32>(s, layer, Ab, Bb, (bf16_t *)X, st);
            case 5: return launch_reconstruct_kept<40>(s, layer, Ab, Bb, (bf16_t *)X, st);
            case 6: return launch_reconstruct_kept<48>(s, layer, Ab, Bb, (bf16_t *)X, st);
            }
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
