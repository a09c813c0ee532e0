// Attention over the selected rows where nothing is applied to the reconstructed rows (no rotation), bf16 products:
//   out_h = softmax(scale K^_g q_h)^T V^_g,  K^_g = A^K[I_g,:] B^K_{l,g},  V^_g = A^V[I_g,:] B^V_{l,g}   (Sec. 3.2, Eq. 3)
// regrouped so that B_l meets one vector per query head instead of every selected row:
//   z_h = scale A^K[I_g,:] (B^K_{l,g} q_h),   U_h = w_h^T A^V[I_g,:],   out_h = U_h B^V_{l,g}.
//
// What bounds it: the gather of the rows.  Multiplying every row with B^K and B^V (the form that rows which are rotated
// still need, gather_attend_mfma.hip) takes 272 matrix instructions of 32 x 32 x 16 per 32 rows at ranks 512 and streams
// both B through LDS behind a barrier per 128 ranks; regrouped it is 32 + 16 of that size, no operand is shared by the
// wavefronts but the 32 KiB of projected queries, and the main loop has no barrier.
//
// A wavefront owns 32 rows of a tile from the first load to its own sums U.  Rows arrive line-wise (16 lanes x 16 B of
// four rows per request, 128 ranks of the 32 rows = one group = 8 requests), RG groups ahead in registers, and turn into
// operands in a wavefront-private 8 KiB LDS tile:
//   logits  v_mfma_f32_32x32x16_bf16, rows of A^K x projected queries; the 32 columns are 16 head slots twice, the high
//           part of the projected query and its remainder, so that the logits carry single-precision accuracy;
//   sums    v_mfma_f32_16x16x32_bf16, softmax weights [16 slots x 32 rows] x rows of A^V; the rows are the summed index
//           here, so the operand comes out of the tile through the transposing LDS read (4 rows x 16 ranks a time).
// The 16 result lanes of a logit tile hold, slot by slot, exactly the rows that the weights operand wants in that lane, so
// logits become weights without leaving the registers (online softmax, U rescaled once per tile).  At the end the wavefronts' U are added in LDS,
// split into a bf16 high part and remainder (again 16 + 16 rows of one operand; KEPT with three parts: see there) and multiplied with B^V.
//
// KEPT: the logits are there already, so that the keys' half falls away and a row costs its values alone: from the score stage
// (the absorbed step: every query head's score of every token) or, for rotated keys, from rope_keys_kernel
// or the KEYS form of gather_attend_mfma_kernel (of every selected row).  The weights meet the rows in parts of 8 bits, a matrix instruction each: in
// the absorbed step three, all 24 bits of them, as the general kernels have them (with two, 16 bits, and their exponentials short of a
// unit or two, sums that cancel showed it: test_sums_keep_single_precision); with rotated keys two, where the weights of the other form are
// rounded to 8.  Quantised rows are not rounded to bf16 either: the operand is the code itself (exact; with two parts 16 + c, which
// takes no conversion, and whose sixteens the offsets take off again), the group's step goes into the weights (w step, split as
// before), and what is left of the affine map, w lo or w (lo - 16 step), is one product per tile for all groups of 32 ranks.
// (4 x 8 x 4096 rows of ranks 512: 4 bits 27 us, and 1.5 for packing B^V beside the projection, against 27 of vector multiply-adds and
// 12 for merging them and B^V; bf16 33 us against 53.  Two parts instead of three: 24 and 32.)
#include "xkv_common.h"

#include "prepass.h"

namespace xkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
typedef __attribute__((ext_vector_type(8))) float f32x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((ext_vector_type(8))) short s16x8_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

// Projected queries of the heads of one KV head as operand fragments (see project_z_block), 4 wavefronts per block, then
// B^V_l and, for the rotated form, B^K_l and the query fragments: what the selected-row kernels need of q and B_l.
__global__ __launch_bounds__(256) void gather_prepare_kernel(PackArgs a) { gather_prepare_block(a, (int)blockIdx.x); }

hipError_t launch_gather_prepare(const PackArgs &a, hipStream_t st)
{
    const int blocks = a.blocks();
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_prepare_kernel, dim3(blocks), dim3(256), 0, st, a);
    return hipGetLastError();
}

constexpr int kAbWaves = 4;     // wavefronts per workgroup, 32 rows each
constexpr int kOutPitch = 132;  // floats per row of the last product's result
// The wavefronts' sums U are merged PG groups of 128 ranks at a time, [wavefront][rank][head slots, whole quads] floats: a
// lane of U holds a quad of slots of one rank.
__host__ __device__ inline int slab_quads(int n_rep) { return (n_rep + 3) / 4; }
__host__ __device__ inline int slab_bytes(int n_rep, int pg) { return kAbWaves * pg * 128 * slab_quads(n_rep) * 16; }
// (two workgroups share the LDS at occ 2; third: an operand for the third parts of U lies beside the slab)
__host__ __device__ inline int slab_groups(int n_rep, int ngv, int occ, bool third)
{
    int pg = ngv;
    while (pg > 1 && slab_bytes(n_rep, pg) > (occ == 2 ? 44 : third ? 84 : 100) * 1024) --pg;
    return pg;
}

// A group of quantised rows: 128 ranks = 4 quantisation groups of 32 rows, lane = (row lane / 4, group lane % 4) of 16 rows
// a request; 4-bit rows bring the group's (step, lo) word along, 3-bit pieces hold it.
template <int QB> struct RowGroup {
    static constexpr int N = QB == 0 ? 8 : 2;  // 16-byte requests per group and lane
    u32x4_t piece[N];
    uint32_t param[QB == 4 ? 2 : 1];
};

// 16 bytes of codes (32 ranks) and the group's (step, lo) -> 32 bf16 values, four 16-byte pieces in rank order.  A code c
// or-ed onto 0x4300 is the bf16 number 128 + c, so x^ = step (128 + c) + (lo - 128 step) is one multiply-add per element.
template <int QB> __device__ __forceinline__ u32x4_t dequant_word(uint32_t codes, float step, float lo2)
{
    constexpr uint32_t kMask = QB == 4 ? 0x000F000Fu : 0x00070007u;
    f32x8_t x;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t pr = ((codes >> (QB * i)) & kMask) | 0x43004300u;
        x[2 * i] = fmaf(step, __uint_as_float(pr << 16), lo2);
        x[2 * i + 1] = fmaf(step, __uint_as_float(pr & 0xFFFF0000u), lo2);
    }
    return __builtin_bit_cast(u32x4_t, __builtin_convertvector(x, bf16x8_t));
}

// The eight codes of a word (pairs of adjacent ranks 16 bits apart) of piece u of a request, and its (step, lo) word.
template <int QB> __device__ __forceinline__ void group_words(const RowGroup<QB> &g, int i, uint32_t (&codes)[4], uint32_t &par)
{
    const u32x4_t w = g.piece[i];
    if constexpr (QB == 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) codes[u] = w[u];
        par = g.param[i];
    } else {  // 96 bits of codes, four units of 24, then (step, lo)
        const uint32_t u4[4] = {w[0], (w[0] >> 24) | (w[1] << 8), (w[1] >> 16) | (w[2] << 16), w[2] >> 8};
#pragma unroll
        for (int u = 0; u < 4; ++u) codes[u] = (u4[u] & 0xFFFu) | ((u4[u] << 4) & 0x0FFF0000u);
        par = w[3];
    }
}

// The group into the wavefront's tile.  For the logits row t sits at 272 t (a lane reads 16 bytes of its own row: 16 rows
// then cover every bank once).  For the sums a transposing read takes 32 bytes of the four rows 4 q + i of each of the
// quarters q of the wavefront; row t = 16 a + 8 b + 4 c + d goes to place 16 b + 8 c + 4 a + d at a pitch of 288, which
// puts the rows of a read next to each other and their pieces on different banks.  Every access is one lane register
// plus a constant.
constexpr int kTileK = 272, kTileV = 288, kTileBytes = 32 * kTileV;
template <int QB, bool IS_K>
__device__ __forceinline__ void group_to_tile(const RowGroup<QB> &g, unsigned char *At, int lane)
{
    constexpr int PITCH = IS_K ? kTileK : kTileV;
    if constexpr (QB == 0) {
        unsigned char *dst = At + (lane >> 4) * PITCH + 16 * (lane & 15);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int place = IS_K ? 4 * j : 16 * ((j >> 1) & 1) + 8 * (j & 1) + 4 * (j >> 2);
            *reinterpret_cast<u32x4_t *>(dst + place * PITCH) = g.piece[j];
        }
    } else {
        const int r = lane >> 2, place = IS_K ? r : 16 * (r >> 3) + 8 * ((r >> 2) & 1) + (r & 3);
        unsigned char *dst = At + place * PITCH + 64 * (lane & 3);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            uint32_t codes[4], par;
            group_words<QB>(g, i, codes, par);
            const float step = __uint_as_float(par << 16), lo = __uint_as_float(par & 0xFFFF0000u);
            const float lo2 = fmaf(-128.0f, step, lo);
#pragma unroll
            for (int u = 0; u < 4; ++u)
                *reinterpret_cast<u32x4_t *>(dst + (IS_K ? 16 : 4) * i * PITCH + 16 * u) = dequant_word<QB>(codes[u], step, lo2);
        }
    }
}

// KEPT, quantised rows: the codes as bf16 numbers, c (4 bits; EXACT) or 16 + c (0x4180 with the code in the upper mantissa bits), laid
// out like the values above; the steps of every row of the four groups of 32 ranks, [group][row] floats in the order in which a lane
// takes the rows, and the offsets, lo or lo - 16 step, likewise.
constexpr int kStepBytes = 4 * 32 * 4;
__host__ __device__ constexpr int param_bytes(int ngv) { return (1 + ngv) * kStepBytes; }  // steps of one group of 128 ranks, offsets of all
template <int QB, bool EXACT> __device__ __forceinline__ void codes_to_tile(const RowGroup<QB> &g, unsigned char *At, float *steps, float *offsets, int lane)
{
    constexpr uint32_t kMask = QB == 4 ? 0x00780078u : 0x00380038u;
    const int r = lane >> 2, q = lane & 3, place = 16 * (r >> 3) + 8 * ((r >> 2) & 1) + (r & 3);
    unsigned char *dst = At + place * kTileV + 64 * q;
    const int at = 32 * q + 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3);
    uint32_t sixteen = 0x41804180u;
    asm("" : "+v"(sixteen));  // (in a register: an and-or instruction takes one constant)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        uint32_t codes[4], word;
        group_words<QB>(g, i, codes, word);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t w = codes[u];
            u32x4_t &to = *reinterpret_cast<u32x4_t *>(dst + 4 * i * kTileV + 16 * u);
            if constexpr (EXACT) {
                static_assert(QB == 4, "");
                // the bytes 0 .. 15 are the 8-bit floating-point numbers (e4m3) 0 .. 15 times 2^-9
                const uint32_t a = __builtin_amdgcn_perm(0u, w & 0x0F0F0F0Fu, 0x03010200u);         // bytes: ranks 0 1 4 5
                const uint32_t b = __builtin_amdgcn_perm(0u, (w >> 4) & 0x0F0F0F0Fu, 0x03010200u);  // ranks 2 3 6 7
                to = u32x4_t{__builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a, 512.0f, false)),
                             __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(b, 512.0f, false)),
                             __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(a, 512.0f, true)),
                             __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(b, 512.0f, true))};
            } else {
                to = u32x4_t{((w << 3) & kMask) | sixteen, (QB == 4 ? (w >> 1) & kMask : w & kMask) | sixteen,
                             ((w >> (2 * QB - 3)) & kMask) | sixteen, ((w >> (3 * QB - 3)) & kMask) | sixteen};
            }
        }
        const float step = __uint_as_float(word << 16), lo = __uint_as_float(word & 0xFFFF0000u);
        steps[at + 8 * i] = step;
        offsets[at + 8 * i] = EXACT ? lo : fmaf(-16.0f, step, lo);
    }
}

// x as a sum of N bf16 numbers, the largest first (three hold every bit of x)
template <int N> __device__ __forceinline__ void split_bf16(f32x8_t x, bf16x8_t (&part)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) {
        part[i] = __builtin_convertvector(x, bf16x8_t);
        if (i + 1 < N) x -= __builtin_convertvector(part[i], f32x8_t);
    }
}

// Row (16 lanes) and half-wavefront exchanges on the vector ALU.  permlane16_swap(x, y) trades the odd rows of x for the
// even rows of y: x' = (x0, y0, x2, y2), y' = (x1, y1, x3, y3); permlane32_swap does the same with the two halves.
__device__ __forceinline__ float add_row_pairs(float x, float y)  // lanes of row 0: x0 + x1, of row 1: y0 + y1, ...
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float max_over_rows(float x)  // over the four lanes with the same number in their row
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    const float a = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(a), false, false);
    return fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
}

// NGV groups of 128 ranks of A^V (U has NGV * 32 registers); RG groups in flight (a
// divisor of NGV).  QB: 0 = rows of A in bf16, 4 or 3 = quantised rows.  KEPT: see above; `heads` [batch][H_kv][L][hp] are the
// scaled logits of the tokens (by_place: [batch][H_kv][k][hp], of the places in the lists), A_k and Pz are not read, FZ is 0.
// KEPT (1, 2 or 4) is how often the query heads fit the 16 slots.  Copy c stands for group c of 32 ranks (modulo KEPT): a product for
// that group has zero weights in the other copies, so that the sums of KEPT groups share their registers (U of four heads and 512
// ranks 32 instead of 128, which is what lets two workgroups share a compute unit with four groups in flight each), and the
// weights times steps of KEPT groups of quantised rows are formed together.  PARTS: 8-bit parts of a weight; with three U is split into
// three as well before it meets B^V, and exponentials are those of the general kernels.
template <int NGV, int RG, int QB, int OCC, int KEPT, int PARTS>
__global__ __launch_bounds__(kAbWaves * 64, OCC) void gather_absorb_kernel(
    const void *__restrict__ A_k, const void *__restrict__ A_v, const u32x4_t *__restrict__ Pz, size_t pz_head_stride,
    const u32x4_t *__restrict__ pack_v, size_t pack_seq_stride, size_t pack_head_stride, const int32_t *__restrict__ idx,
    const int32_t *__restrict__ counts, float *__restrict__ part_o, float *__restrict__ part_ml, int L, int r_k, int r_v,
    int H_kv, int H_q, int k, int splits, int chunk, int FZ, float scale, const float *__restrict__ heads, int hp, bool by_place)
{
    static_assert(NGV % RG == 0, "a tile's groups of A^V start at ring entry 0");
    static_assert(KEPT ? PARTS == 2 || PARTS == 3 : PARTS == 1, "");
    constexpr bool FULL = PARTS == 3;
    auto exponential = [](float x) __attribute__((always_inline)) { return FULL ? expf(x) : __expf(x); };
    constexpr int WAVES = kAbWaves, TILE = WAVES * 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    // workgroup id -> (KV head fastest: the heads of a sequence gather from the same rows' lines), split, sequence
    const int g = blockIdx.x % H_kv, split = (blockIdx.x / H_kv) % splits, b = blockIdx.x / (H_kv * splits);
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5, l16 = lane & 15, q4 = lane >> 4;
    const int n_rep = H_q / H_kv;

    const int NGK = FZ / 8, nkp = (NGK + RG - 1) / RG * RG;  // groups of A^K, and padded to whole rings
    u32x4_t *Pl = reinterpret_cast<u32x4_t *>(smem_raw);     // [nkp][512], zero for the padding
    constexpr int kWaveBytes = kTileBytes + (KEPT && QB != 0 ? param_bytes(NGV) : 0), SLOTS = 16 / (KEPT ? KEPT : 1);  // slots per copy
    unsigned char *At = smem_raw + (size_t)nkp * 8192 + w * kWaveBytes;
    float *steps = reinterpret_cast<float *>(At + kTileBytes), *offsets = steps + kStepBytes / 4;
    int *toks = reinterpret_cast<int *>(smem_raw + (size_t)nkp * 8192 + WAVES * kWaveBytes) + w * (chunk / WAVES + 32);  // this wavefront's ids, tile by tile, then 32 times the first

    int k_eff = k;  // with `counts`, only the first counts[sequence][head] ids of a row are attended over
    if (counts) {
        const int cn = counts[b * H_kv + g];
        k_eff = cn < k ? (cn > 0 ? cn : 0) : k;
    }
    const int m_begin = split * chunk;
    const int m_end_raw = m_begin + chunk < k_eff ? m_begin + chunk : k_eff;
    const int m_end = m_end_raw > m_begin ? m_end_raw : m_begin;
    const int n_tiles = __builtin_amdgcn_readfirstlane((m_end - m_begin + TILE - 1) / TILE);

    // ids of this wavefront's rows (clamped into [0, L); rows past the end repeat the last one), then the projected
    // queries: requested before the ids are waited for
    const int32_t *ids = idx + ((size_t)b * H_kv + g) * k;
    const int n_ids = n_tiles * 32;
    int first_id[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + 64 * u;
        int m = m_begin + (i >> 5) * TILE + w * 32 + (i & 31);
        m = m < m_end ? m : (m_end > m_begin ? m_end - 1 : 0);
        first_id[u] = ids[m];
    }
    const u32x4_t *psrc = KEPT ? nullptr : Pz + ((size_t)b * H_kv + g) * pz_head_stride;
    const int p_total = FZ * 64;  // a multiple of 512
    constexpr int PN = 8;
    u32x4_t ptmp[PN];
#pragma unroll
    for (int j = 0; j < PN; ++j) {
        const int e = tid + j * WAVES * 64;
        if constexpr (!KEPT) ptmp[j] = psrc[e < p_total ? e : 0];
    }
    asm volatile("" : "+v"(first_id[0]), "+v"(first_id[1]));  // (keeps both loads ahead of the others, outside the branches)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = lane + 64 * u, t = first_id[u];
        const int tc = t < 0 ? 0 : (t >= L ? L - 1 : t);
        if (i < n_ids) toks[i] = tc;
        if (u == 0 && lane < 32) toks[chunk / WAVES + lane] = __builtin_amdgcn_readfirstlane(tc);
    }
    for (int i = lane + 128; i < n_ids; i += 64) {
        int m = m_begin + (i >> 5) * TILE + w * 32 + (i & 31);
        m = m < m_end ? m : m_end - 1;
        const int t = ids[m];
        toks[i] = t < 0 ? 0 : (t >= L ? L - 1 : t);
    }
    __builtin_amdgcn_wave_barrier();

    // ---- the sequence of groups of this wavefront: per tile all groups of A^K (padded to whole rings), then those of A^V.
    // (it_*) walks RG groups ahead of the group being multiplied; groups that do not exist (padding, past the end) are
    // requested from one row, a cache hit.
    // (a sequence has fewer than 2^24 rows and less than 4 GiB of them: byte offsets are 32-bit)
    const uint32_t pitch_k = QB == 0 ? (uint32_t)r_k * 2 : (uint32_t)quant_row_bytes(r_k, QB);
    const uint32_t pitch_v = QB == 0 ? (uint32_t)r_v * 2 : (uint32_t)quant_row_bytes(r_v, QB);
    const unsigned char *Ak = reinterpret_cast<const unsigned char *>(A_k) + (size_t)b * L * pitch_k;
    const unsigned char *Av = reinterpret_cast<const unsigned char *>(A_v) + (size_t)b * L * pitch_v;
    int it_i = 0, it_tile = 0;
    auto advance = [&]() __attribute__((always_inline)) {
        if (++it_i == nkp + NGV) {
            it_i = 0;
            ++it_tile;
        }
    };
    // what a group's requests need: the row base, the row pitch, the byte within the row (lane's piece, and its (step, lo)
    // word for 4-bit rows; pieces beyond the row are replaced by the first: they meet zero operands) and the row ids
    struct Request {
        const unsigned char *base;
        uint32_t pitch, off, par;
        const int *rows;  // this lane's first row id in LDS
    };
    auto request_of = [&]() __attribute__((always_inline)) {
        Request q;
        const bool is_k = it_i < nkp, real = it_tile < n_tiles && (it_i < NGK || it_i >= nkp);
        const int r = is_k ? r_k : r_v, it_g = is_k ? it_i : it_i - nkp;
        q.base = is_k ? Ak : Av;
        q.pitch = is_k ? pitch_k : pitch_v;
        if constexpr (QB == 0) {
            const int pc = 16 * it_g + (lane & 15);
            q.off = 16 * (pc < (r >> 3) ? pc : 0);
            q.par = 0;
        } else {
            const int gq = 4 * it_g + (lane & 3);
            const int gc = gq < (r >> 5) ? gq : 0;
            q.off = 16 * gc;
            q.par = (r >> 1) + 4 * gc;
        }
        q.rows = toks + (real ? it_tile * 32 : chunk / WAVES) + (QB == 0 ? lane >> 4 : lane >> 2);
        return q;
    };
    constexpr int NF = RowGroup<QB>::N, HS = KEPT && QB != 0 ? 8 : OCC == 2 ? 2 : 4;  // requests per group; steps whose operands are read together
    RowGroup<QB> ring[RG];
    // the rows of the requests [J0, J0 + N) of a group (read together, ahead of the requests), and request j
    auto rows_of = [&](const Request &q, int (&tk)[NF], int j0, int jn) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NF; ++j)
            if (j >= j0 && j < jn) tk[j] = q.rows[(QB == 0 ? 4 : 16) * j];
    };
    auto fetch = [&](RowGroup<QB> &e, const Request &q, const int (&tk)[NF], int j) __attribute__((always_inline)) {
        const uint32_t row = __umul24((uint32_t)tk[j], q.pitch);
        e.piece[j] = *reinterpret_cast<const u32x4_t *>(q.base + (row + q.off));
        if constexpr (QB == 4) e.param[j] = *reinterpret_cast<const uint32_t *>(q.base + (row + q.par));
    };
#pragma unroll
    for (int s = 0; s < RG; ++s) {
        const Request q = request_of();
        advance();
        int tk[NF];
        rows_of(q, tk, 0, NF);
#pragma unroll
        for (int j = 0; j < NF; ++j) fetch(ring[s], q, tk, j);
        __builtin_amdgcn_sched_barrier(0);
    }
    // projected queries into LDS
#pragma unroll
    for (int j = 0; j < PN; ++j) {
        const int e = tid + j * WAVES * 64;
        if (!KEPT && e < nkp * 512) Pl[e] = e < p_total ? ptmp[j] : u32x4_t{0u, 0u, 0u, 0u};
    }
    for (int e = tid + PN * WAVES * 64; !KEPT && e < nkp * 512; e += WAVES * 64)
        Pl[e] = e < p_total ? psrc[e] : u32x4_t{0u, 0u, 0u, 0u};
    if constexpr (!KEPT) lds_barrier();
    // KEPT: the logits of this lane's slot for the eight rows whose weights it holds, a tile ahead
    const int lrow = (n & 16) + 4 * hf;  // rows lrow + 8 (e / 4) + e % 4
    float zk[8];
    const float *hsrc = KEPT ? heads + ((size_t)b * H_kv + g) * (by_place ? k : L) * hp + (l16 % SLOTS < n_rep ? l16 % SLOTS : 0) : nullptr;
    auto request_logits = [&](int tile) __attribute__((always_inline)) {
        if (by_place) {
            const int m0 = m_begin + tile * TILE + w * 32 + lrow;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int m = m0 + 8 * (e / 4) + e % 4;
                zk[e] = hsrc[__umul24((uint32_t)(m < k ? m : k - 1), (uint32_t)hp)];
            }
        } else {
            const int *r = toks + (tile < n_tiles ? tile * 32 + lrow : chunk / WAVES);
#pragma unroll
            for (int e = 0; e < 8; ++e) zk[e] = hsrc[__umul24((uint32_t)r[8 * (e / 4) + e % 4], (uint32_t)hp)];
        }
    };
    if constexpr (KEPT) request_logits(0);
    constexpr int NO = KEPT && QB != 0 ? (NGV * 4 + 15) / 16 : 1;
    f32x4_t off_sum[NO];  // sums of w (lo - 16 step): rows the slots, columns the groups of 32 ranks
#pragma unroll
    for (f32x4_t &x : off_sum) x = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    constexpr int CP = KEPT ? KEPT : 1, NU = NGV * 8 / CP;  // copies; quads of sums: [set of CP groups of 32 ranks][half of 16 ranks]
    f32x4_t U[NU];
#pragma unroll
    for (int i = 0; i < NU; ++i) U[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const int copy = l16 / SLOTS;
    // a weights operand with all copies but `c` zero
    auto only = [&](const bf16x8_t &x, int c) __attribute__((always_inline)) {
        if constexpr (CP == 1) return x;
        u32x4_t u = __builtin_bit_cast(u32x4_t, x);
#pragma unroll
        for (int i = 0; i < 4; ++i) u[i] = copy == c ? u[i] : 0u;
        return __builtin_bit_cast(bf16x8_t, u);
    };
    float m_run = -INFINITY, l_run = 0.0f;  // of slot lane % 16 (the sum: this lane's share)
    const unsigned char *krd = At + n * kTileK + 16 * hf, *vrd = At + (4 * q4 + (l16 >> 2)) * kTileV + 8 * (l16 & 3);

    for (int tile = 0; tile < n_tiles; ++tile) {
        // ---- logits
        [[maybe_unused]] f32x16_t Z;
#pragma unroll
        for (int v = 0; v < 16; ++v) Z[v] = 0.0f;
        for (int i = 0; i < nkp; i += RG) {
#pragma unroll
            for (int s = 0; s < RG; ++s) {
                const Request q = request_of();
                advance();
                int tk[NF];
                if constexpr (OCC == 1) rows_of(q, tk, 0, NF);  // (two wavefronts per SIMD: registers are short instead)
                group_to_tile<QB, true>(ring[s], At, lane);
                __builtin_amdgcn_sched_barrier(0);
                const u32x4_t *pf = Pl + (i + s) * 512 + lane;
                // operands of HS steps are read together, the requests go out between the reads and the products
#pragma unroll
                for (int h4 = 0; h4 < 8; h4 += HS) {
                    u32x4_t a4[HS], p4[HS];
                    if constexpr (OCC == 2) rows_of(q, tk, h4, h4 + HS);
#pragma unroll
                    for (int fl = 0; fl < HS; ++fl) {
                        a4[fl] = *reinterpret_cast<const u32x4_t *>(krd + 32 * (h4 + fl));
                        p4[fl] = pf[(h4 + fl) * 64];
                    }
#pragma unroll
                    for (int fl = h4; fl < h4 + HS; ++fl)
                        if (fl < NF) fetch(ring[s], q, tk, fl);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int fl = 0; fl < HS; ++fl)
                        Z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a4[fl]),
                                                                    __builtin_bit_cast(bf16x8_t, p4[fl]), Z, 0, 0, 0);
                    if (OCC == 2 || h4 + HS == 8) __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // lane (slot column n, hf), register v = row 8 (v / 4) + 4 hf + v % 4; columns 16 .. 31 are the remainders of the
        // projected queries.  Of the two lanes of a slot, the first keeps registers 0 .. 7, the second 8 .. 15.
        const int base = m_begin + tile * TILE + w * 32;
        float z8[8], m_loc = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float z;
            if constexpr (KEPT)
                z = zk[e];
            else
                z = scale * add_row_pairs(Z[e], Z[8 + e]);
            const int t = base + lrow + 8 * (e / 4) + e % 4;
            z8[e] = t < m_end && (!KEPT || l16 % SLOTS < n_rep) ? z : -INFINITY;
            m_loc = fmaxf(m_loc, z8[e]);
        }
        // ---- logits -> weights (bf16, as the operand); rescaling of U and of the running sum
        const float m_new = fmaxf(m_run, max_over_rows(m_loc));
        const float alpha = (m_new == -INFINITY) ? 1.0f : exponential(m_run - m_new);
        f32x8_t wv;
        float l_add = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            wv[e] = z8[e] == -INFINITY ? 0.0f : exponential(z8[e] - m_new);
            l_add += wv[e];
        }
        bf16x8_t wp[PARTS];
        if constexpr (KEPT) request_logits(tile + 1);
        split_bf16<PARTS>(wv, wp);
        bf16x8_t wc[PARTS][QB == 0 ? CP : 1];
        if constexpr (KEPT && QB == 0) {
#pragma unroll
            for (int c = 0; c < CP; ++c)
#pragma unroll
                for (int p = 0; p < PARTS; ++p) wc[p][c] = only(wp[p], c);
        }
        l_run = l_run * alpha + l_add;
        m_run = m_new;
        if (tile > 0) {  // rows of U are slots 4 (lane / 16) + v
            if (lane < 16) reinterpret_cast<float *>(At)[lane] = alpha;  // (the tile is between two groups)
            const f32x4_t a = reinterpret_cast<const f32x4_t *>(At)[q4];
#pragma unroll
            for (int i = 0; i < NU; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) U[i][v] *= a[v];
            if constexpr (KEPT && QB != 0) {
#pragma unroll
                for (f32x4_t &x : off_sum) x *= a;
            }
        }
        // ---- U += W A^V[rows]
        [[maybe_unused]] bf16x8_t sp[PARTS], gp[PARTS];
#pragma unroll
        for (int gv = 0; gv < NGV; ++gv) {
            const Request q = request_of();
            advance();
            int tk[NF];
            if constexpr (OCC == 1) rows_of(q, tk, 0, NF);
            if constexpr (KEPT && QB != 0)
                codes_to_tile<QB, FULL>(ring[gv % RG], At, steps, offsets + gv * (kStepBytes / 4), lane);
            else
                group_to_tile<QB, false>(ring[gv % RG], At, lane);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h4 = 0; h4 < 8; h4 += HS) {
                s16x4_t v4[HS][2];
                constexpr int NB = KEPT && QB != 0 ? (HS / 2 + KEPT - 1) / KEPT : 1;  // sets of weights for these steps
                f32x4_t pq[NB][2];  // the steps of this lane's eight rows in its copy's group
                if constexpr (OCC == 2) rows_of(q, tk, h4, h4 + HS);
                if constexpr (KEPT && QB != 0) {
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        const f32x4_t *ps = reinterpret_cast<const f32x4_t *>(steps + 16 * h4 + 32 * (KEPT * j + l16 / SLOTS) + 8 * q4);
                        pq[j][0] = ps[0], pq[j][1] = ps[1];
                    }
                }
#pragma unroll
                for (int j = 0; j < HS; ++j) {
                    const unsigned char *p = vrd + 32 * (h4 + j);
                    v4[j][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)p);
                    v4[j][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(p + 16 * kTileV));
                }
#pragma unroll
                for (int j = h4; j < h4 + HS; ++j)
                    if (j < NF) fetch(ring[gv % RG], q, tk, j);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < HS; ++j) {
                    const bf16x8_t v8 = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(v4[j][0], v4[j][1], 0, 1, 2, 3, 4, 5, 6, 7));
                    if constexpr (KEPT && QB != 0) {
                        if (j % (2 * KEPT) == 0) {
                            f32x8_t ws;
#pragma unroll
                            for (int e = 0; e < 8; ++e) ws[e] = wv[e] * pq[j / (2 * KEPT)][e / 4][e % 4];
                            split_bf16<PARTS>(ws, sp);
                        }
                        if (j % 2 == 0) {
#pragma unroll
                            for (int p = 0; p < PARTS; ++p) gp[p] = only(sp[p], (h4 + j) / 2 % CP);
                        }
                        f32x4_t &u = U[(gv * 4 + (h4 + j) / 2) / CP * 2 + j % 2];
#pragma unroll
                        for (int p = 0; p < PARTS; ++p) u = __builtin_amdgcn_mfma_f32_16x16x32_bf16(gp[p], v8, u, 0, 0, 0);
                    } else if constexpr (KEPT) {
                        f32x4_t &u = U[(gv * 4 + (h4 + j) / 2) / CP * 2 + j % 2];
#pragma unroll
                        for (int p = 0; p < PARTS; ++p)
                            u = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wc[p][(h4 + j) / 2 % CP], v8, u, 0, 0, 0);
                    } else {
                        U[gv * 8 + h4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[0], v8, U[gv * 8 + h4 + j], 0, 0, 0);
                    }
                }
                if (OCC == 2 || h4 + HS == 8) __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (KEPT && QB != 0) {
#pragma unroll
            for (int c = 0; c < NO; ++c) {
                const int grp = 16 * c + l16 < NGV * 4 ? 16 * c + l16 : 0;  // (columns beyond the groups are not used)
                const f32x4_t *ps = reinterpret_cast<const f32x4_t *>(offsets + 32 * grp + 8 * q4);
                const f32x8_t o8 = __builtin_shufflevector(ps[0], ps[1], 0, 1, 2, 3, 4, 5, 6, 7);
                constexpr int OP = FULL ? 1 : PARTS;  // (lo is a bf16 number)
                bf16x8_t op[OP];
                split_bf16<OP>(o8, op);
#pragma unroll
                for (int i = 0; i < OP; ++i)
#pragma unroll
                    for (int p = 0; p < PARTS - i; ++p)  // (remainder by remainder is left out)
                        off_sum[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wp[p], op[i], off_sum[c], 0, 0, 0);
            }
        }
    }

    const int row_copy = q4 / (SLOTS / 4);  // of this lane's rows of U
    if constexpr (KEPT && QB != 0) {  // the rest of the affine map: column group -> all ranks of the group
#pragma unroll
        for (int i = 0; i < NU / 2; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float y = __shfl(off_sum[i * CP / 16][v], 16 * q4 + (i * CP) % 16 + row_copy, kWave);
                U[2 * i][v] += y;
                U[2 * i + 1][v] += y;
            }
    }
    // ---- merge of the wavefronts and the product with B^V.  The rows of B^V that this wavefront multiplies are requested
    // first: fragments of 16 ranks x its 32 channels.
    constexpr int NFB = NGV * 8;
    const u32x4_t *pv = pack_v + (size_t)b * pack_seq_stride + (size_t)g * pack_head_stride + w * 64 + lane;
    // fragments requested ahead of the merge: what the registers hold beside U.  (Six groups: 32 instead of 16 take 0.5 us off a
    // step of one tile per workgroup, 24.6 -> 24.1 us; with 3-bit rows they cost 2 % of 16 x 8 x 4096 rows, 180 -> 184 us.)
    constexpr int NPF = OCC == 2 || (NGV == 6 && QB == 3) ? 16 : NFB < 32 ? NFB : 32;
    u32x4_t bv[NPF];
#pragma unroll
    for (int f = 0; f < NPF; ++f) bv[f] = pv[(size_t)f * 256];

    const float l_a = l_run + __shfl_xor(l_run, 16, kWave), l_tot = l_a + __shfl_xor(l_a, 32, kWave);
    const int PG = slab_groups(n_rep, NGV, OCC, FULL && CP == 1), NQ = slab_quads(n_rep);
    // Rows of an operand: the high parts of the slots, then their remainders.  Three parts fit it where there are eight slots; else the
    // third is an operand of its own, Uf3, whose other rows repeat it.
    constexpr bool THIRD = FULL && CP == 1;
    constexpr int PROWS = FULL && !THIRD ? 8 : 16;
    uint16_t *Uf = reinterpret_cast<uint16_t *>(smem_raw);                         // [NGV * 8][64][8]
    float *ml = reinterpret_cast<float *>(smem_raw + NGV * 8 * 1024);               // [2][WAVES][16]
    uint16_t *Uf3 = reinterpret_cast<uint16_t *>(ml + 2 * WAVES * 16);              // THIRD: [NGV * 8][2][16][8]
    float *slab = ml + 2 * WAVES * 16 + (THIRD ? NGV * 1024 : 0);
    __syncthreads();  // everybody is done with the operands
    if (lane < 16) {
        ml[w * 16 + lane] = m_run;
        ml[(WAVES + w) * 16 + lane] = l_tot;
    }
    __syncthreads();
    f32x4_t f4;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int hh = 4 * q4 + v;
        float M = -INFINITY;
#pragma unroll
        for (int ww = 0; ww < WAVES; ++ww) M = fmaxf(M, ml[ww * 16 + hh]);
        const float mw = ml[w * 16 + hh];
        f4[v] = mw == -INFINITY ? 0.0f : exponential(mw - M);
    }
    for (int g0 = 0; g0 < NGV; g0 += PG) {
#pragma unroll
        for (int gv = 0; gv < NGV; ++gv)
            if (gv >= g0 && gv < g0 + PG) {
                // (a quad of slots per lane, of the copy that its rows belong to)
                f32x4_t *dst = reinterpret_cast<f32x4_t *>(slab) + ((w * PG + gv - g0) * 128 + 32 * row_copy + l16) * NQ + q4 % (SLOTS / 4);
                if (q4 % (SLOTS / 4) < NQ) {
#pragma unroll
                    for (int i = 0; i < 8 / CP; ++i) dst[(i / 2 * 32 * CP + 16 * (i % 2)) * NQ] = f4 * U[gv * (8 / CP) + i];
                }
            }
        __syncthreads();
        const int ng = NGV - g0 < PG ? NGV - g0 : PG;
        for (int item = tid; item < NQ * ng * 32; item += WAVES * 64) {  // four ranks of four slots
            const int hq = item % NQ, c = 4 * (item / NQ);
            const f32x4_t *src = reinterpret_cast<const f32x4_t *>(slab) + c * NQ + hq;
            f32x4_t sum[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] = src[e * NQ];
#pragma unroll
            for (int ww = 1; ww < WAVES; ++ww)
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += src[(ww * PG * 128 + e) * NQ];
            uint16_t *dst = Uf + (((g0 * 8 + (c >> 4)) * 64 + ((c >> 3) & 1) * 32 + 4 * hq) * 8 + (c & 7));
            [[maybe_unused]] uint16_t *dst3 = Uf3 + (((g0 * 8 + (c >> 4)) * 32 + ((c >> 3) & 1) * 16 + 4 * hq) * 8 + (c & 7));
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                f32x4_t x = f32x4_t{sum[0][v], sum[1][v], sum[2][v], sum[3][v]};
#pragma unroll
                for (int p = 0; p < (FULL ? 3 : 2); ++p) {
                    const bf16x4_t part = __builtin_convertvector(x, bf16x4_t);
                    uint16_t *to = THIRD && p == 2 ? dst3 + v * 8 : dst + (PROWS * p + v) * 8;
                    *reinterpret_cast<bf16x4_t *>(to) = part;
                    x -= __builtin_convertvector(part, f32x4_t);
                }
            }
        }
        __syncthreads();
    }
    const u32x4_t *Uq = reinterpret_cast<const u32x4_t *>(Uf) + lane, *Uq3 = reinterpret_cast<const u32x4_t *>(Uf3) + 16 * hf + l16;
    float *po = slab;  // [16][kOutPitch]
    f32x16_t o, o3;
#pragma unroll
    for (int v = 0; v < 16; ++v) o[v] = o3[v] = 0.0f;
#pragma unroll
    for (int f = 0; f < NFB; ++f) {
        const bf16x8_t b8 = __builtin_bit_cast(bf16x8_t, f < NPF ? bv[f < NPF ? f : 0] : pv[(size_t)f * 256]);
        o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, Uq[f * 64]), b8, o, 0, 0, 0);
        if constexpr (THIRD) o3 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, Uq3[f * 32]), b8, o3, 0, 0, 0);
    }
    // register v is row 8 (v / 4) + 4 hf + v % 4
    if constexpr (PROWS == 8) {
#pragma unroll
        for (int v = 0; v < 4; ++v) po[(4 * hf + v) * kOutPitch + w * 32 + n] = o[v] + (o[v + 4] + o[v + 8]);
    } else {
#pragma unroll
        for (int v = 0; v < 8; ++v) po[(8 * (v / 4) + 4 * hf + (v % 4)) * kOutPitch + w * 32 + n] = THIRD ? o[v] + (o[v + 8] + o3[v]) : o[v] + o[v + 8];
    }
    __syncthreads();
    for (int item = tid; item < n_rep * 128; item += WAVES * 64) {
        const int hh = item >> 7, dim = item & 127;
        const size_t slot = ((size_t)b * H_q + g * n_rep + hh) * splits + split;
        part_o[slot * 128 + dim] = po[hh * kOutPitch + dim];
        if (dim == 0) {
            float M = -INFINITY, den = 0.0f;
#pragma unroll
            for (int ww = 0; ww < WAVES; ++ww) M = fmaxf(M, ml[ww * 16 + hh]);
#pragma unroll
            for (int ww = 0; ww < WAVES; ++ww) {
                const float mw = ml[ww * 16 + hh];
                den += (mw == -INFINITY ? 0.0f : exponential(mw - M)) * ml[(WAVES + ww) * 16 + hh];
            }
            part_ml[slot * 2 + 0] = M;
            part_ml[slot * 2 + 1] = den;
        }
    }
}

constexpr size_t kAbsorbLdsMax = 160 * 1024 - 512, kAbsorbLdsPair = 80 * 1024;  // for one workgroup, for each of two

// Groups in flight per wavefront.  The groups of A^K are padded to whole rings; the deep ring of four is left where it would
// add two groups or more to a tile (r_k = 640 or 768 with r_v = 512, 16 x 8 x 4096 rows: 199 -> 197 us in bf16, 194 -> 169
// in 4 bits, where the padding is de-quantised too).  Three for six groups of A^V are slower (384 : 576 175 -> 191 us).
static constexpr int absorb_rg(int ngv, int occ, bool deep) { return ngv == 3 ? 3 : ngv == 4 && occ == 1 && deep ? 4 : 2; }
static bool absorb_deep(int FZ) { return (FZ / 8 + 3) % 4 >= 2; }

static size_t absorb_lds(int ngv, int occ, int n_rep, int FZ, int chunk, int parts = 1)
{
    const int rg = absorb_rg(ngv, occ, absorb_deep(FZ));
    const size_t main = (size_t)(FZ / 8 + rg - 1) / rg * rg * 8192 + (size_t)kAbWaves * (kTileBytes + 128 + (parts > 1 ? param_bytes(ngv) : 0)) + (size_t)chunk * 4;
    const bool third = parts == 3 && n_rep > 8;
    const int slab = slab_bytes(n_rep, slab_groups(n_rep, ngv, occ, third)), out = 16 * kOutPitch * 4;
    const size_t merge = (size_t)ngv * (third ? 8192 + 4096 : 8192) + (size_t)2 * kAbWaves * 16 * 4 + (size_t)(slab > out ? slab : out);
    return main > merge ? main : merge;
}

// Groups of 128 ranks of A^V that a wavefront keeps sums for: 2, 3, 4 or 6 (0: more than the registers hold).
static int absorb_ngv(int r_v)
{
    const int g = (r_v + 127) / 128;
    return g <= 2 ? 2 : g <= 4 ? g : g <= 6 ? 6 : 0;
}

bool gather_absorb_shape_ok(const xkv_shape &s)
{
    // (up to r_k = 1024 the projected queries, 64 KiB there, fit the LDS beside the tiles and the ids)
    const long long widest = s.r_k > s.r_v ? s.r_k : s.r_v;
    return s.L < (1 << 24) && s.L * widest * 2 < (1LL << 32) && s.r_k <= 1024 && absorb_ngv(s.r_v) != 0;
}

// What the matrix cores save grows with the query heads; what they cost is the packing of B^V (rows * r_v) and, per number
// gathered, a little more than the general kernels need for rows of bf16.  Whole steps with 8 KV heads, budgets a sixteenth, us general
// / matrix cores: 4 query heads each, ranks 512, 8 sequences x 4096 rows 198.8 / 198.8, 16 x 4096 363 / 399, ranks 256 221 / 230; in
// 4 bits 16 x 4096 216 / 212, but 16 x 16384 (row sums alone) 234 / 247; ranks 768 (two groups in flight) 4 x 2048 102 / 101, 16 x 1024
// 169 / 171, in 4 bits 110 / 112 and 170 / 176.  One query head: ranks 512, 1 x 4096 68 / 57, 4 x 512 40 / 42, 16 x 4096 340 / 366;
// ranks 128, 16 x 512 41 / 44, 16 x 1024 the same, 16 x 4096 137 / 129; ranks 768, 1 x 512 38 / 40, 1 x 2048 52 / 50.  Two are like one;
// from nine on the general row sums take 1.6 to 3.4 times as long.
bool absorbed_mfma_pays(const xkv_shape &s, bool q4)
{
    const int n_rep = s.H_q / s.H_kv;
    const long long rows = (long long)s.batch * s.H_kv, numbers = rows * s.k * s.r_v;
    if (n_rep > 8) return true;
    if (n_rep <= 2 && (s.k < (s.r_v > 512 ? 2048 : 1024) || (rows * s.r_v >= 16384 && s.r_v > (q4 ? 256 : 128)))) return false;
    if (s.r_v > 512 && n_rep <= 4) return numbers < 1LL << 25;
    return numbers < (q4 ? 1LL << 30 : 1LL << 27);
}

void gather_absorb_plan(const xkv_shape &s, Plan &p)
{
    // Tiles are 128 rows.  Where every compute unit gets more than one, U fits 256 registers a lane and two workgroups fit the
    // LDS, two share a compute unit, so that the one streams while the other merges; else one with twice the registers, all of
    // them for requests in flight.  (At 16 sequences x 8 heads x 4096 rows of ranks 512 a pass of four layers took 1489 us; one
    // workgroup of eight wavefronts per compute unit 1513: its wavefronts finish up to 12 us apart.  A workgroup of the first
    // kind without room for its partner has neither: 85 us at 4 x 8 x 4096 rows of ranks 768 : 512 where one of the second
    // kind takes 66, 217 and 196 at 16 x 8 x 4096 of 640 : 512.)
    const int tile = 128, rows = p.rows > 0 ? p.rows : 1;
    const int tiles = (s.k + tile - 1) / tile, ngv = absorb_ngv(s.r_v), FZ = (s.r_k / 16 + 7) / 8 * 8;
    // a workgroup keeps 4096 ids at most where the partials allow it; the merge takes these partials and those of an
    // uncompressed tail (one sequence of one KV head, k of a million)
    const int fewest = (s.k + 4095) / 4096;
    int most = kMaxCombineParts - kTailParts;
    if (most < fewest) most = fewest;
    if (most > p.max_splits) most = p.max_splits;
    // Lists are cut so that the workgroups make whole rounds of the chip: a few more than a round take as long as two (6 x 8 x
    // 2048 rows of ranks 768 as 288 workgroups 92 us, as 192 67).  A round is one workgroup per compute unit; where two share
    // one it is counted as two rounds of both, so that later workgroups fill the gaps that uneven ends leave.  Of the cuts
    // into the first rounds possible the one that is done first is taken, the start and the merge of a workgroup counted as
    // one tile.  (One round of both is 0 to 8 % faster at two to eight tiles per workgroup, 177 against 180 us at 16 x 8 x 4096 rows
    // of ranks 512, but a weight is exact only for the largest logit of a wavefront's list, and with longer lists the
    // rounding of the others shows more: error 2.14e-3 against 2.09e-3; forming every row 3.20e-3.)
    auto cut = [&](int slots, int start, int *chunk, int *used_splits) {
        const int first = (rows + slots - 1) / slots;
        long long best = 0;
        for (int rounds = first; rounds < first + 4; ++rounds) {
            int splits = (int)((long long)slots * rounds / rows);
            splits = splits > most ? most : splits;
            splits = splits < fewest ? fewest : splits;
            splits = splits > tiles ? tiles : splits;
            const int per = (tiles + splits - 1) / splits, used = (tiles + per - 1) / per;
            const long long time = ((long long)rows * used + slots - 1) / slots * (per + start);
            if (best > 0 && time >= best) continue;
            best = time;
            *chunk = per * tile;
            *used_splits = used;
        }
    };
    auto cut_for = [&](int occ) {
        cut(occ == 2 ? 1024 : 256, 1, &p.ab_chunk, &p.ab_splits);
        p.ab_occ = occ;
        p.ab_lds = absorb_lds(ngv, occ, p.n_rep, FZ, p.ab_chunk);
    };
    if (ngv <= 4 && (long long)rows * tiles > 256) cut_for(2);
    if (p.ab_occ != 2 || p.ab_lds > kAbsorbLdsPair) cut_for(1);
    // given logits: a tile is half the work or less beside the same start and merge
    cut(p.n_rep <= 8 ? 512 : 256, 2, &p.ak_chunk, &p.ak_splits);
}

hipError_t launch_gather_absorb(const xkv_shape &s, const Plan &p, const PackArgs &pa, const void *A_k, const void *A_v,
                                const void *B_packed, int layer, const int32_t *idx, const int32_t *counts, float *part_o,
                                float *part_ml, int qbits, hipStream_t st, const float *heads, bool by_place)
{
    const size_t per_head = (size_t)(pa.F8k + pa.F8v) * 256;  // pieces of 16 B
    const u32x4_t *pv = (B_packed ? (const u32x4_t *)B_packed + (size_t)layer * s.H_kv * per_head : (const u32x4_t *)pa.pack) +
                        (size_t)pa.F8k * 256;
    const size_t seq_stride = (B_packed ? (size_t)s.G : 1) * s.H_kv * per_head;
    const int ngv = absorb_ngv(s.r_v);
    const int hp = head_pitch_of(p.n_rep), FZ = heads ? 0 : pa.FZ;
    const int occ = p.ab_occ, splits = heads ? p.ak_splits : p.ab_splits, chunk = heads ? p.ak_chunk : p.ab_chunk;
    const size_t lds = heads ? absorb_lds(ngv, p.n_rep <= 8 ? 2 : 1, p.n_rep, 0, chunk, by_place ? 2 : 3) : p.ab_lds;
    if (ngv == 0 || lds > kAbsorbLdsMax || splits > p.max_splits) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((long long)splits * s.H_kv * s.batch));
    const int stage = heads ? 4 : 1;
#define XKV_AB(NV, OC, DP, QB, KP, PT)                                                                                  \
    do {                                                                                                                \
        static DynamicLdsOnce attr;                                                                                     \
        constexpr int RG = KP ? (NV == 3 ? 3 : NV == 4 ? 4 : 2) : absorb_rg(NV, OC, DP);                                \
        const hipError_t e = attr.ensure((const void *)gather_absorb_kernel<NV, RG, QB, OC, KP, PT>, kAbsorbLdsMax);    \
        if (e != hipSuccess) return e;                                                                                  \
        if (!by_place) profile_begin(stage, st);                                                                        \
        hipLaunchKernelGGL((gather_absorb_kernel<NV, RG, QB, OC, KP, PT>), grid, dim3(256), lds, st, A_k, A_v,          \
                           (const u32x4_t *)pa.Pz, pa.z_stride / 8, pv, seq_stride, per_head, idx, counts, part_o,      \
                           part_ml, s.L, s.r_k, s.r_v, s.H_kv, s.H_q, s.k, splits, chunk, FZ, p.scale,                  \
                           heads, hp, by_place);                                                                        \
        if (!by_place) profile_end(stage, st);                                                                          \
    } while (0)
#define XKV_AB_Q(NV, OC, DP)                  \
    do {                                      \
        if (qbits == 0)                       \
            XKV_AB(NV, OC, DP, 0, 0, 1);      \
        else if (qbits == 4)                  \
            XKV_AB(NV, OC, DP, 4, 0, 1);      \
        else                                  \
            XKV_AB(NV, OC, DP, 3, 0, 1);      \
    } while (0)
#define XKV_AB_KC(NV, OC, CPS)                 \
    do {                                       \
        if (by_place) {                        \
            if constexpr (CPS > 1 && NV <= 4) {      \
                if (qbits == 0)                      \
                    XKV_AB(NV, OC, true, 0, CPS, 2); \
                else if (qbits == 4)                 \
                    XKV_AB(NV, OC, true, 4, CPS, 2); \
                else                                 \
                    XKV_AB(NV, OC, true, 3, CPS, 2); \
            } else {                           \
                return hipErrorInvalidValue;   \
            }                                  \
        } else if (qbits == 0)                 \
            XKV_AB(NV, OC, true, 0, CPS, 3);   \
        else                                   \
            XKV_AB(NV, OC, true, 4, CPS, 3);   \
    } while (0)
#define XKV_AB_K(NV)                        \
    do {                                    \
        if (p.n_rep <= 4)                   \
            XKV_AB_KC(NV, 2, 4);            \
        else if (p.n_rep <= 8)              \
            XKV_AB_KC(NV, 2, 2);            \
        else                                \
            XKV_AB_KC(NV, 1, 1);            \
    } while (0)
    // (The order here is the order in the code object: with the given-logits forms first, 0.8 MB, the others, code for code the same, began
    // past 1.2 MB and a step of one sequence of 32768 tokens took 179 us instead of 176.6.)
    if (!heads && occ == 2) {
        if (ngv == 2)
            XKV_AB_Q(2, 2, false);
        else if (ngv == 3)
            XKV_AB_Q(3, 2, false);
        else
            XKV_AB_Q(4, 2, false);
    } else if (!heads) {
        if (ngv == 2)
            XKV_AB_Q(2, 1, false);
        else if (ngv == 3)
            XKV_AB_Q(3, 1, false);
        else if (ngv == 4 && absorb_deep(pa.FZ))
            XKV_AB_Q(4, 1, true);
        else if (ngv == 4)
            XKV_AB_Q(4, 1, false);
        else
            XKV_AB_Q(6, 1, false);
    } else {
        if (ngv == 2)
            XKV_AB_K(2);
        else if (ngv == 3)
            XKV_AB_K(3);
        else if (ngv == 4)
            XKV_AB_K(4);
        else
            XKV_AB_K(6);
    }
#undef XKV_AB_K
#undef XKV_AB_KC
#undef XKV_AB_Q
#undef XKV_AB
    return hipGetLastError();
}

}  // namespace xkv
