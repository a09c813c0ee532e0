// Query projection into the rank space and the low-rank score stream with GQA max-pooling.
//   p_h = B^K_{l,rho(h)} q_h                      (Eq. 3 regrouped by associativity)
//   s[h,t] = scale * A^K[t,:] . p_h               (App. B.1 Alg. 2, scaled scores, per token)
//   S[g,t] = max_{h: rho(h)=g} s[h,t]             (App. B.1 Alg. 2, GQA pooling)
#include "xkv_common.h"
#include "prepass.h"
#include "dense_block.h"

namespace xkv {

// ------------------------------------------------------------------------------------------
// project_q: one wavefront per (rank index i, KV head g); lanes run over the head dimension.
// P is written as fp32 [batch][H_q][r_k].
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void project_q_kernel(const T *__restrict__ B_k,  // [batch][G][r_k][d]
                                                        const T *__restrict__ q,    // [batch][H_q][d_h]
                                                        float *__restrict__ P,      // [batch][H_q][r_k]
                                                        int G, int layer, int r_k, int H_kv, int H_q, int d_h)
{
    const int b = blockIdx.y;
    const int item = blockIdx.x * 4 + wave_id();  // (i, g) pair
    if (item >= r_k * H_kv) return;
    const int i = item / H_kv, g = item % H_kv;
    const int n_rep = H_q / H_kv, d = H_kv * d_h;
    const int lane = lane_id();
    const T *Brow = B_k + (((size_t)b * G + layer) * r_k + i) * d + (size_t)g * d_h;
    const T *qg = q + ((size_t)b * H_q + (size_t)g * n_rep) * d_h;
    float acc[16];
#pragma unroll
    for (int hh = 0; hh < 16; ++hh) acc[hh] = 0.0f;
    for (int j = lane; j < d_h; j += kWave) {
        const float bv = to_f32(Brow[j]);
#pragma unroll
        for (int hh = 0; hh < 16; ++hh)
            if (hh < n_rep) acc[hh] = fmaf(bv, to_f32(qg[(size_t)hh * d_h + j]), acc[hh]);
    }
#pragma unroll
    for (int hh = 0; hh < 16; ++hh) {
        if (hh < n_rep) {
            const float v = wave_sum(acc[hh]);
            if (lane == 0) P[((size_t)b * H_q + g * n_rep + hh) * r_k + i] = v;
        }
    }
}

// ------------------------------------------------------------------------------------------
// score, general path: one thread per token, fp32 FMA.  Each thread walks its row of A^K once
// per block of up to 8 query heads; P is read through wave-uniform (scalar) loads.
// ------------------------------------------------------------------------------------------
template <typename T, int HB>  // query heads per walk over the row
__global__ __launch_bounds__(256) void score_generic_kernel(const T *__restrict__ A_k,      // [batch][L][r_k]
                                                            const float *__restrict__ P,   // [batch][H_q][r_k]
                                                            float *__restrict__ S,         // [batch][H_kv][L]
                                                            int L, int r_k, int H_kv, int H_q, float scale)
{
    const int b = blockIdx.y;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= L) return;
    const int n_rep = H_q / H_kv;
    const T *Arow = A_k + ((size_t)b * L + t) * r_k;
    const float *Pb = P + (size_t)b * H_q * r_k;
    for (int g = 0; g < H_kv; ++g) {
        float best = -INFINITY;
        for (int h0 = 0; h0 < n_rep; h0 += HB) {
            float acc[HB];
#pragma unroll
            for (int hh = 0; hh < HB; ++hh) acc[hh] = 0.0f;
            const float *Pg = Pb + (size_t)(g * n_rep + h0) * r_k;
            const int nh = n_rep - h0 < HB ? n_rep - h0 : HB;
            // (heads beyond nh take the last one's P again and are not used: no branch between the loads)
            const float *Ph[HB];
#pragma unroll
            for (int hh = 0; hh < HB; ++hh) Ph[hh] = Pg + (size_t)(hh < nh ? hh : nh - 1) * r_k;
#pragma unroll (HB == 4 ? 8 : 2)
            for (int i = 0; i < r_k; ++i) {
                const float a = to_f32(Arow[i]);
#pragma unroll
                for (int hh = 0; hh < HB; ++hh) acc[hh] = fmaf(a, Ph[hh][i], acc[hh]);
            }
#pragma unroll
            for (int hh = 0; hh < HB; ++hh)
                if (hh < nh) best = fmaxf(best, scale * acc[hh]);
        }
        S[((size_t)b * H_kv + g) * L + t] = best;
    }
}

// Same walk, but every query head's score is kept as well: S_heads is [batch][H_kv][L][nrp] with nrp the
// number of query heads per KV head rounded up to a power of two (the padding is written as zero).  The pooled
// score is the maximum of exactly the values stored, so a softmax over stored head scores agrees with the
// selection made on S.
template <typename T>
__global__ __launch_bounds__(256) void score_heads_generic_kernel(const T *__restrict__ A_k,     // [batch][L][r_k]
                                                                  const float *__restrict__ P,  // [batch][H_q][r_k]
                                                                  float *__restrict__ S,        // [batch][H_kv][L]
                                                                  float *__restrict__ S_heads, int L, int r_k,
                                                                  int H_kv, int H_q, int nrp, float scale)
{
    const int b = blockIdx.y;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= L) return;
    const int n_rep = H_q / H_kv;
    const T *Arow = A_k + ((size_t)b * L + t) * r_k;
    const float *Pb = P + (size_t)b * H_q * r_k;
    for (int g = 0; g < H_kv; ++g) {
        float best = -INFINITY;
        float *dst = S_heads + (((size_t)b * H_kv + g) * L + t) * nrp;
        for (int h0 = 0; h0 < nrp; h0 += 8) {
            float acc[8];
#pragma unroll
            for (int hh = 0; hh < 8; ++hh) acc[hh] = 0.0f;
            const float *Pg = Pb + (size_t)(g * n_rep + h0) * r_k;
            const int nh = n_rep - h0 < 8 ? n_rep - h0 : 8;  // may be <= 0 inside the padding
            for (int i = 0; i < r_k && nh > 0; ++i) {
                const float a = to_f32(Arow[i]);
#pragma unroll
                for (int hh = 0; hh < 8; ++hh)
                    if (hh < nh) acc[hh] = fmaf(a, Pg[(size_t)hh * r_k + i], acc[hh]);
            }
#pragma unroll
            for (int hh = 0; hh < 8; ++hh) {
                if (hh < nh) best = fmaxf(best, scale * acc[hh]);
                if (h0 + hh < nrp) dst[h0 + hh] = hh < nh ? scale * acc[hh] : 0.0f;
            }
        }
        S[((size_t)b * H_kv + g) * L + t] = best;
    }
}

// ==========================================================================================
// bf16 MFMA path.  The contraction S^T = P_slots (32 x r) . A^T (r x tokens) runs on
// v_mfma_f32_32x32x16_bf16: the MFMA "A" operand is a fragment of P (32 head slots x 16 ranks)
// read from LDS, the "B" operand is 16 B of a token's row of A^K loaded straight from global
// memory (lane (n, hf) holds ranks 16f + 8hf .. +7 of token n for fragment f), so A^K is
// streamed exactly once and never staged.  In the 32x32 result lane (n, hf) holds, for token n,
// the 16 head slots 8(v/4) + 4hf + v%4, v = 0..15.  Query heads are placed in slots so that all
// heads of a KV head sit in one lane's registers: the GQA max-pool needs no cross-lane traffic.
//
// Slot map: half hf holds gph = 16 / n_rep KV heads; KV head g sits in block g / (2 gph), half
// (g % (2 gph)) / gph, position u = g % gph, and its query head hh in register v = u n_rep + hh.
// P is kept as a sum of two bf16 values (high part and remainder) so that the scores carry
// fp32-accumulation accuracy even though the MFMA operands are bf16.
// ==========================================================================================
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;


__global__ __launch_bounds__(256) void project_q_frag_kernel(ProjArgs a)
{
    project_q_frag_block(a, blockIdx.x, blockIdx.y);
}

// One launch for the small passes that precede the score kernel and depend on nothing but the call's inputs: with TAIL first
// the blocks that attend over the uncompressed tail (dense_block.h), then n_proj blocks that project the queries, n_pack that make what
// the selected-row kernels need of q and (unless the caller brought a packed B) B_l (see prepass.h), and the rest clear the
// row histograms that the score kernel adds to (zero_words a multiple of 4).
// The tail was a launch of its own behind the selected rows: a few workgroups, 5 us for one round of loads, as long as the
// projection takes beside them (four layers of one sequence, ranks 512, 100 tokens of tail: 20 of 202 us).
template <bool TAIL>
__global__ __launch_bounds__(256, TAIL ? 2 : 1) void prepass_kernel(DenseArgs tail, int n_tail, ProjArgs pj, PackArgs pk, int n_proj,
                                                                    int n_pack, uint32_t *__restrict__ zero, int zero_words)
{
    int blk = (int)blockIdx.x;
    if constexpr (TAIL) {
        extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
        if (blk < n_tail) {
            const int row = blk / tail.splits;
            dense::mfma_block(tail, blk % tail.splits, row % tail.H_kv, row / tail.H_kv, smem);
            return;
        }
        blk -= n_tail;
    }
    if (blk < n_proj) {
        project_q_frag_block(pj, blk % pj.blocks_x, blk / pj.blocks_x);
    } else if (blk < n_proj + n_pack) {
        gather_prepare_block(pk, blk - n_proj);
    } else {
        const int i = 4 * ((blk - n_proj - n_pack) * 256 + (int)threadIdx.x);
        if (i < zero_words) *reinterpret_cast<u32x4_t *>(zero + i) = u32x4_t{0u, 0u, 0u, 0u};
    }
}

// The launch before the scores: projection of the queries into pj.Pfrag, and whatever of the rest is asked for.
static hipError_t launch_prepass(const xkv_shape &s, ProjArgs pj, const PackArgs *fuse_pack, const DenseArgs *tail, uint32_t *zero,
                                 int zero_words, hipStream_t st)
{
    if (!fuse_pack && !tail && zero_words == 0) {
        hipLaunchKernelGGL(project_q_frag_kernel, dim3(pj.blocks_x, s.batch), dim3(256), 0, st, pj);
        return hipGetLastError();
    }
    PackArgs pk = fuse_pack ? *fuse_pack : PackArgs{};
    const int n_rep = s.H_q / s.H_kv;
    // The selected-row kernel's projected queries are the same ones unless the scores come from other factors (landmarks).
    // Where a second pass has the chip's idle wavefronts to itself it is done sooner than the further stores of the first
    // (one sequence of 8 heads, ranks 512: 191 against 194 us for four layers; 16 sequences 1485 against 1470), and so with
    // one query head per KV head, where a wavefront stores more for less (16 sequences: 391 against 398).
    const bool same = pj.B_k && pj.B_k == pk.B_k && pj.q == pk.q && pj.layer == pk.layer && s.G == pk.G && s.r_k == pk.r_k &&
                      s.H_kv == pk.H_kv && s.H_q == pk.H_q && s.batch == pk.batch && pj.F8 == pk.FZ;
    if (same && pk.blocks_z > 0 && n_rep > 1 && (long long)s.batch * s.H_kv * (pj.F8 / 2) >= 512) {
        pj.Pz = pk.Pz;
        pj.z_stride = pk.z_stride;
        pk.blocks_z = 0;
    }
    const int n_proj = pj.blocks_x * s.batch, n_pack = fuse_pack ? pk.blocks() : 0, n_tail = tail ? tail->blocks() : 0;
    const dim3 grid(n_tail + n_proj + n_pack + (zero_words + 1023) / 1024);
    if (tail) {
        static DynamicLdsOnce attr;
        const hipError_t e = attr.ensure((const void *)prepass_kernel<true>, dense::kLdsBytes);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(prepass_kernel<true>, grid, dim3(256), dense::kLdsBytes, st, *tail, n_tail, pj, pk, n_proj, n_pack, zero,
                           zero_words);
    } else {
        hipLaunchKernelGGL(prepass_kernel<false>, grid, dim3(256), 0, st, DenseArgs{}, 0, pj, pk, n_proj, n_pack, zero, zero_words);
    }
    return hipGetLastError();
}

// Heads per KV head rounded up to a power of two: the row length of the per-head score array.
constexpr int head_pitch(int n_rep) { return n_rep <= 1 ? 1 : n_rep <= 2 ? 2 : n_rep <= 4 ? 4 : n_rep <= 8 ? 8 : 16; }

// HEADS: also write every query head's score, S_heads [batch][H_kv][L][head_pitch(N_REP)] (padding zero); the
// pooled score is the maximum of exactly those values.
template <int N_REP, bool HEADS>
__global__ __launch_bounds__(256) void score_mfma_kernel(const bf16_t *__restrict__ A_k,    // [batch][L][r_k]
                                                         const bf16_t *__restrict__ Pfrag,  // see above
                                                         float *__restrict__ S,             // [batch][H_kv][L]
                                                         int L, int r_k, int H_kv, int F8, int tiles_per_wg,
                                                         float scale, float *__restrict__ S_heads)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4_t *Pl = reinterpret_cast<u32x4_t *>(smem);  // [2][F8][64] fragments of 16 B per lane
    constexpr int GPH = 16 / N_REP;
    const int b = blockIdx.z, blk = blockIdx.y, nblk = gridDim.y;
    const int lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5;
    const int F = r_k / 16;

    // stage this block's P fragments (hi and lo parts) in LDS, eight 16 B loads in flight per thread
    {
        const u32x4_t *src = reinterpret_cast<const u32x4_t *>(Pfrag) + ((size_t)b * nblk + blk) * 2 * F8 * 64;
        const int total = 2 * F8 * 64;  // a multiple of 4 * 256
        for (int e0 = threadIdx.x; e0 < total; e0 += 4 * 256) {
            u32x4_t tmp[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) tmp[j] = src[e0 + j * 256];
#pragma unroll
            for (int j = 0; j < 4; ++j) Pl[e0 + j * 256] = tmp[j];
        }
    }
    __syncthreads();

    const bf16_t *Ab = A_k + (size_t)b * L * r_k;
    const int n_tiles = (L + 31) / 32;
    const int tile_begin = blockIdx.x * tiles_per_wg;
    const int tile_end = tile_begin + tiles_per_wg < n_tiles ? tile_begin + tiles_per_wg : n_tiles;
    const int n_steps = F8 / 8;  // steps of 8 fragments per tile
    // 16 B pieces of a token's row for one step; fragments beyond the rank meet zero P fragments, so the
    // address is only clamped, never skipped: the loop body is straight-line code
    auto load_step = [&](int tile, int step, u32x4_t (&a)[8]) __attribute__((always_inline)) {
        const int t = tile * 32 + n;
        const u32x4_t *row = reinterpret_cast<const u32x4_t *>(Ab + (size_t)(t < L ? t : L - 1) * r_k) + hf;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int f = step * 8 + j;
            a[j] = row[2 * (f < F ? f : F - 1)];
        }
    };
    int tile = tile_begin + w;
    if (tile >= tile_end) return;
    u32x4_t a_cur[8], a_nxt[8];
    load_step(tile, 0, a_cur);
    f32x16_t acc_h, acc_l;  // separate chains for the high parts and the remainders of P
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_h[v] = acc_l[v] = 0.0f;
    int step = 0;
    while (true) {
        // pieces of the next step (of this tile, or the first of the wavefront's next tile) before this step's MFMAs
        const bool last_step = step + 1 == n_steps;
        const int tile_n = last_step ? tile + 4 : tile, step_n = last_step ? 0 : step + 1;
        load_step(tile_n < tile_end ? tile_n : tile, step_n, a_nxt);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const u32x4_t ph = Pl[(step * 8 + j) * 64 + lane];
            const u32x4_t pl = Pl[(F8 + step * 8 + j) * 64 + lane];
            acc_h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ph),
                                                            __builtin_bit_cast(bf16x8_t, a_cur[j]), acc_h, 0, 0, 0);
            acc_l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pl),
                                                            __builtin_bit_cast(bf16x8_t, a_cur[j]), acc_l, 0, 0, 0);
        }
        if (last_step) {
            const int t = tile * 32 + n;
            if (t < L) {
#pragma unroll
                for (int u = 0; u < GPH; ++u) {
                    const int g = blk * 2 * GPH + hf * GPH + u;
                    if constexpr (HEADS) {
                        constexpr int NRP = head_pitch(N_REP);
                        float hv[16];
#pragma unroll
                        for (int hh = 0; hh < 16; ++hh)
                            hv[hh] = hh < N_REP ? scale * (acc_h[(u * N_REP + hh) & 15] + acc_l[(u * N_REP + hh) & 15]) : 0.0f;
                        float best = hv[0];
#pragma unroll
                        for (int hh = 1; hh < N_REP; ++hh) best = fmaxf(best, hv[hh]);
                        if (g < H_kv) {
                            S[((size_t)b * H_kv + g) * L + t] = best;
                            float *dst = S_heads + (((size_t)b * H_kv + g) * L + t) * NRP;
                            if constexpr (NRP >= 4) {
#pragma unroll
                                for (int c = 0; c < NRP / 4; ++c)
                                    *reinterpret_cast<float4 *>(dst + 4 * c) =
                                        make_float4(hv[4 * c], hv[4 * c + 1], hv[4 * c + 2], hv[4 * c + 3]);
                            } else {
#pragma unroll
                                for (int hh = 0; hh < NRP; ++hh) dst[hh] = hv[hh];
                            }
                        }
                    } else {
                        float best = acc_h[u * N_REP] + acc_l[u * N_REP];
#pragma unroll
                        for (int hh = 1; hh < N_REP; ++hh)
                            best = fmaxf(best, acc_h[u * N_REP + hh] + acc_l[u * N_REP + hh]);
                        if (g < H_kv) __builtin_nontemporal_store(scale * best, &S[((size_t)b * H_kv + g) * L + t]);
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_h[v] = acc_l[v] = 0.0f;
            if (tile_n >= tile_end) break;
        }
        tile = tile_n;
        step = step_n;
#pragma unroll
        for (int j = 0; j < 8; ++j) a_cur[j] = a_nxt[j];
    }
}

typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// One token's head scores (NRP consecutive floats, v[] already zero beyond the real heads), as hidden stores
// like the pooled ones below.
template <int NRP> __device__ __forceinline__ void store_head_row(float *dst, const float (&v)[16])
{
    if constexpr (NRP == 1) {
        asm volatile("global_store_dword %0, %1, off" : : "v"(dst), "v"(v[0]) : "memory");
    } else if constexpr (NRP == 2) {
        const f32x2_t x = {v[0], v[1]};
        asm volatile("global_store_dwordx2 %0, %1, off" : : "v"(dst), "v"(x) : "memory");
    } else {
#pragma unroll
        for (int c = 0; c < NRP / 4; ++c) {
            const f32x4_t x = {v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]};
            // (a store of more than 64 bits reads its data registers a cycle or two after issue; the compiler inserts
            // the wait states for stores it knows, not for these)
            asm volatile("global_store_dwordx4 %0, %1, off\n\ts_nop 1" : : "v"(dst + 4 * c), "v"(x) : "memory");
        }
    }
}

// The same for ranks above 256 where a wavefront has one tile, of several steps, and a compute unit one workgroup.  What counts there is how soon
// the rows are requested: the projected queries go straight to LDS, the first kScoreRing steps of rows (8 pieces of 16 B each) are
// requested behind them before anything is waited for, and a step's registers are refilled as soon as it is multiplied.  (With the
// projection, us: 9000 tokens of rank 512 12.0 -> 11.1, 32768 14.9 -> 14.3, 4096 of rank 768 14.0 -> 13.1.  With one or two steps, or several tiles per
// wavefront, the kernel above is as fast or ahead by up to 0.6.)
constexpr int kScoreRing = 4;

template <int N_REP, bool HEADS>
__global__ __launch_bounds__(256, 2) void score_ring_kernel(const bf16_t *__restrict__ A_k,    // [batch][L][r_k]
                                                            const bf16_t *__restrict__ Pfrag,  // see above
                                                            float *__restrict__ S,             // [batch][H_kv][L]
                                                            int L, int r_k, int H_kv, int F8, int tiles_per_wg,
                                                            float scale, float *__restrict__ S_heads)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4_t *Pl = reinterpret_cast<u32x4_t *>(smem);  // [2][F8][64] fragments of 16 B per lane
    constexpr int GPH = 16 / N_REP;
    const int b = blockIdx.z, blk = blockIdx.y, nblk = gridDim.y;
    const int lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5;
    const int F = r_k / 16;

    // this block's P fragments (hi and lo parts): 2 F8 KiB, each wavefront every fourth
    {
        const u32x4_t *src = reinterpret_cast<const u32x4_t *>(Pfrag) + ((size_t)b * nblk + blk) * 2 * F8 * 64 + lane;
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem;
        for (int f = w; f < 2 * F8; f += 4) copy16_global_to_lds(src + f * 64, lds0 + f * 1024);
    }
    const bf16_t *Ab = A_k + (size_t)b * L * r_k;
    const int n_tiles = (L + 31) / 32;
    const int tile_begin = blockIdx.x * tiles_per_wg;
    const int tile_end = tile_begin + tiles_per_wg < n_tiles ? tile_begin + tiles_per_wg : n_tiles;
    const int n_steps = F8 / 8;  // steps of 8 fragments per tile
    int tile = tile_begin + w;
    const bool has_work = tile < tile_end;
    // 16 B pieces of a token's row for one step; fragments beyond the rank meet zero P fragments, so the address is only
    // clamped, never skipped: the loop body is straight-line code.  (tile_p, step_p) is the step to request next; past the
    // wavefront's last tile every lane requests the same piece of one row.
    int tile_p = has_work ? tile : n_tiles - 1, step_p = 0, n_p = has_work ? n : 0, hf_p = has_work ? hf : 0;
    auto request = [&](u32x4_t (&a)[8]) __attribute__((always_inline)) {
        const int t = tile_p * 32 + n_p;
        const u32x4_t *row = reinterpret_cast<const u32x4_t *>(Ab + (size_t)(t < L ? t : L - 1) * r_k) + hf_p;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int f = step_p * 8 + j;
            a[j] = row[2 * (f < F ? f : F - 1)];
        }
        if (++step_p == n_steps) {
            step_p = 0;
            if (tile_p + 4 < tile_end) {
                tile_p += 4;
            } else {
                n_p = 0;
                hf_p = 0;
            }
        }
    };
    u32x4_t ring[kScoreRing][8];
#pragma unroll
    for (int s = 0; s < kScoreRing; ++s) {
        request(ring[s]);
        __builtin_amdgcn_sched_barrier(0);
    }
    XKV_WAIT_VMCNT(8 * kScoreRing);  // the copies of P came first
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (!has_work) return;
    f32x16_t acc_h, acc_l;  // separate chains for the high parts and the remainders of P
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_h[v] = acc_l[v] = 0.0f;
    const int my_steps = (tile_end - tile + 3) / 4 * n_steps;
    int step = 0;
    for (int i = 0; i < my_steps; i += kScoreRing) {
#pragma unroll
        for (int s = 0; s < kScoreRing; ++s) {
            const bool real = i + s < my_steps;  // (no way out of the loop here: it would make the waits for the ring stricter)
            if (real) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const u32x4_t ph = Pl[(step * 8 + j) * 64 + lane];
                    const u32x4_t pl = Pl[(F8 + step * 8 + j) * 64 + lane];
                    acc_h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ph),
                                                                    __builtin_bit_cast(bf16x8_t, ring[s][j]), acc_h, 0, 0, 0);
                    acc_l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pl),
                                                                    __builtin_bit_cast(bf16x8_t, ring[s][j]), acc_l, 0, 0, 0);
                }
            }
            request(ring[s]);
            __builtin_amdgcn_sched_barrier(0);
            if (!real || ++step < n_steps) continue;
            step = 0;
            // (stores that the compiler does not know of: it would wait for every request at the next use of the ring)
            const int t = tile * 32 + n;
            if (t < L) {
#pragma unroll
                for (int u = 0; u < GPH; ++u) {
                    const int g = blk * 2 * GPH + hf * GPH + u;
                    float hv[16];
#pragma unroll
                    for (int hh = 0; hh < 16; ++hh)
                        hv[hh] = hh < N_REP ? acc_h[(u * N_REP + hh) & 15] + acc_l[(u * N_REP + hh) & 15] : 0.0f;
                    if constexpr (HEADS) {
#pragma unroll
                        for (int hh = 0; hh < N_REP; ++hh) hv[hh] *= scale;
                    }
                    float best = hv[0];
#pragma unroll
                    for (int hh = 1; hh < N_REP; ++hh) best = fmaxf(best, hv[hh]);
                    if constexpr (!HEADS) best *= scale;
                    if (g < H_kv) {
                        asm volatile("global_store_dword %0, %1, off" : : "v"(&S[((size_t)b * H_kv + g) * L + t]), "v"(best) : "memory");
                        if constexpr (HEADS) {
                            constexpr int NRP = head_pitch(N_REP);
                            store_head_row<NRP>(S_heads + (((size_t)b * H_kv + g) * L + t) * NRP, hv);
                        }
                    }
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) acc_h[v] = acc_l[v] = 0.0f;
            tile += 4;
        }
    }
}

// Variant for long streams: the same contraction, but A^K is fetched line-wise and turned into operand
// fragments through a wavefront-private LDS tile.  A group is 128 ranks (256 B) of each of the wavefront's 32
// token rows; instruction j of a group covers rows 4j..4j+3, lane l loading the 16 B piece l%16 of row 4j + l/16,
// so every 128 B line is requested by exactly one instruction (with one lane per row, four instructions share
// each line and the stream runs well below the memory rate).  The tile is written row-wise, rotated by the row
// number so that neither side has bank conflicts (piece c of row t at 16 t + (c + t) % 16, in 16 B units), and
// read back as one fragment per step.  Two groups are in flight in registers per wavefront; nothing in the
// main loop needs a barrier (P is read-only in LDS, the tiles are private).
constexpr int kScoreWaves = 8;  // wavefronts per workgroup; 4 when the P fragments leave no room for 8 tiles

template <int SLOT0>
__device__ __forceinline__ void score_group(f32x16_t &acc_h, f32x16_t &acc_l, u32x4_t (&areg)[16], u32x4_t *At,
                                            const u32x4_t *Ph, const u32x4_t *Pl_, const u32x4_t *arow, int pieces,
                                            int t0, int row_step, int L, const int (&woff)[4], int rbase)
{
    // all but the 8 youngest loads (the other half of the ring) have landed: vmcnt(8), other counters untouched
    __builtin_amdgcn_s_waitcnt(8 | (7 << 4) | (0xF << 8));
#pragma unroll
    for (int j = 0; j < 8; ++j) At[64 * j + woff[j & 3]] = areg[SLOT0 + j];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int fl = 0; fl < 8; ++fl) {
        const bf16x8_t a0 = __builtin_bit_cast(bf16x8_t, At[(rbase & ~15) + ((rbase + 2 * fl) & 15)]);
        acc_h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, Ph[fl * 64]), a0, acc_h, 0, 0, 0);
        acc_l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, Pl_[fl * 64]), a0, acc_l, 0, 0, 0);
        // instruction fl of the group two groups on, into the ring entry written out above
        const int t = t0 + row_step * fl;
        areg[SLOT0 + fl] = __builtin_nontemporal_load(&arow[(size_t)(t < L ? t : L - 1) * pieces]);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// HEADS: also write every query head's score, S_heads [batch][H_kv][L][head_pitch(N_REP)] (padding zero); the
// pooled score is the maximum of exactly those values.
template <int N_REP, int WAVES, bool HEADS>
__global__ __launch_bounds__(WAVES * 64) void score_stream_kernel(const bf16_t *__restrict__ A_k,
                                                                        const bf16_t *__restrict__ Pfrag,
                                                                        float *__restrict__ S, int L, int r_k,
                                                                        int H_kv, int F8, int tiles_per_wg,
                                                                        float scale, uint32_t *__restrict__ row_hist,
                                                                        uint32_t *__restrict__ chunk_hist,
                                                                        float *__restrict__ S_heads)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4_t *Pl = reinterpret_cast<u32x4_t *>(smem);  // [2][F8][64] fragments of 16 B per lane
    constexpr int GPH = 16 / N_REP;
    // Pooled scores are kept in registers and written in bursts of RT tiles: 4 B per (KV head, token) are only 3 %
    // of the bytes, but dribbled out between the reads they cost the memory system as much as 15 % of the stream.
    // (with HEADS all 16 head slots of a tile are kept instead, and bursts are four tiles)
    constexpr int RT = HEADS ? 4 : 64 / GPH;
    constexpr int RW = HEADS ? 16 : GPH;
    constexpr int NRP = head_pitch(N_REP);
    const int b = blockIdx.z, blk = blockIdx.y, nblk = gridDim.y;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5;
    u32x4_t *At = Pl + 2 * F8 * 64 + w * 512;
    // Optional first pass of the top-k stage: histogram of the top 8 bits of the order key of every pooled
    // score of this workgroup, one 256-bin histogram per KV head slot of the block.
    uint32_t *hist = reinterpret_cast<uint32_t *>(Pl + 2 * F8 * 64 + WAVES * 512);  // [2 GPH][256]
    const bool do_hist = row_hist != nullptr;
    if (do_hist)
        for (int i = tid; i < 2 * GPH * kTopkBins; i += WAVES * 64) hist[i] = 0;

    const int pieces = r_k >> 3;  // 16 B pieces per row
    const u32x4_t *Ab = reinterpret_cast<const u32x4_t *>(A_k + (size_t)b * L * r_k);
    const int n_tiles = (L + 31) / 32;
    const int n_groups = F8 / 8;  // groups per tile
    const int wg_end = (blockIdx.x + 1) * tiles_per_wg < n_tiles ? (blockIdx.x + 1) * tiles_per_wg : n_tiles;
    // The wavefronts of a workgroup interleave their tiles (stride TS), so that at any moment the workgroup reads
    // one compact window of the sequence: measurably faster than eight separate runs per workgroup.
    constexpr int TS = WAVES;
    int tile = blockIdx.x * tiles_per_wg + w;
    const int tile_end = wg_end;
    const bool has_work = tile < tile_end;  // wave-uniform

    int woff[4];
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) woff[qd] = 16 * (lane >> 4) + (((lane & 15) + (lane >> 4) + 4 * qd) & 15);
    const int rbase = 16 * n + ((hf + n) & 15);
    // this lane's piece of group S (beyond the row: piece 0, it meets zero P fragments) and first row of a tile
    auto piece_of = [&](int S_) __attribute__((always_inline)) {
        const int pc = 16 * S_ + (lane & 15);
        return pc < pieces ? pc : 0;
    };
    const int trow = lane >> 4;

    // first part of this block's P fragments (hi and lo parts), eight 16 B loads in flight per thread ...
    const u32x4_t *psrc = reinterpret_cast<const u32x4_t *>(Pfrag) + ((size_t)b * nblk + blk) * 2 * F8 * 64;
    const int total = 2 * F8 * 64;  // a multiple of 1024
    u32x4_t ptmp[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int e0 = tid + j * WAVES * 64;
        ptmp[j] = psrc[e0 < total ? e0 : tid];
    }
    // ... and behind them already the first two groups of A^K.  (tile, group) two groups ahead of the one being
    // multiplied; past the end it stays on the last tile.
    int tile_p = has_work ? tile : 0, S_p = 0;
    // (the prefetches keep being issued past the wavefront's last tile -- the waits count outstanding loads -- but
    // then every one of them goes to one row, a cache hit, instead of streaming the last tile from memory again)
    int row_step = 4, row_lane = 1;  // rows between the instructions of a group, and between a lane's row and lane/16
    auto advance_p = [&]() __attribute__((always_inline)) {
        if (++S_p == n_groups) {
            S_p = 0;
            if (tile_p + TS < tile_end) {
                tile_p += TS;
            } else {
                row_step = 0;
                row_lane = 0;
            }
        }
    };
    u32x4_t areg[16];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const u32x4_t *arow = Ab + piece_of(S_p);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int t = tile_p * 32 + trow + 4 * j;
            areg[half * 8 + j] = __builtin_nontemporal_load(&arow[(size_t)(t < L ? t : L - 1) * pieces]);
            __builtin_amdgcn_sched_barrier(0);
        }
        advance_p();
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int e0 = tid + j * WAVES * 64;
        if (e0 < total) Pl[e0] = ptmp[j];
    }
    for (int e0 = tid + 8 * WAVES * 64; e0 < total; e0 += 2 * WAVES * 64) {
        u32x4_t tmp[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) tmp[j] = psrc[e0 + j * WAVES * 64];
#pragma unroll
        for (int j = 0; j < 2; ++j) Pl[e0 + j * WAVES * 64] = tmp[j];
    }
    __syncthreads();
    if (has_work) {
    f32x16_t acc_h, acc_l;  // separate chains for the high parts and the remainders of P
#pragma unroll
    for (int v = 0; v < 16; ++v) acc_h[v] = acc_l[v] = 0.0f;
    float res[RT][RW];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int u = 0; u < RW; ++u) res[i][u] = 0.0f;
    int S_c = 0, ti = 0, tile0 = tile;  // group within the tile, tiles held in res, first of them
    // Stores go through inline assembly: a store the compiler knows of inside conditional code makes its count of
    // outstanding memory operations uncertain, and it then waits for *all* prefetches at the top of the loop.
    // Unknown to it, the stores only make those waits stricter for a moment.
    auto flush = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const int t = (tile0 + i * TS) * 32 + n;
            if (i < ti && t < L) {
#pragma unroll
                for (int u = 0; u < GPH; ++u) {
                    const int g = blk * 2 * GPH + hf * GPH + u;
                    if (g < H_kv) {
                        float *dst = S + ((size_t)b * H_kv + g) * L + t;
                        if constexpr (HEADS) {
                            float hv[16];
#pragma unroll
                            for (int hh = 0; hh < 16; ++hh) hv[hh] = hh < N_REP ? res[i][(u * N_REP + hh) & 15] : 0.0f;
                            float best = hv[0];
#pragma unroll
                            for (int hh = 1; hh < N_REP; ++hh) best = fmaxf(best, hv[hh]);
                            asm volatile("global_store_dword %0, %1, off" : : "v"(dst), "v"(best) : "memory");
                            store_head_row<NRP>(S_heads + (((size_t)b * H_kv + g) * L + t) * NRP, hv);
                        } else {
                            asm volatile("global_store_dword %0, %1, off" : : "v"(dst), "v"(res[i][u]) : "memory");
                        }
                    }
                }
            }
        }
        tile0 += ti * TS;
        ti = 0;
    };
    auto finish_group = [&]() __attribute__((always_inline)) {  // closes a tile after its last group
        if (++S_c < n_groups) return;
        S_c = 0;
#pragma unroll
        for (int u = 0; u < GPH; ++u) {
            float best = acc_h[u * N_REP] + acc_l[u * N_REP];
#pragma unroll
            for (int hh = 1; hh < N_REP; ++hh) best = fmaxf(best, acc_h[u * N_REP + hh] + acc_l[u * N_REP + hh]);
            best *= scale;
            if constexpr (HEADS) {
#pragma unroll
                for (int hh = 0; hh < N_REP; ++hh) {
                    const float hs = scale * (acc_h[u * N_REP + hh] + acc_l[u * N_REP + hh]);
#pragma unroll
                    for (int i = 0; i < RT; ++i) res[i][u * N_REP + hh] = (i == ti) ? hs : res[i][u * N_REP + hh];
                }
            } else {
#pragma unroll
                for (int i = 0; i < RT; ++i) res[i][u] = (i == ti) ? best : res[i][u];
            }
            if (do_hist) {
                // Done per tile, where it hides behind the other wavefronts' memory waits.  Scores cluster in few
                // bins: one LDS add per distinct (head slot, bin) of the wavefront.
                const int g = blk * 2 * GPH + hf * GPH + u;
                const uint32_t slot = (uint32_t)(hf * GPH + u) * kTopkBins + (order_key(best) >> 24);
                const bool active = tile * 32 + n < L && g < H_kv;
                uint64_t m = __ballot(active);
                while (m != 0) {
                    const int first = __ffsll((unsigned long long)m) - 1;
                    const uint32_t s0 = (uint32_t)__builtin_amdgcn_readlane((int)slot, first);
                    const uint64_t same = __ballot(active && slot == s0);
                    if (lane == first) atomicAdd(&hist[s0], (uint32_t)__popcll(same));
                    m &= ~same;
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc_h[v] = acc_l[v] = 0.0f;
        tile += TS;
        ++ti;
    };
    // groups of this wavefront, two per iteration (one per half of the ring); an odd total leaves one surplus
    // group at the end, which multiplies re-fetched rows of the last tile and is dropped
    const int my_groups = (tile_end - tile + TS - 1) / TS * n_groups;
    for (int gi = 0; gi < my_groups; gi += 2) {
        {
            const u32x4_t *arow = Ab + piece_of(S_p);
            const int t0 = tile_p * 32 + trow * row_lane, rs = row_step;
            advance_p();
            score_group<0>(acc_h, acc_l, areg, At, Pl + (S_c * 8) * 64 + lane, Pl + (F8 + S_c * 8) * 64 + lane, arow,
                           pieces, t0, rs, L, woff, rbase);
            finish_group();
        }
        {
            const u32x4_t *arow = Ab + piece_of(S_p);
            const int t0 = tile_p * 32 + trow * row_lane, rs = row_step;
            advance_p();
            score_group<8>(acc_h, acc_l, areg, At, Pl + (S_c * 8) * 64 + lane, Pl + (F8 + S_c * 8) * 64 + lane, arow,
                           pieces, t0, rs, L, woff, rbase);
            if (gi + 1 < my_groups) finish_group();
        }
        if (ti > RT - 2) flush();  // up to two tiles complete per iteration
    }
    flush();
    }
    if (do_hist) {
        // this workgroup is chunk blockIdx.x of its rows: keep the chunk histograms, add them to the rows'
        __syncthreads();
        const int chunks = gridDim.x;
        for (int i = tid; i < 2 * GPH * kTopkBins; i += WAVES * 64) {
            const int g = blk * 2 * GPH + i / kTopkBins, bin = i % kTopkBins;
            if (g < H_kv) {
                const size_t row = (size_t)b * H_kv + g;
                const uint32_t cnt = hist[i];
                chunk_hist[(row * chunks + blockIdx.x) * kTopkLevels * kTopkBins + bin] = cnt;
                if (cnt != 0) atomicAdd(&row_hist[row * kTopkLevels * kTopkBins + bin], cnt);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Scores from a 4-bit quantised token basis (quant.hip: per row r/8 words of codes, then (step, lo) per group of
// 32 ranks).  Same contraction and head-slot layout as above, with the codes themselves as the matrix-core
// operand: a code c in 0..15 is the bf16 number 128 + c when 0x4300 is or-ed on top of it, and a pair of adjacent
// ranks is one shift and one mask away from a packed bf16 pair.  Per group g and token t the matrix cores give
//   acc_g[slot] = sum_{i in g} (128 + c_ti) p[slot][i]      (exact products, fp32 sums, P as bf16 hi + lo)
// and the affine map of the group is applied to the sum, not to the elements:
//   s[slot] += step_tg (acc_g[slot] - 128 Ps_g[slot]) + lo_tg Ps_g[slot],   Ps_g[slot] = sum_{i in g} p[slot][i].
// (In this kernel the second part is kept in fp32 multiply-adds; the line-wise kernel below runs it on the matrix
// cores with exact three-way splits.)
// Lane (n, hf) loads the 16 bytes of each of token n's groups (both halves load the same pieces) and the parameter
// words.  Always writes the per-head scores as well as the pooled ones.
// ------------------------------------------------------------------------------------------
// (above: 0x43004300, in a register: an and-or instruction takes one constant)
__device__ __forceinline__ bf16x8_t q4_fragment(uint32_t w, uint32_t above = 0x43004300u)
{
    u32x4_t o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = ((w >> (4 * i)) & 0x000F000Fu) | above;
    return __builtin_bit_cast(bf16x8_t, o);
}

// One pass of a token's quantised row: GP groups of codes from group g0 on (clamped to the last real group) and
// their parameter words.  n_groups is a multiple of 4.
template <int GP>
__device__ __forceinline__ void q4_load_pass(u32x4_t (&cw)[GP], u32x4_t (&pw)[GP / 4], const unsigned char *Ab, size_t pitch,
                                             int r_k, int t, int L, int g0, int n_groups)
{
    const unsigned char *rowp = Ab + (size_t)(t < L ? t : L - 1) * pitch;
    const u32x4_t *codes = reinterpret_cast<const u32x4_t *>(rowp);
    const u32x4_t *params = reinterpret_cast<const u32x4_t *>(rowp + (r_k >> 1));
#pragma unroll
    for (int j = 0; j < GP; ++j) cw[j] = codes[g0 + j < n_groups ? g0 + j : n_groups - 1];
#pragma unroll
    for (int j = 0; j < GP / 4; ++j) pw[j] = params[g0 + 4 * j < n_groups ? (g0 >> 2) + j : (n_groups >> 2) - 1];
}

template <int N_REP, int WAVES, int GP>
__global__ __launch_bounds__(WAVES * 64) void score_q4_kernel(const unsigned char *__restrict__ Aq,  // [batch][L][5 r_k / 8]
                                                       const bf16_t *__restrict__ Pfrag, float *__restrict__ S,
                                                       float *__restrict__ S_heads, int L, int r_k, int H_kv, int F8,
                                                       int tiles_per_wg, float scale)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    u32x4_t *Pl = reinterpret_cast<u32x4_t *>(smem);                   // [2][F8][64] fragments of 16 B per lane
    float *Ps = reinterpret_cast<float *>(Pl + 2 * F8 * 64);            // [F8 / 2 groups][32 slots]
    constexpr int GPH = 16 / N_REP;
    constexpr int NRP = head_pitch(N_REP);
    const int b = blockIdx.z, blk = blockIdx.y, nblk = gridDim.y;
    const int lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5;
    const int n_groups = r_k >> 5;  // = F8 / 2 for the ranks this kernel takes (multiples of 128)
    {
        const u32x4_t *src = reinterpret_cast<const u32x4_t *>(Pfrag) + ((size_t)b * nblk + blk) * 2 * F8 * 64;
        const int total = 2 * F8 * 64;  // a multiple of 1024
        for (int e0 = threadIdx.x; e0 < total; e0 += 4 * WAVES * 64) {
            u32x4_t tmp[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) tmp[j] = src[e0 + j * WAVES * 64 < total ? e0 + j * WAVES * 64 : e0];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (e0 + j * WAVES * 64 < total) Pl[e0 + j * WAVES * 64] = tmp[j];
        }
    }
    __syncthreads();
    // Ps: lane (slot m, hf) sums its 8 ranks of both fragments and both parts of a group, the halves are added
    for (int g = w; g < F8 / 2; g += WAVES) {
        float sum = 0.0f;
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
            for (int ff = 0; ff < 2; ++ff) {
                const u32x4_t v = Pl[(part * F8 + 2 * g + ff) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) sum += __uint_as_float(v[e] << 16) + __uint_as_float(v[e] & 0xFFFF0000u);
            }
        sum += __shfl_xor(sum, 32, kWave);
        if (hf == 0) Ps[g * 32 + n] = sum;
    }
    __syncthreads();

    const size_t pitch = (size_t)r_k * 5 / 8;
    const unsigned char *Ab = Aq + (size_t)b * L * pitch;
    const int n_tiles = (L + 31) / 32;
    const int tile_begin = blockIdx.x * tiles_per_wg;
    const int tile_end = tile_begin + tiles_per_wg < n_tiles ? tile_begin + tiles_per_wg : n_tiles;
    // A token's row is requested a pass at a time (a pass = GP groups = 16 GP bytes of codes and 4 GP bytes of
    // parameters per lane), and the next pass -- of this tile or of the wavefront's next tile -- is requested
    // before the products of the current one: with one group in flight per lane the stream is bound by load
    // latency, not by bytes.
    const int n_pass = (n_groups + GP - 1) / GP;
    int tile = tile_begin + w;
    if (tile >= tile_end) return;
    u32x4_t cw[GP], pw[GP / 4];
    q4_load_pass<GP>(cw, pw, Ab, pitch, r_k, tile * 32 + n, L, 0, n_groups);
    f32x16_t tot;
#pragma unroll
    for (int v = 0; v < 16; ++v) tot[v] = 0.0f;
    const f32x16_t zero = tot;
    int pass = 0;
    while (true) {
        const bool last_pass = pass + 1 == n_pass;
        const int tile_n = last_pass ? tile + WAVES : tile, pass_n = last_pass ? 0 : pass + 1;
        u32x4_t cw_n[GP], pw_n[GP / 4];
        q4_load_pass<GP>(cw_n, pw_n, Ab, pitch, r_k, (tile_n < tile_end ? tile_n : tile) * 32 + n, L, pass_n * GP, n_groups);
        const int g0 = pass * GP;
#pragma unroll
        for (int j = 0; j < GP; ++j) {
            const int g = g0 + j;
            if (g < n_groups) {  // wave-uniform
                f32x16_t acc = zero;
#pragma unroll
                for (int ff = 0; ff < 2; ++ff) {
                    // fragment 2g + ff covers ranks 32g + 16ff ..; this half takes word 2ff + hf of the group
                    const uint32_t word = hf ? (ff ? cw[j][3] : cw[j][1]) : (ff ? cw[j][2] : cw[j][0]);
                    const bf16x8_t bop = q4_fragment(word);
                    const u32x4_t ph = Pl[(2 * g + ff) * 64 + lane];
                    const u32x4_t pl = Pl[(F8 + 2 * g + ff) * 64 + lane];
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ph), bop, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pl), bop, acc, 0, 0, 0);
                }
                const uint32_t pword = pw[j >> 2][j & 3];
                const float step = __uint_as_float(pword << 16), lo = __uint_as_float(pword & 0xFFFF0000u);
                const float c2 = fmaf(-128.0f, step, lo);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float4 ps = *reinterpret_cast<const float4 *>(Ps + g * 32 + 8 * i + 4 * hf);
                    tot[4 * i + 0] = fmaf(step, acc[4 * i + 0], fmaf(c2, ps.x, tot[4 * i + 0]));
                    tot[4 * i + 1] = fmaf(step, acc[4 * i + 1], fmaf(c2, ps.y, tot[4 * i + 1]));
                    tot[4 * i + 2] = fmaf(step, acc[4 * i + 2], fmaf(c2, ps.z, tot[4 * i + 2]));
                    tot[4 * i + 3] = fmaf(step, acc[4 * i + 3], fmaf(c2, ps.w, tot[4 * i + 3]));
                }
            }
        }
#pragma unroll
        for (int j = 0; j < GP; ++j) cw[j] = cw_n[j];
#pragma unroll
        for (int j = 0; j < GP / 4; ++j) pw[j] = pw_n[j];
        if (!last_pass) {
            pass = pass_n;
            continue;
        }
        const int t = tile * 32 + n;
        if (t < L) {
#pragma unroll
            for (int u = 0; u < GPH; ++u) {
                const int g = blk * 2 * GPH + hf * GPH + u;
                if (g < H_kv) {
                    float hv[16];
#pragma unroll
                    for (int hh = 0; hh < 16; ++hh) hv[hh] = hh < N_REP ? scale * tot[(u * N_REP + hh) & 15] : 0.0f;
                    float best = hv[0];
#pragma unroll
                    for (int hh = 1; hh < N_REP; ++hh) best = fmaxf(best, hv[hh]);
                    S[((size_t)b * H_kv + g) * L + t] = best;
                    float *dst = S_heads + (((size_t)b * H_kv + g) * L + t) * NRP;
                    if constexpr (NRP >= 4) {
#pragma unroll
                        for (int c = 0; c < NRP / 4; ++c)
                            *reinterpret_cast<float4 *>(dst + 4 * c) =
                                make_float4(hv[4 * c], hv[4 * c + 1], hv[4 * c + 2], hv[4 * c + 3]);
                    } else {
#pragma unroll
                        for (int hh = 0; hh < NRP; ++hh) dst[hh] = hv[hh];
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) tot[v] = 0.0f;
        if (tile_n >= tile_end) break;
        tile = tile_n;
        pass = 0;
    }
}

// The same kernel with the rows fetched line-wise: the 32 token rows of a tile are one contiguous block of
// 32 * 5r/8 bytes, which a wavefront requests as whole 1 KiB runs (lane l = 16-byte piece i * 64 + l, NL requests)
// and passes to the lanes that need them through a wavefront-private LDS tile.  With one lane per row (kernel
// above) every request touches 32 different lines and the load path, not the arithmetic, bounds the kernel (measured:
// 81 of 175 us).  Rows sit in the tile at a pitch of an odd number of 16-byte units, so the per-row reads are free
// of bank conflicts.  The next tile waits in registers while the current one is multiplied; nothing needs a
// barrier (P is read-only, the tiles are private).
// What bounds it: vector instructions (900 per tile of 32 tokens at ranks 512, of which 450 are the codes' conversion and the groups'
// multiply-adds) and matrix instructions (70), which two wavefronts per SIMD overlap only in part, and the stores, 20 bytes per
// token and KV head.  Two groups of 32 ranks go side by side, so that neither waits for the other's products; the first tile is
// requested with the operands, awaited after them; a tile's results are stored as they come (held back for bursts of four tiles
// they cost registers, and at the end of a short range nothing was left to hide them behind).  4 x 65536 tokens of ranks 512
// 37.4 -> 34.2 us, 16 x 65536 with the projection 134 -> 121, 7 query heads 4 x 131072 of 384 61 -> 53.
constexpr int kQ4TileWaves = 8;
constexpr int kQ4MaxLoads = 10;  // 16-byte requests per lane and tile: 32 rows * 5r/8 bytes <= 10 KiB, r <= 512

__host__ __device__ inline int q4_tile_pitch(int r) { return r * 5 / 8 + ((r / 128) % 2 == 0 ? 16 : 0); }  // bytes
// (the offset term reads a row's parameters in runs of 64 bytes; the last run may reach up to 48 bytes past the
// row, into the next row of the tile or, for the last row, the 64 bytes of slack behind the wavefront's tile)
constexpr int kQ4TileSlack = 64;

template <int N_REP>
__global__ __launch_bounds__(kQ4TileWaves * 64) void score_q4_tile_kernel(const unsigned char *__restrict__ Aq,
                                                                          const bf16_t *__restrict__ Pfrag,
                                                                          float *__restrict__ S,
                                                                          float *__restrict__ S_heads, int L, int r_k,
                                                                          int H_kv, int F8, int tiles_per_wg, float scale)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int WAVES = kQ4TileWaves;
    u32x4_t *Pl = reinterpret_cast<u32x4_t *>(smem);         // [2][F8][64] fragments of 16 B per lane
    float *Ps = reinterpret_cast<float *>(Pl + 2 * F8 * 64);  // [F8 / 2 groups][32 slots]
    constexpr int GPH = 16 / N_REP;
    constexpr int NRP = head_pitch(N_REP);
    const int b = blockIdx.z, blk = blockIdx.y, nblk = gridDim.y;
    const int lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5;
    const int n_groups = r_k >> 5;
    const int tpitch = q4_tile_pitch(r_k);
    const int n_pass = (n_groups + 15) >> 4;  // passes of 16 groups of the offset term
    u32x4_t *PsF = reinterpret_cast<u32x4_t *>(Ps + (F8 / 2) * 32);  // [n_pass][3 parts][64]: Ps as operand fragments
    unsigned char *tile_lds = reinterpret_cast<unsigned char *>(PsF + n_pass * 3 * 64) + (size_t)w * (32 * tpitch + kQ4TileSlack);
    const int pitch = r_k * 5 / 8;
    const int ppr = pitch >> 4;            // 16-byte pieces per row
    const int pieces = 32 * ppr;           // per tile
    const unsigned char *Ab = Aq + (size_t)b * L * pitch;
    const size_t seq_last = (size_t)L * pitch - 16;  // last piece of the sequence: requests beyond it are redirected
    const int n_tiles = (L + 31) / 32;
    const int tile_begin = blockIdx.x * tiles_per_wg;
    const int tile_end = tile_begin + tiles_per_wg < n_tiles ? tile_begin + tiles_per_wg : n_tiles;
    int tile = tile_begin + w;
    u32x4_t stage[kQ4MaxLoads];
    // (a tile whose requests all lie within the sequence, all but the last ones: one address and constant offsets)
    auto request = [&](int tl) __attribute__((always_inline)) {
        const size_t at = (size_t)tl * 32 * pitch;
        if (at + kQ4MaxLoads * 1024 <= seq_last + 16) {
            const unsigned char *from = Ab + at;
#pragma unroll
            for (int i = 0; i < kQ4MaxLoads; ++i)
                stage[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(from + (uint32_t)(lane * 16) + i * 1024));
        } else {
#pragma unroll
            for (int i = 0; i < kQ4MaxLoads; ++i) {
                const size_t off = at + (size_t)(i * 64 + lane) * 16;
                stage[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(Ab + (off < seq_last ? off : seq_last)));
            }
        }
    };
    {
        const u32x4_t *src = reinterpret_cast<const u32x4_t *>(Pfrag) + ((size_t)b * nblk + blk) * 2 * F8 * 64;
        const int total = 2 * F8 * 64;  // a multiple of 1024, and no more than 4096 (r <= 512)
        u32x4_t tmp[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) tmp[j] = src[(int)threadIdx.x + j * WAVES * 64 < total ? threadIdx.x + j * WAVES * 64 : threadIdx.x];
        request(tile);  // (behind the operands, which are awaited first; a wavefront without a tile asks for the sequence's last bytes)
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if ((int)threadIdx.x + j * WAVES * 64 < total) Pl[threadIdx.x + j * WAVES * 64] = tmp[j];
    }
    lds_barrier();
    for (int g = w; g < F8 / 2; g += WAVES) {
        float sum = 0.0f;
#pragma unroll
        for (int part = 0; part < 2; ++part)
#pragma unroll
            for (int ff = 0; ff < 2; ++ff) {
                const u32x4_t v = Pl[(part * F8 + 2 * g + ff) * 64 + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) sum += __uint_as_float(v[e] << 16) + __uint_as_float(v[e] & 0xFFFF0000u);
            }
        sum += __shfl_xor(sum, 32, kWave);
        if (hf == 0) Ps[g * 32 + n] = sum;
    }
    lds_barrier();
    // The offset term sum_g (lo_tg - 128 step_tg) Ps_g[slot] is a product [slots x groups] . [groups x tokens] and
    // runs on the matrix cores, 16 groups per instruction.  Because 128 step Ps cancels against the first term it
    // needs full fp32 accuracy: both factors are split *exactly* into three bf16 numbers (8 + 8 + 8 mantissa bits,
    // by truncation) and the six largest of the nine partial products are taken; the dropped ones are below 2^-24
    // of the term.  Here: Ps as operand fragments, lane (slot m, hf), position e = group 16 pass + 8 hf + e.
    for (int ps = w; ps < n_pass; ps += WAVES) {
        u32x4_t f3[3];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
            uint32_t part[2][3];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const int g = 16 * ps + 8 * hf + 2 * e2 + o;
                float v = g < n_groups ? Ps[g * 32 + n] : 0.0f;
#pragma unroll
                for (int q3 = 0; q3 < 3; ++q3) {
                    part[o][q3] = __float_as_uint(v) & 0xFFFF0000u;
                    v -= __uint_as_float(part[o][q3]);
                }
            }
#pragma unroll
            for (int q3 = 0; q3 < 3; ++q3) f3[q3][e2] = (part[0][q3] >> 16) | part[1][q3];
        }
#pragma unroll
        for (int q3 = 0; q3 < 3; ++q3) PsF[(ps * 3 + q3) * 64 + lane] = f3[q3];
    }
    lds_barrier();

    if (tile >= tile_end) return;
    // where this lane's pieces go in the LDS tile (the same for every tile); -1: no such piece
    int dst_off[kQ4MaxLoads];
#pragma unroll
    for (int i = 0; i < kQ4MaxLoads; ++i) {
        const int pc = i * 64 + lane;
        dst_off[i] = pc < pieces ? (pc / ppr) * tpitch + (pc % ppr) * 16 : -1;
    }
    f32x16_t tot;
#pragma unroll
    for (int v = 0; v < 16; ++v) tot[v] = 0.0f;
    const f32x16_t zero = tot;
    const unsigned char *my_row = tile_lds + n * tpitch;
    uint32_t above = 0x43004300u;
    asm("" : "+v"(above));
    while (true) {
#pragma unroll
        for (int i = 0; i < kQ4MaxLoads; ++i)
            if (64 * (i + 1) <= pieces || dst_off[i] >= 0) *reinterpret_cast<u32x4_t *>(tile_lds + dst_off[i]) = stage[i];
        const int tile_n = tile + WAVES;
        request(tile_n < tile_end ? tile_n : tile);
        for (int ps = 0; ps < n_pass; ++ps) {
            // (lo - 128 step) of this half's eight groups of the pass, split like Ps
            const u32x4_t *par = reinterpret_cast<const u32x4_t *>(my_row + (r_k >> 1) + 64 * ps + 32 * hf);
            const u32x4_t pa = par[0], pb = par[1];
            u32x4_t c3[3];
#pragma unroll
            for (int e2 = 0; e2 < 4; ++e2) {
                uint32_t part[2][3];
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    const int e = 2 * e2 + o;
                    const uint32_t pword = e < 4 ? pa[e & 3] : pb[e & 3];
                    float v = fmaf(-128.0f, __uint_as_float(pword << 16), __uint_as_float(pword & 0xFFFF0000u));
                    v = 16 * ps + 8 * hf + e < n_groups ? v : 0.0f;  // beyond the row: whatever the tile holds there
#pragma unroll
                    for (int q3 = 0; q3 < 3; ++q3) {
                        part[o][q3] = __float_as_uint(v) & 0xFFFF0000u;
                        v -= __uint_as_float(part[o][q3]);
                    }
                }
#pragma unroll
                for (int q3 = 0; q3 < 3; ++q3) c3[q3][e2] = (part[0][q3] >> 16) | part[1][q3];
            }
            const u32x4_t *pf = PsF + ps * 3 * 64 + lane;
            const bf16x8_t p0 = __builtin_bit_cast(bf16x8_t, pf[0]), p1 = __builtin_bit_cast(bf16x8_t, pf[64]);
            const bf16x8_t p2 = __builtin_bit_cast(bf16x8_t, pf[128]);
            const bf16x8_t c0 = __builtin_bit_cast(bf16x8_t, c3[0]), c1 = __builtin_bit_cast(bf16x8_t, c3[1]);
            const bf16x8_t c2v = __builtin_bit_cast(bf16x8_t, c3[2]);
            // smallest products first
            tot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1, c1, tot, 0, 0, 0);
            tot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p2, c0, tot, 0, 0, 0);
            tot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0, c2v, tot, 0, 0, 0);
            tot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p1, c0, tot, 0, 0, 0);
            tot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0, c1, tot, 0, 0, 0);
            tot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p0, c0, tot, 0, 0, 0);
        }
        // Four groups a round (a row's groups are a multiple of that), two at a time: their products do not wait for each other.  The codes of
        // the next two are on their way.
        u32x4_t codes[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) codes[j] = *reinterpret_cast<const u32x4_t *>(my_row + 16 * j);
        for (int g4 = 0; g4 < n_groups; g4 += 4) {
            const u32x4_t par = *reinterpret_cast<const u32x4_t *>(my_row + (r_k >> 1) + 4 * g4);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int g = g4 + 2 * h;
                f32x16_t acc[2];
                u32x4_t ph[2][2], pl[2][2];
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int ff = 0; ff < 2; ++ff) {
                        ph[j][ff] = Pl[(2 * (g + j) + ff) * 64 + lane];
                        pl[j][ff] = Pl[(F8 + 2 * (g + j) + ff) * 64 + lane];
                    }
                uint32_t now[2][2];
                const int gn = g + 2 < n_groups ? g + 2 : 0;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
#pragma unroll
                    for (int ff = 0; ff < 2; ++ff) now[j][ff] = hf ? codes[j][2 * ff + 1] : codes[j][2 * ff];
                    codes[j] = *reinterpret_cast<const u32x4_t *>(my_row + 16 * (gn + j));
                }
#pragma unroll
                for (int ff = 0; ff < 2; ++ff) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const bf16x8_t c8 = q4_fragment(now[j][ff], above);
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ph[j][ff]), c8, ff == 0 ? zero : acc[j], 0, 0, 0);
                        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, pl[j][ff]), c8, acc[j], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const float step = __uint_as_float(par[2 * h + j] << 16);
#pragma unroll
                    for (int v = 0; v < 16; ++v) tot[v] = fmaf(step, acc[j][v], tot[v]);
                }
            }
        }
        const int t = tile * 32 + n;
        if (t < L) {
#pragma unroll
            for (int u = 0; u < GPH; ++u) {
                const int g = blk * 2 * GPH + hf * GPH + u;
                if (g < H_kv) {
                    float hv[16];
#pragma unroll
                    for (int hh = 0; hh < 16; ++hh) hv[hh] = hh < N_REP ? scale * tot[(u * N_REP + hh) & 15] : 0.0f;
                    float best = hv[0];
#pragma unroll
                    for (int hh = 1; hh < N_REP; ++hh) best = fmaxf(best, hv[hh]);
                    S[((size_t)b * H_kv + g) * L + t] = best;
                    float *dst = S_heads + (((size_t)b * H_kv + g) * L + t) * NRP;
                    if constexpr (NRP >= 4) {
#pragma unroll
                        for (int c = 0; c < NRP / 4; ++c)
                            *reinterpret_cast<float4 *>(dst + 4 * c) =
                                make_float4(hv[4 * c], hv[4 * c + 1], hv[4 * c + 2], hv[4 * c + 3]);
                    } else {
#pragma unroll
                        for (int hh = 0; hh < NRP; ++hh) dst[hh] = hv[hh];
                    }
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) tot[v] = 0.0f;
        if (tile_n >= tile_end) break;
        tile = tile_n;
    }
}

static bool score_mfma_ok(const xkv_shape &s, const void *A_k)
{
    const int n_rep = s.H_q / s.H_kv;
    const bool rep_ok = (n_rep >= 1 && n_rep <= 8) || n_rep == 16;
    return s.dtype == XKV_BF16 && rep_ok && s.r_k % 16 == 0 && s.d_h % 16 == 0 && (((uintptr_t)A_k) & 15u) == 0 &&
           s.r_k <= 2048;
}

static hipError_t launch_score_generic(const xkv_shape &s, const Plan &p, int layer, const void *A_k,
                                       const void *B_k, const void *q, float *P, float *S, float *S_heads,
                                       hipStream_t st)
{
    dim3 pgrid((s.r_k * s.H_kv + 3) / 4, s.batch), grid((s.L + 255) / 256, s.batch), block(256);
    if (S_heads) {
        const int nrp = head_pitch(s.H_q / s.H_kv);
        if (s.dtype == XKV_F32) {
            hipLaunchKernelGGL(project_q_kernel<float>, pgrid, block, 0, st, (const float *)B_k, (const float *)q, P,
                               s.G, layer, s.r_k, s.H_kv, s.H_q, s.d_h);
            profile_begin(0, st);
            hipLaunchKernelGGL(score_heads_generic_kernel<float>, grid, block, 0, st, (const float *)A_k, P, S, S_heads,
                               s.L, s.r_k, s.H_kv, s.H_q, nrp, p.scale);
            profile_end(0, st);
        } else {
            hipLaunchKernelGGL(project_q_kernel<bf16_t>, pgrid, block, 0, st, (const bf16_t *)B_k, (const bf16_t *)q,
                               P, s.G, layer, s.r_k, s.H_kv, s.H_q, s.d_h);
            profile_begin(0, st);
            hipLaunchKernelGGL(score_heads_generic_kernel<bf16_t>, grid, block, 0, st, (const bf16_t *)A_k, P, S,
                               S_heads, s.L, s.r_k, s.H_kv, s.H_q, nrp, p.scale);
            profile_end(0, st);
        }
        return hipGetLastError();
    }
    if (s.dtype == XKV_F32) {
        hipLaunchKernelGGL(project_q_kernel<float>, pgrid, block, 0, st, (const float *)B_k, (const float *)q, P, s.G,
                           layer, s.r_k, s.H_kv, s.H_q, s.d_h);
        profile_begin(0, st);
        hipLaunchKernelGGL((s.H_q <= 4 * s.H_kv ? score_generic_kernel<float, 4> : score_generic_kernel<float, 8>), grid, block, 0, st, (const float *)A_k, P, S, s.L, s.r_k,
                           s.H_kv, s.H_q, p.scale);
        profile_end(0, st);
    } else {
        hipLaunchKernelGGL(project_q_kernel<bf16_t>, pgrid, block, 0, st, (const bf16_t *)B_k, (const bf16_t *)q, P,
                           s.G, layer, s.r_k, s.H_kv, s.H_q, s.d_h);
        profile_begin(0, st);
        hipLaunchKernelGGL((s.H_q <= 4 * s.H_kv ? score_generic_kernel<bf16_t, 4> : score_generic_kernel<bf16_t, 8>), grid, block, 0, st, (const bf16_t *)A_k, P, S, s.L, s.r_k,
                           s.H_kv, s.H_q, p.scale);
        profile_end(0, st);
    }
    return hipGetLastError();
}

// Tiles per workgroup of the other kernels: about two workgroups of four wavefronts per compute unit in a single round, each streaming
// one contiguous range of a sequence (staging P costs a fixed 2 KiB per rank-16 fragment, so fewer, longer workgroups win).
static int score_tiles_per_wg(int pairs, int n_tiles)
{
    const int wgs_per_pair = pairs >= 512 ? 1 : 512 / pairs;
    const int tiles = (n_tiles + wgs_per_pair - 1) / wgs_per_pair;
    return tiles < 4 ? 4 : (tiles + 3) / 4 * 4;
}

// Whether a shape goes to the long-stream kernel, with how many 32-token tiles per workgroup, and whether its
// LDS also has room for the top-digit histograms.  One 8-wavefront workgroup per compute unit in a single
// round, a whole round of its wavefronts' tiles at a time (spread over all compute units instead, 3073 tiles of ranks 512 take 9 %
// longer, 16385 of ranks 128 7 %: a workgroup is as long as its longest wavefront).
// It pays in any case where every wavefront gets eight tiles of its own.  Below that it pays where the others' workgroups leave the
// compute units with one or two each (us with the projection, rows in the caches / from memory, the others against this kernel:
// 8 KV heads of 4, ranks 512: 1100 tiles 16.9 / 14.7 and 20.2 / 15.5, 2304 25.3 / 21.0 and 30.2 / 22.1, 4097 33.4 / 30.0 and 41.7 / 30.7;
// ranks 192: 1100 12.0 / 11.7 and 14.4 / 12.5; ranks 320: 10000 42.8 / 46.4 and 55.7 / 47.5), and not where they get one each and a few over (1025 tiles, ranks 256 13.2 / 14.8), with
// ranks that fill less than half of their last group of 128 (144: 1537 tiles 10.1 / 11.6 and 12.7 / 13.4) or have but one, with
// sixteen query heads (ranks 256, 641 tiles of two pairs 15.8 / 17.7), or for many (sequence, heads) pairs of few tiles (350 of three,
// ranks 256 50.7 / 56.7; 64 of 20 20.3 / 21.6, but ranks 512 32.4 / 31.0).
bool score_stream_plan(const xkv_shape &s, int *tiles_per_wg, bool *hist_fits, int *waves)
{
    *tiles_per_wg = 0;
    *hist_fits = false;
    *waves = 0;
    if (s.H_kv <= 0 || s.H_q % s.H_kv != 0) return false;
    const int n_rep = s.H_q / s.H_kv;
    const bool rep_ok = (n_rep >= 1 && n_rep <= 8) || n_rep == 16;
    if (s.dtype != XKV_BF16 || !rep_ok || s.r_k % 16 != 0 || s.d_h % 16 != 0 || s.r_k > 2048) return false;
    const int F8 = (s.r_k / 16 + 7) / 8 * 8;
    const int n_tiles = (s.L + 31) / 32;
    const int pairs = s.batch * mfma_blocks(s.H_kv, n_rep);
    if ((long long)pairs * n_tiles < 256 * kScoreWaves * 8) {
        const int per = score_tiles_per_wg(pairs, n_tiles), others = pairs * ((n_tiles + per - 1) / per);
        if (pairs > (s.r_k >= 512 ? 256 : 32) || n_rep > 8 || s.r_k < 192 || others <= 264) return false;
    }
    const size_t lds_max = 160 * 1024 - 512, lds_p = (size_t)2 * F8 * 64 * 16;
    const size_t lds_hist = (size_t)2 * mfma_gph(n_rep) * kTopkBins * 4;
    int wv = kScoreWaves;
    if (lds_p + (size_t)wv * 512 * 16 > lds_max) wv = 4;
    if (lds_p + (size_t)wv * 512 * 16 > lds_max) return false;
    const int wgs = pairs >= 256 ? 1 : 256 / pairs;
    const int tpw = (n_tiles + wgs - 1) / wgs;
    *tiles_per_wg = (tpw + wv - 1) / wv * wv;
    *hist_fits = lds_p + (size_t)wv * 512 * 16 + lds_hist <= lds_max;
    *waves = wv;
    return true;
}

// The long-stream kernel, with or without the per-head output (S_heads only read when HEADS).
template <int N_REP, int WAVES, bool HEADS>
static hipError_t launch_score_stream_t(const xkv_shape &s, const Plan &p, const bf16_t *A_k, const bf16_t *Pfrag,
                                        float *S, int F8, dim3 sgrid, size_t lds_stream, uint32_t *row_hist,
                                        uint32_t *chunk_hist, float *S_heads, hipStream_t st)
{
    static DynamicLdsOnce attr;
    if (hipError_t e0 = attr.ensure((const void *)score_stream_kernel<N_REP, WAVES, HEADS>, 160 * 1024 - 512); e0 != hipSuccess)
        return e0;
    profile_begin(0, st);
    hipLaunchKernelGGL((score_stream_kernel<N_REP, WAVES, HEADS>), sgrid, dim3(WAVES * 64), lds_stream, st, A_k, Pfrag, S,
                       s.L, s.r_k, s.H_kv, F8, p.score_tpw, p.scale, row_hist, chunk_hist, S_heads);
    profile_end(0, st);
    return hipGetLastError();
}

template <int N_REP>
static hipError_t launch_score_mfma_t(const xkv_shape &s, const Plan &p, const bf16_t *A_k, const bf16_t *Pfrag,
                                      float *S, int F8, uint32_t *row_hist, uint32_t *chunk_hist, bool *hist_done,
                                      float *S_heads, hipStream_t st)
{
    const int nblk = mfma_blocks(s.H_kv, N_REP);
    const int n_tiles = (s.L + 31) / 32;
    const size_t lds = (size_t)2 * F8 * 64 * 16;
    if (p.score_stream) {
        const bool with_hist = p.score_hist && row_hist && chunk_hist;
        const size_t lds_stream = lds + (size_t)p.score_waves * 512 * 16 +
                                  (with_hist ? (size_t)2 * mfma_gph(N_REP) * kTopkBins * 4 : 0);
        dim3 sgrid((n_tiles + p.score_tpw - 1) / p.score_tpw, nblk, s.batch);
        uint32_t *rh = with_hist ? row_hist : nullptr, *ch = with_hist ? chunk_hist : nullptr;
        hipError_t e;
        if (p.score_waves == kScoreWaves)
            e = S_heads ? launch_score_stream_t<N_REP, kScoreWaves, true>(s, p, A_k, Pfrag, S, F8, sgrid, lds_stream, rh,
                                                                          ch, S_heads, st)
                        : launch_score_stream_t<N_REP, kScoreWaves, false>(s, p, A_k, Pfrag, S, F8, sgrid, lds_stream,
                                                                           rh, ch, nullptr, st);
        else
            e = S_heads ? launch_score_stream_t<N_REP, 4, true>(s, p, A_k, Pfrag, S, F8, sgrid, lds_stream, rh, ch,
                                                                S_heads, st)
                        : launch_score_stream_t<N_REP, 4, false>(s, p, A_k, Pfrag, S, F8, sgrid, lds_stream, rh, ch,
                                                                 nullptr, st);
        if (e != hipSuccess) return e;
        if (hist_done) *hist_done = with_hist;
        return hipSuccess;
    }
    const int tiles_per_wg = score_tiles_per_wg(s.batch * nblk, n_tiles);
    static DynamicLdsOnce attr_pooled, attr_heads, attr_ring, attr_ring_heads;
    // a tile per wavefront, of several steps; where a second workgroup fits the compute units and some get one, its kernel has the
    // loads in flight already (1025 tiles, ranks 512 13.0 us against 14.3, 640 15.3 / 18.3; 768 22.6 / 20.2: one per compute unit)
    const dim3 rgrid((n_tiles + 3) / 4, nblk, s.batch);
    if (F8 > 16 && tiles_per_wg == 4 && (2 * lds > 160 * 1024 || (long long)rgrid.x * nblk * s.batch <= 256)) {
        auto launch = [&](auto kernel, DynamicLdsOnce &attr) {
            if (hipError_t e0 = attr.ensure((const void *)kernel, 160 * 1024 - 512); e0 != hipSuccess) return e0;
            profile_begin(0, st);
            hipLaunchKernelGGL(kernel, rgrid, dim3(256), lds, st, A_k, Pfrag, S, s.L, s.r_k, s.H_kv, F8, tiles_per_wg, p.scale, S_heads);
            profile_end(0, st);
            return hipGetLastError();
        };
        return S_heads ? launch(score_ring_kernel<N_REP, true>, attr_ring_heads) : launch(score_ring_kernel<N_REP, false>, attr_ring);
    }
    if (hipError_t e0 = attr_pooled.ensure((const void *)score_mfma_kernel<N_REP, false>, 160 * 1024 - 512); e0 != hipSuccess)
        return e0;
    if (hipError_t e0 = attr_heads.ensure((const void *)score_mfma_kernel<N_REP, true>, 160 * 1024 - 512); e0 != hipSuccess)
        return e0;
    dim3 grid((n_tiles + tiles_per_wg - 1) / tiles_per_wg, nblk, s.batch), block(256);
    profile_begin(0, st);
    if (S_heads)
        hipLaunchKernelGGL((score_mfma_kernel<N_REP, true>), grid, block, lds, st, A_k, Pfrag, S, s.L, s.r_k, s.H_kv, F8,
                           tiles_per_wg, p.scale, S_heads);
    else
        hipLaunchKernelGGL((score_mfma_kernel<N_REP, false>), grid, block, lds, st, A_k, Pfrag, S, s.L, s.r_k, s.H_kv, F8,
                           tiles_per_wg, p.scale, (float *)nullptr);
    profile_end(0, st);
    return hipGetLastError();
}

bool score_stage_uses_mfma(const xkv_shape &s, const void *A_k, const void *B_k, const void *q, const void *P_ws,
                           const float *S_heads)
{
    return score_mfma_ok(s, A_k) && ((((uintptr_t)B_k | (uintptr_t)q | (uintptr_t)P_ws)) & 15u) == 0 &&
           (!S_heads || (((uintptr_t)S_heads) & 15u) == 0);
}

hipError_t launch_score_stage(const xkv_shape &s, const Plan &p, int layer, const void *A_k, const void *B_k,
                              const void *q, void *P_ws, float *S, uint32_t *row_hist, uint32_t *chunk_hist,
                              bool *hist_done, const PackArgs *fuse_pack, bool *packed_done, hipStream_t st,
                              float *S_heads, const DenseArgs *tail)
{
    if (hist_done) *hist_done = false;
    if (packed_done) *packed_done = false;
    // per-head scores come from either matrix-core kernel, or from the general one
    const bool mfma = score_stage_uses_mfma(s, A_k, B_k, q, P_ws, S_heads);
    if (!mfma && !B_k) return hipErrorInvalidValue;  // only the matrix-core projection generates an identity B_l
    if (!mfma && tail) return hipErrorInvalidValue;
    if (!mfma) return launch_score_generic(s, p, layer, A_k, B_k, q, (float *)P_ws, S, S_heads, st);
    const int n_rep = s.H_q / s.H_kv;
    const int F8 = (s.r_k / 16 + 7) / 8 * 8;
    const int gph = mfma_gph(n_rep), nblk = mfma_blocks(s.H_kv, n_rep);
    bf16_t *Pfrag = (bf16_t *)P_ws;
    ProjArgs pj{};
    pj.B_k = (const bf16_t *)B_k;
    pj.q = (const bf16_t *)q;
    pj.Pfrag = Pfrag;
    pj.G = s.G;
    pj.layer = layer;
    pj.r_k = s.r_k;
    pj.H_kv = s.H_kv;
    pj.H_q = s.H_q;
    pj.d_h = s.d_h;
    pj.F8 = F8;
    pj.blocks_x = ((F8 / 2) * 2 * gph * nblk + 3) / 4;
    // the row histograms of the top-k stage are cleared in the same launch when the score kernel will add to them
    const bool zero_hist = p.score_stream && p.score_hist && row_hist && chunk_hist;
    const int zero_words = zero_hist ? p.rows * kTopkLevels * kTopkBins : 0;  // a multiple of 1024
    const hipError_t e = launch_prepass(s, pj, fuse_pack, tail, row_hist, zero_words, st);
    if (e != hipSuccess) return e;
    if (packed_done) *packed_done = fuse_pack != nullptr;
    const bf16_t *A = (const bf16_t *)A_k;
    switch (n_rep) {
    case 1: return launch_score_mfma_t<1>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 2: return launch_score_mfma_t<2>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 3: return launch_score_mfma_t<3>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 4: return launch_score_mfma_t<4>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 5: return launch_score_mfma_t<5>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 6: return launch_score_mfma_t<6>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 7: return launch_score_mfma_t<7>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    case 8: return launch_score_mfma_t<8>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    default: return launch_score_mfma_t<16>(s, p, A, Pfrag, S, F8, row_hist, chunk_hist, hist_done, S_heads, st);
    }
}

// The line-wise kernel (eight wavefronts, one workgroup per compute unit) whenever its LDS fits -- ranks up to 512 --
// else the kernel with one lane per row (four wavefronts, long passes).
template <int N_REP>
static hipError_t launch_score_q4_t(const xkv_shape &s, const Plan &p, const unsigned char *Aq, const bf16_t *Pfrag, float *S,
                                    float *S_heads, int F8, hipStream_t st)
{
    const int nblk = mfma_blocks(s.H_kv, N_REP);
    const int n_tiles = (s.L + 31) / 32;
    const size_t lds = (size_t)2 * F8 * 64 * 16 + (size_t)(F8 / 2) * 32 * 4;
    const size_t lds_tile = lds + (size_t)((F8 / 2 + 15) / 16) * 3 * 64 * 16 +
                            (size_t)kQ4TileWaves * (32 * q4_tile_pitch(s.r_k) + kQ4TileSlack);
    const bool tiled = lds_tile <= 160 * 1024 - 512 && 32 * (s.r_k * 5 / 8) <= kQ4MaxLoads * 1024;
    const int waves = tiled ? kQ4TileWaves : 4;
    // one (line-wise) or two workgroups per compute unit, each over one contiguous range of a sequence
    const int pairs = s.batch * nblk;
    const int want = tiled ? 256 : 512;
    const int wgs_per_pair = pairs >= want ? 1 : want / pairs;
    int tiles_per_wg = (n_tiles + wgs_per_pair - 1) / wgs_per_pair;
    tiles_per_wg = tiles_per_wg < waves ? waves : (tiles_per_wg + waves - 1) / waves * waves;
    dim3 grid((n_tiles + tiles_per_wg - 1) / tiles_per_wg, nblk, s.batch);
    hipError_t e = hipSuccess;
    if (tiled) {
        static DynamicLdsOnce attr8;
        e = attr8.ensure((const void *)score_q4_tile_kernel<N_REP>, 160 * 1024 - 512);
        if (e != hipSuccess) return e;
        profile_begin(0, st);
        hipLaunchKernelGGL((score_q4_tile_kernel<N_REP>), grid, dim3(kQ4TileWaves * 64), lds_tile, st, Aq, Pfrag, S, S_heads,
                           s.L, s.r_k, s.H_kv, F8, tiles_per_wg, p.scale);
        profile_end(0, st);
    } else {
        static DynamicLdsOnce attr4;
        e = attr4.ensure((const void *)score_q4_kernel<N_REP, 4, 16>, 160 * 1024 - 512);
        if (e != hipSuccess) return e;
        profile_begin(0, st);
        hipLaunchKernelGGL((score_q4_kernel<N_REP, 4, 16>), grid, dim3(256), lds, st, Aq, Pfrag, S, S_heads, s.L, s.r_k,
                           s.H_kv, F8, tiles_per_wg, p.scale);
        profile_end(0, st);
    }
    return hipGetLastError();
}

bool score_q4_shape_ok(const xkv_shape &s)
{
    if (s.H_kv <= 0 || s.H_q % s.H_kv != 0) return false;
    const int n_rep = s.H_q / s.H_kv;
    const bool rep_ok = (n_rep >= 1 && n_rep <= 8) || n_rep == 16;
    return s.dtype == XKV_BF16 && rep_ok && s.r_k > 0 && s.r_k % 128 == 0 && s.r_k <= 2048 && s.d_h % 16 == 0;
}

// Projection (as for the bf16 stream) and the score kernel over quantised rows; S and S_heads are both written.
hipError_t launch_score_q4_stage(const xkv_shape &s, const Plan &p, int layer, const void *Aq_k, const void *B_k,
                                 const void *q, void *P_ws, float *S, float *S_heads, hipStream_t st, const PackArgs *fuse_pack,
                                 const DenseArgs *tail)
{
    const int n_rep = s.H_q / s.H_kv;
    const int F8 = (s.r_k / 16 + 7) / 8 * 8;
    const int gph = mfma_gph(n_rep), nblk = mfma_blocks(s.H_kv, n_rep);
    bf16_t *Pfrag = (bf16_t *)P_ws;
    ProjArgs pj{};
    pj.B_k = (const bf16_t *)B_k;
    pj.q = (const bf16_t *)q;
    pj.Pfrag = Pfrag;
    pj.G = s.G;
    pj.layer = layer;
    pj.r_k = s.r_k;
    pj.H_kv = s.H_kv;
    pj.H_q = s.H_q;
    pj.d_h = s.d_h;
    pj.F8 = F8;
    pj.blocks_x = ((F8 / 2) * 2 * gph * nblk + 3) / 4;
    const hipError_t e = launch_prepass(s, pj, fuse_pack, tail, nullptr, 0, st);
    if (e != hipSuccess) return e;
    const unsigned char *A = (const unsigned char *)Aq_k;
    switch (n_rep) {
    case 1: return launch_score_q4_t<1>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 2: return launch_score_q4_t<2>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 3: return launch_score_q4_t<3>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 4: return launch_score_q4_t<4>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 5: return launch_score_q4_t<5>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 6: return launch_score_q4_t<6>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 7: return launch_score_q4_t<7>(s, p, A, Pfrag, S, S_heads, F8, st);
    case 8: return launch_score_q4_t<8>(s, p, A, Pfrag, S, S_heads, F8, st);
    default: return launch_score_q4_t<16>(s, p, A, Pfrag, S, S_heads, F8, st);
    }
}

}  // namespace xkv
