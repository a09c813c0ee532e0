// The matrix-core kernel of attention over an uncompressed range of tokens, as a block function: a launch of its own for a
// whole cache, blocks of the launch that projects the queries for the tail of a decode step.
#ifndef XKV_DENSE_BLOCK_H
#define XKV_DENSE_BLOCK_H

#include "xkv_common.h"

namespace xkv {
namespace dense {

// ==========================================================================================
// bf16 matrix-core path (d_h = 128).  A wavefront walks 32-token blocks of its workgroup's range:
//   Z^T [tokens x head slots] = K block (loaded line-wise, operand fragments through an LDS tile)  x  Q^T (registers)
//   O [head slots x dims]    += W = exp(Z^T - max) (the result registers of Z^T, packed)   x  V block
// The contraction of the second product runs over tokens, so each lane needs eight token rows of one
// column of V: the V block goes through a wavefront-private LDS tile, which the transposing LDS read (4 rows x 16 columns a time) turns.
// The rows of the next block, K and V together, are requested once this one's have left the registers for LDS.
// The four wavefronts merge their partials in LDS before writing.
// What bounds it: the stream where it is long, 4 x 8 x 65536 tokens 164 us (6.5 TB/s; 167 with V read back two bytes at a time and the rows
// requested at the start of their block), latencies where it is short: 8 x 4096 with the merge 10.0 us (11.3), 8 x 32768 29.3 (30.3).
// Where a compute unit has two workgroups of two blocks each, the next rows of K requested ahead of those of V, before the logits,
// were slower than no early request: 18 x 8 x 684 tokens, 16 query heads each, 17.5 us, at the start of their block 17.0, as it is 16.9; 32 x 8
// x 400, four heads, 14.0, 13.6 and 13.2.
// ==========================================================================================
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) float f32x8_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

typedef __attribute__((ext_vector_type(4))) short s16x4_t;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;

constexpr int kVPitch = 288;  // bytes per token row of the LDS tile of V (256 + 32: the 32 B of eight rows lie on different banks)

__device__ __forceinline__ bf16x8_t pack8_bf16(const f32x16_t &c, int j)
{
    f32x8_t x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = c[8 * j + e];
    return __builtin_convertvector(x, bf16x8_t);
}

// LDS: per wavefront a V tile (32 x 288 B) and a K tile (32 x 256 B), 68 KiB; the V part is reused for the merge
constexpr int kLdsBytes = 4 * 32 * kVPitch + 4 * 32 * 256;

// A workgroup of 256 threads: tokens [split chunk, (split + 1) chunk) of one (sequence b, KV head g), one partial per query head.
__device__ __forceinline__ void mfma_block(const DenseArgs &a, int split, int g, int b, unsigned char *smem)
{
    const bf16_t *__restrict__ K = a.K, *__restrict__ V = a.V, *__restrict__ q = a.q;
    float *__restrict__ part_o = a.part_o, *__restrict__ part_ml = a.part_ml;
    const int L = a.L, H_kv = a.H_kv, H_q = a.H_q, splits = a.splits, chunk = a.chunk;
    const float scale = a.scale;
    const int lane = lane_id(), w = wave_id();
    const int n = lane & 31, hf = lane >> 5;
    const int n_rep = H_q / H_kv;

    // Q^T fragments: lane (head slot n, hf), fragment f, position e: q[n][16 f + 8 hf + e]
    bf16x8_t Qf[8];
    {
        const u32x4_t *qh = reinterpret_cast<const u32x4_t *>(q + ((size_t)b * H_q + (size_t)g * n_rep +
                                                                    (n < n_rep ? n : 0)) * 128);
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            u32x4_t raw = qh[2 * f + hf];
            if (n >= n_rep) raw = u32x4_t{0u, 0u, 0u, 0u};
            Qf[f] = __builtin_bit_cast(bf16x8_t, raw);
        }
    }
    const bf16_t *Kg = K + ((size_t)b * H_kv + g) * (size_t)L * 128;
    const bf16_t *Vg = V + ((size_t)b * H_kv + g) * (size_t)L * 128;
    const int t_begin = split * chunk;
    const int t_end = t_begin + chunk < L ? t_begin + chunk : L;
    unsigned char *vt = smem + w * 32 * kVPitch;  // this wavefront's V tile
    // ... and its K tile, in 16 B units: piece c of token row t sits at 16 t + (c + t) % 16 (conflict-free for the
    // row-wise writes and for the fragment reads: lane (n, hf) reads piece 2 f + hf of row n)
    u32x4_t *kt = reinterpret_cast<u32x4_t *>(smem + 4 * 32 * kVPitch) + w * 512;
    const int kw_row = lane >> 4, kw_piece = lane & 15;
    const int kr_base = 16 * n, kr_rot = hf + n;

    float m_run = -INFINITY, l_run = 0.0f;
    // Only head slots 0..15 can hold a query head (n_rep <= 16): of the 16 result registers of an O tile the
    // first 8 (slots 8(v/4) + 4hf + v%4, v < 8) are kept between blocks, the rest is dropped.
    float O[4][8];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int v = 0; v < 8; ++v) O[db][v] = 0.0f;

    // K and V rows, whole lines per instruction: 16 lanes cover one 256 B row, the wavefront 4 rows per load
    // (with one lane per row four instructions would share every 128 B line, which streams measurably slower)
    u32x4_t kr[8], vr[8];
    auto request = [&](u32x4_t (&to)[8], const bf16_t *from, int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = t0 + i * 4 + (lane >> 4), tv = row < t_end ? row : t_end - 1;
            to[i] = __builtin_nontemporal_load(&reinterpret_cast<const u32x4_t *>(from + (size_t)tv * 128)[lane & 15]);
        }
    };
    // this lane's place in the tile of V for the transposing read: row 4 hf + l16 / 4, columns 16 (lane / 16 % 2) + 4 (l16 % 4) ..
    const unsigned char *vrd = vt + (4 * hf + ((lane & 15) >> 2)) * kVPitch + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    if (t_begin + w * 32 < t_end) {
        request(kr, Kg, t_begin + w * 32);
        request(vr, Vg, t_begin + w * 32);
    }
    for (int t0 = t_begin + w * 32; t0 < t_end; t0 += 128) {
        // K through its LDS tile: written row-wise, read back as the operand fragment of each 16 head dims
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = i * 4 + kw_row;
            kt[16 * row + ((kw_piece + row) & 15)] = kr[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        f32x16_t Z;
#pragma unroll
        for (int v = 0; v < 16; ++v) Z[v] = 0.0f;
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const u32x4_t kf = kt[kr_base + ((kr_rot + 2 * f) & 15)];
            Z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kf), Qf[f], Z, 0, 0, 0);
        }
        // lane (head slot n, hf): register v is token 8(v/4) + 4hf + v%4 of the block
        float m_loc = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int tt = t0 + 8 * (v / 4) + 4 * hf + (v % 4);
            Z[v] = tt < t_end ? scale * Z[v] : -INFINITY;
            m_loc = fmaxf(m_loc, Z[v]);
        }
        m_loc = fmaxf(m_loc, __shfl_xor(m_loc, 32, kWave));
        const float m_new = fmaxf(m_run, m_loc);
        const float alpha = (m_new == -INFINITY) ? 1.0f : __expf(m_run - m_new);
        float l_add = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float wv = (Z[v] == -INFINITY) ? 0.0f : __expf(Z[v] - m_new);
            Z[v] = wv;
            l_add += wv;
        }
        l_run = l_run * alpha + l_add;
        m_run = m_new;
        const bf16x8_t W0 = pack8_bf16(Z, 0), W1 = pack8_bf16(Z, 1);

        // stage V in LDS and read it back as [8 tokens of one column] fragments
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = i * 4 + (lane >> 4);
            *reinterpret_cast<u32x4_t *>(vt + row * kVPitch + (lane & 15) * 16) = vr[i];
        }
        if (t0 + 128 < t_end) {
            request(kr, Kg, t0 + 128);
            request(vr, Vg, t0 + 128);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const float a = __shfl(alpha, 8 * (v / 4) + 4 * hf + (v % 4), kWave);
#pragma unroll
            for (int db = 0; db < 4; ++db) O[db][v] *= a;
        }
#pragma unroll
        for (int db = 0; db < 4; ++db) {
            f32x16_t ot;
#pragma unroll
            for (int v = 0; v < 16; ++v) ot[v] = 0.0f;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                // position e of lane (column n, hf): token 16 j + 8 (e / 4) + 4 hf + e % 4
                const unsigned char *from = vrd + 16 * j * kVPitch + 64 * db;
                const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)from);
                const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t *)(from + 8 * kVPitch));
                ot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(j == 0 ? W0 : W1,
                                                             __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7)),
                                                             ot, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 8; ++v) O[db][v] += ot[v];
        }
        __builtin_amdgcn_wave_barrier();
    }

    // merge the four wavefronts: LDS holds per (wavefront, head) the max, the sum and 128 outputs
    __syncthreads();
    float *mg = reinterpret_cast<float *>(smem);  // [4][16][132]
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    if (lane < n_rep) {
        mg[(w * 16 + lane) * 132 + 128] = m_run;
        mg[(w * 16 + lane) * 132 + 129] = l_tot;
    }
#pragma unroll
    for (int v = 0; v < 8; ++v) {
        const int hh = 8 * (v / 4) + 4 * hf + (v % 4);
        if (hh < n_rep) {
#pragma unroll
            for (int db = 0; db < 4; ++db) mg[(w * 16 + hh) * 132 + db * 32 + n] = O[db][v];
        }
    }
    __syncthreads();
    for (int item = threadIdx.x; item < n_rep * 128; item += 256) {
        const int hh = item >> 7, dim = item & 127;
        float M = -INFINITY;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) M = fmaxf(M, mg[(ww * 16 + hh) * 132 + 128]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) {
            const float mw = mg[(ww * 16 + hh) * 132 + 128];
            const float wgt = (mw == -INFINITY) ? 0.0f : __expf(mw - M);
            num = fmaf(wgt, mg[(ww * 16 + hh) * 132 + dim], num);
            den = fmaf(wgt, mg[(ww * 16 + hh) * 132 + 129], den);
        }
        const size_t slot = ((size_t)b * H_q + g * n_rep + hh) * splits + split;
        part_o[slot * 128 + dim] = num;
        if (dim == 0) {
            part_ml[slot * 2 + 0] = M;
            part_ml[slot * 2 + 1] = den;
        }
    }
}

}  // namespace dense
}  // namespace xkv
#endif
