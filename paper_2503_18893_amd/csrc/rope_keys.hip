// Logits of the selected rows where the keys are rotated after the reconstruction (bf16 products, d_h = 128):
//   z_h[m] = scale R(t_m) (A^K[t_m,:] B^K_{l,g}) . q_h,   t_m the selected tokens of KV head g.
//
// The factor B^K of a head stays in registers.  A workgroup is four wavefronts; wavefront w holds channels 16 w .. + 15 and 64 + 16 w ..
// of all ranks as operands (128 registers at 512 ranks), so that both channels of a rotated pair sit in the same lane of a
// result.  The workgroup walks its rows 32 at a time:
//   (1) K^T [dims x tokens] = B^K^T (registers) x rows of A^K (operands read from LDS);
//   (2) the rotation, in the result's registers;
//   (3) Z [head slots x tokens] = Q x K^: eight result registers, packed to bf16, are the operand.  The wavefronts' sums over their 32
//       channels are added through LDS.
// Two images of 32 rows lie in LDS as bf16, piece p (8 ranks) of row t in place p ^ (t % 16) (quantised rows, whose lanes write a group of
// 32 ranks a word of eight at a time: word u of group q as piece u r / 32 + q): while one is multiplied, the next is filled -- bf16 rows go global -> LDS directly, quantised rows come in registers two tiles ahead and are de-quantised --
// and (2) and (3) run for the tile before.  Matrix instructions issue in order with the rest of a wavefront, so each is followed by
// vector work that fits under it.
// What bounds it: LDS (every wavefront reads the whole image: 128 KiB per 32 rows of ranks 512, and 32 to fill it), vector
// instructions (360 per wavefront and tile, of which 110 de-quantise and 70 rotate) and matrix instructions (34) in
// about equal parts, with two wavefronts per SIMD to overlap them: 8 x 8 x 4128 rows of ranks 512 in 4 bits 51 us under the profiler
// (62 in the KEYS form of gather_attend_mfma_kernel, which streams B^K through LDS for every 256 rows and rounds up to them);
// without its products 40, without de-quantising 36, without the rotation 46.  Two wavefronts of 64 channels with 512 registers
// each, half the LDS traffic but nothing to hide a wait behind: 58 to 63 us.  Both halves and merge: 112 -> 99 us (16 x 8: 207 -> 176;
// 3 bits 194 -> 171; bf16 251 -> 228; 16 x 8 x 2080 in 4 bits 139 -> 113).
#include "xkv_common.h"

#include <cmath>

namespace xkv {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(8))) float f32x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;

constexpr int kRows = 32;            // selected rows per tile
constexpr int kMaxRunTiles = 32;     // tiles per workgroup (their ids lie in LDS)
constexpr int kZBytes = 2 * 4 * kRows * 32;  // partial logits [tile parity][wavefront][row][8 slots]
template <int NF> constexpr int rope_keys_lds() { return 2 * kRows * NF * 32 + kZBytes + 512 + kMaxRunTiles * kRows * 4; }

// Two ranks of a group of quantised rows, their codes in the halves of a word as whole numbers c 2^s below 1024: the 16-bit numbers
// c 2^(s - 24) (subnormal, exact), so that step' = step 2^(24 - s) and a multiply-add that takes 16-bit sources give step c + lo with one
// rounding.
__device__ __forceinline__ uint32_t two_values(uint32_t codes, float step, float lo)
{
    const f16x2_t c = __builtin_bit_cast(f16x2_t, codes);
    const f32x2_t x = f32x2_t{__builtin_fmaf(step, (float)c[0], lo), __builtin_fmaf(step, (float)c[1], lo)};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
}

struct RopeFactors {
    float f0[64], f1[64];  // theta^(-j/64) / 2 pi, and frac(256 * that)
};

template <int NF, int QB>  // steps of 16 ranks; rows of A^K in bf16 (0) or of 4- or 3-bit codes
__global__ __launch_bounds__(256, 2) void rope_keys_kernel(const void *__restrict__ A_k, const u32x4_t *__restrict__ pack, size_t pack_seq_stride,
                                                           size_t pack_head_stride, const u32x4_t *__restrict__ pack_q,
                                                           const int32_t *__restrict__ idx, const int32_t *__restrict__ counts, int L,
                                                           int r_k, int H_kv, int k, int splits, int run_tiles, float scale,
                                                           const RopeFactors rope, float *__restrict__ logits, int hp)
{
    constexpr int NP = 2 * NF, kImage = kRows * NF * 32;  // 16-byte pieces of a row, bytes of an image
    constexpr int GR = NF / 2, NQ = QB ? (NF + 15) / 16 : 1;  // groups of 32 ranks of a row; pieces of codes per lane and tile
    constexpr int NC = NF / 4;                            // bf16: copies of 1 KiB per wavefront and tile
    constexpr int RING = NF > 24 ? (QB ? 2 : 3) : 4, H = NF / 2;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    f32x4_t *Zb = reinterpret_cast<f32x4_t *>(smem_raw + 2 * kImage);
    float *angle = reinterpret_cast<float *>(smem_raw + 2 * kImage + kZBytes);  // [64][2]
    int *toks = reinterpret_cast<int *>(smem_raw + 2 * kImage + kZBytes + 512);

    const int g = blockIdx.x % H_kv, split = (blockIdx.x / H_kv) % splits, b = blockIdx.x / (H_kv * splits);
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id(), n = lane & 31, hf = lane >> 5;
    int k_eff = k;  // with `counts`, only the first counts[sequence][head] ids of a row are real
    if (counts) {
        const int cn = counts[b * H_kv + g];
        k_eff = cn < k ? (cn > 0 ? cn : 0) : k;
    }
    const int m_begin = split * run_tiles * kRows, m_left = k_eff - m_begin;
    if (m_left <= 0) return;
    const int rows = m_left < run_tiles * kRows ? m_left : run_tiles * kRows, n_tiles = (rows + kRows - 1) / kRows;

    const int32_t *ids = idx + ((size_t)b * H_kv + g) * k + m_begin;
    for (int m = tid; m < n_tiles * kRows; m += 256) {  // rows past the end repeat the last one
        const int t = ids[m < rows ? m : rows - 1];
        toks[m] = t < 0 ? 0 : (t >= L ? L - 1 : t);
    }
    if (tid < 128) angle[tid] = tid & 1 ? rope.f1[tid >> 1] : rope.f0[tid >> 1];
    lds_barrier();

    // (a sequence has fewer than 2^24 rows and less than 4 GiB of them)
    const uint32_t pitch = QB == 0 ? (uint32_t)r_k * 2 : (uint32_t)quant_row_bytes(r_k, QB);
    const unsigned char *Ak = reinterpret_cast<const unsigned char *>(A_k) + (size_t)b * L * pitch;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem_raw;

    // ---- rows of a tile.  bf16: a copy is 64 pieces of the image.  Pieces and groups beyond the row are replaced by the first: they meet
    // zero operands
    auto copy = [&](int tile, int j) __attribute__((always_inline)) {
        const int e = 64 * (w * NC + j) + lane, t = e / NP, pc = (e - t * NP) ^ (t & 15);
        const uint32_t off = __umul24((uint32_t)toks[tile * kRows + t], pitch) + 16 * (pc < (r_k >> 3) ? pc : 0);
        copy16_global_to_lds(Ak + off, __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(tile & 1) * kImage + (uint32_t)(w * NC + j) * 1024));
    };
    struct Codes {
        u32x4_t piece[NQ];
        uint32_t param[NQ];
    };
    auto fetch = [&](Codes &c, int tile, int i, int thread) __attribute__((always_inline)) {
        const int e = 256 * i + thread, t = (e / GR) & (kRows - 1), q0 = e % GR, q = q0 < (r_k >> 5) ? q0 : 0;  // (lanes beyond the last row: any row)
        const unsigned char *row = Ak + __umul24((uint32_t)toks[(tile < n_tiles ? tile : n_tiles - 1) * kRows + t], pitch);
        c.piece[i] = *reinterpret_cast<const u32x4_t *>(row + 16 * q);
        if constexpr (QB == 4) c.param[i] = *reinterpret_cast<const uint32_t *>(row + (r_k >> 1) + 4 * q);
    };
    // word u (8 ranks) of piece i into the image
    auto value_word = [&](const Codes &c, int tile, int i, int u, int half, u32x4_t &x, int thread) __attribute__((always_inline)) {
        const u32x4_t p = c.piece[i];
        const uint32_t par = QB == 4 ? c.param[i] : p[3];
        const float step = __uint_as_float(par << 16) * 16777216.0f, lo = __uint_as_float(par & 0xFFFF0000u);
        if constexpr (QB == 4) {
            const uint32_t wd = half ? p[u] >> 8 : p[u];
            x[2 * half] = two_values(wd & 0x000F000Fu, step, lo);
            x[2 * half + 1] = two_values(wd & 0x00F000F0u, step * 0.0625f, lo);
        } else {  // 96 bits of codes, four units of 24, then (step, lo)
            const uint32_t u24 = u == 0 ? p[0] : u == 1 ? (p[0] >> 24) | (p[1] << 8) : u == 2 ? (p[1] >> 16) | (p[2] << 16) : p[2] >> 8;
            const uint32_t cd = (u24 & 0xFFFu) | ((u24 << 4) & 0x0FFF0000u), wd = half ? cd >> 6 : cd;
            x[2 * half] = two_values(wd & 0x00070007u, step, lo);
            x[2 * half + 1] = two_values(wd & 0x00380038u, step * 0.125f, lo);
        }
        if (half == 1) {
            const int e = 256 * i + thread, t = e / GR, q = e - t * GR;
            if (256 * (i + 1) <= kRows * GR || t < kRows) *reinterpret_cast<u32x4_t *>(smem_raw + (tile & 1) * kImage + t * (NF * 32) + (((GR * u + q) ^ (t & 15)) << 4)) = x;
        }
    };

    // From a step of 2^104 on step' is infinite, and 0 step' no number.  A tile in which a wavefront has one (hardly ever) is read once
    // more and written by it a second time, the codes converted one by one.  (Behind the tile's products: a look at each piece between
    // them cost 1.3 % at ranks 512, both halves at 8 x 8 x 4128 rows in 4 bits 101.8 -> 103.1 us; this costs nothing that shows.)
    auto has_large_step = [&](const Codes &c) __attribute__((always_inline)) {
        uint32_t most = 0;
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const uint32_t step = (QB == 4 ? c.param[i] : c.piece[i][3]) & 0xFFFFu;
            most = most > step ? most : step;
        }
        return __ballot(most >= 0x7380u) != 0;
    };
    auto large_steps = [&](int tile, int thread) __attribute__((always_inline)) {
#pragma unroll 1
        for (int i = 0; i < NQ; ++i) {
            const int e = 256 * i + thread, t = e / GR, q = e - t * GR;
            if (t >= kRows) break;
            const unsigned char *row = Ak + __umul24((uint32_t)toks[(tile < n_tiles ? tile : n_tiles - 1) * kRows + t], pitch);
            const int qr = q < (r_k >> 5) ? q : 0;
            u32x4_t p = *reinterpret_cast<const u32x4_t *>(row + 16 * qr);
            const uint32_t par = QB == 4 ? *reinterpret_cast<const uint32_t *>(row + (r_k >> 1) + 4 * qr) : p[3];
            const float step = __uint_as_float(par << 16), lo = __uint_as_float(par & 0xFFFF0000u);
#pragma unroll 1
            for (int u = 0; u < 4; ++u) {
                const uint32_t wd = QB == 4 ? p[0] : (p[0] & 0xFFFu) | ((p[0] << 4) & 0x0FFF0000u);
                u32x4_t x;
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const uint32_t c0 = (wd >> (QB * h)) & ((1u << QB) - 1), c1 = (wd >> (16 + QB * h)) & ((1u << QB) - 1);
                    const f32x2_t y = f32x2_t{__builtin_fmaf(step, (float)c0, lo), __builtin_fmaf(step, (float)c1, lo)};
                    x[h] = __builtin_bit_cast(uint32_t, __builtin_convertvector(y, bf16x2_t));
                }
                *reinterpret_cast<u32x4_t *>(smem_raw + (tile & 1) * kImage + t * (NF * 32) + (((GR * u + q) ^ (t & 15)) << 4)) = x;
                if constexpr (QB == 4)
                    p = u32x4_t{p[1], p[2], p[3], 0};
                else
                    p = u32x4_t{(p[0] >> 24) | (p[1] << 8), (p[1] >> 24) | (p[2] << 8), p[2] >> 24, 0};
            }
        }
    };

    // ---- start: the rows of the first tiles, then B^K and the queries
    Codes even, odd;  // of tiles 1, 3, 5 .. (consumed in the even bodies) and 2, 4, ..
    if constexpr (QB == 0) {
#pragma unroll
        for (int j = 0; j < NC; ++j) copy(0, j);
    } else {
#pragma unroll
        for (int i = 0; i < NQ; ++i) fetch(odd, 0, i, tid);
#pragma unroll
        for (int i = 0; i < NQ; ++i) fetch(even, 1, i, tid);
    }
    bf16x8_t bk[NF], qf[2];
    const u32x4_t *src = pack + (size_t)b * pack_seq_stride + (size_t)g * pack_head_stride + ((w >> 1) + 2 * (n >> 4)) * 64 + hf * 32 + 16 * (w & 1) + (n & 15);
    const u32x4_t *qsrc = pack_q + ((size_t)b * H_kv + g) * 512 + w * 64 + lane;
#pragma unroll
    for (int f = 0; f < NF; ++f) bk[f] = __builtin_bit_cast(bf16x8_t, src[f * 256]);
#pragma unroll
    for (int j = 0; j < 2; ++j) qf[j] = __builtin_bit_cast(bf16x8_t, qsrc[j * 256]);
    if constexpr (QB != 0) {
#pragma unroll
        for (int i = 0; i < NQ; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                u32x4_t x;
                value_word(odd, 0, i, u, 0, x, tid);
                value_word(odd, 0, i, u, 1, x, tid);
            }
        if (__builtin_expect(has_large_step(odd), 0)) large_steps(0, tid);
#pragma unroll
        for (int i = 0; i < NQ; ++i) fetch(odd, 2, i, tid);
    }

    // ranks 16 f + 8 hf .. of row n: piece 2 f + hf, or word 2 (f % 2) + hf of group f / 2
    auto a_frag = [&](const unsigned char *image, int f, int l) __attribute__((always_inline)) {
        const int t = l & 31, h = l >> 5, x = t & 15;
        int at;
        if constexpr (QB == 0)
            at = ((f >> 3) << 8) + (((2 * f & 15) ^ (h ^ x)) << 4);
        else if constexpr (GR == 16)
            at = ((f & 1) << 9) + (h << 8) + (((f >> 1) ^ x) << 4);
        else
            at = ((GR * (2 * (f & 1) + h) + (f >> 1)) ^ x) << 4;
        return *reinterpret_cast<const bf16x8_t *>(image + t * (NF * 32) + at);
    };
    // (2) for pair v of a tile's result: channels 16 w + 8 (v / 4) + 4 hf + v % 4 and 64 more, turned by the row's position.  The angle in
    // revolutions is formed from position / 256 and position % 256 against two constants per channel (accurate to 2^-16 of a turn
    // up to any context length) and goes through the hardware sine and cosine.
    float t_hi = 0.0f, t_lo = 0.0f;
    f32x4_t fa;
    float sn = 0.0f, cs = 1.0f;
    auto position = [&](int tile) __attribute__((always_inline)) {
        const int t = toks[tile * kRows + n];
        t_hi = (float)(t >> 8), t_lo = (float)(t & 255);
    };
    auto turn_angle = [&](int v) __attribute__((always_inline)) {
        if (v % 2 == 0) fa = *reinterpret_cast<const f32x4_t *>(angle + 2 * (16 * w + 8 * (v / 4) + 4 * hf + v % 4));
        const float rev = __builtin_amdgcn_fractf(t_hi * fa[2 * (v % 2) + 1] + t_lo * fa[2 * (v % 2)]);
        sn = __builtin_amdgcn_sinf(rev), cs = __builtin_amdgcn_cosf(rev);
    };
    auto turn = [&](f32x16_t &x, int v) __attribute__((always_inline)) {
        const float p = x[v], q = x[8 + v];
        x[v] = p * cs - q * sn;
        x[8 + v] = q * cs + p * sn;
    };
    f32x16_t Z;
    auto meets_q = [&](const f32x16_t &x, int j) __attribute__((always_inline)) {  // product j of two of (3)
        f32x8_t y;
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = x[8 * j + e];
        if (j == 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) Z[v] = 0.0f;
        }
        Z = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[j], __builtin_convertvector(y, bf16x8_t), Z, 0, 0, 0);
    };
    // lane (row n, hf): slots 4 hf .. + 3 in registers 0 .. 3 (no more than eight heads)
    const int quads = (hp + 3) / 4;
    auto leave = [&](int tile) __attribute__((always_inline)) {
        if (hf < quads) Zb[(((tile & 1) * 4 + w) * kRows + n) * 2 + hf] = f32x4_t{Z[0], Z[1], Z[2], Z[3]};
    };
    float *out = logits + (((size_t)b * H_kv + g) * k + m_begin) * hp;
    auto finish = [&](int tile) __attribute__((always_inline)) {  // the wavefronts' partial logits of a tile -> memory
        if (tid >= 64) return;
        const int row = tid & 31, qd = tid >> 5, m = tile * kRows + row;
        if (qd >= quads || m >= rows) return;
        const f32x4_t *from = Zb + ((tile & 1) * 4 * kRows + row) * 2 + qd;
        const f32x4_t z = scale * ((from[0] + from[kRows * 2]) + (from[kRows * 4] + from[kRows * 6]));
        float *to = out + (size_t)m * hp + 4 * qd;
        if (hp >= 4)
            *reinterpret_cast<f32x4_t *>(to) = z;
        else
            for (int e = 0; e < hp; ++e) to[e] = z[e];
    };

    // tile i: (1) into `now`, image i + 1 from `codes`; (2) and (3) for tile i - 1, whose result is `last`; the logits of tile i - 2 leave
    auto body = [&](int i, f32x16_t &now, f32x16_t &last, Codes &codes) __attribute__((always_inline)) {
        const unsigned char *image = smem_raw + (i & 1) * kImage;
        int l = lane;
        asm volatile("" : "+v"(l));  // (addresses in LDS are formed where they are used: two dozen of them would not fit the registers)
        bf16x8_t ring[RING];
#pragma unroll
        for (int f = 0; f < RING; ++f) ring[f] = a_frag(image, f, l);
        position(i > 0 ? i - 1 : 0);
        if (i >= 2) finish(i - 2);
        if constexpr (QB == 0) {
            if (i + 1 < n_tiles) {
#pragma unroll
                for (int j = 0; j < NC; ++j) copy(i + 1, j);
            }
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) now[v] = 0.0f;
        __builtin_amdgcn_sched_barrier(0);
        u32x4_t x;
        bool large = false;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            now = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bk[f], ring[f % RING], now, 0, 0, 0);  // rows channels, columns tokens
            if (f + RING < NF) ring[f % RING] = a_frag(image, f + RING, l);
            if (f < H) {
#pragma unroll
                for (int v = f * 8 / H; v < (f + 1) * 8 / H; ++v) {
                    turn_angle(v);
                    turn(last, v);
                }
            } else {
                if constexpr (QB != 0) {
                    if (f == H) large = has_large_step(codes);
#pragma unroll
                    for (int u = (f - H) * 8 * NQ / H; u < (f - H + 1) * 8 * NQ / H; ++u) {  // half u % 2 of word u / 2 % 4 of piece u / 8
                        value_word(codes, i + 1, u / 8, u / 2 % 4, u % 2, x, 64 * w + l);
                        if (u % 8 == 7) fetch(codes, i + 3, u / 8, 64 * w + l);
                    }
                }
                if (f - H < 2) meets_q(last, f - H);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (i > 0) leave(i - 1);
        if constexpr (QB != 0)
            if (__builtin_expect(large, 0)) large_steps(i + 1, 64 * w + l);
    };
    auto meet = [&]() __attribute__((always_inline)) {  // the next image is there, this one is no longer read
        if constexpr (QB == 0) XKV_WAIT_VMCNT(0);
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto end = [&](f32x16_t &last) __attribute__((always_inline)) {
        const int i = n_tiles - 1;
        position(i);
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            turn_angle(v);
            turn(last, v);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) meets_q(last, j);
        lds_barrier();  // (the room of tile i - 2's logits)
        leave(i);
        lds_barrier();
        if (i > 0) finish(i - 1);
        finish(i);
    };
    f32x16_t acc[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[1][v] = 0.0f;
    meet();
    for (int i = 0;;) {
        body(i, acc[0], acc[1], even);
        if (++i == n_tiles) {
            end(acc[0]);
            break;
        }
        meet();
        body(i, acc[1], acc[0], odd);
        if (++i == n_tiles) {
            end(acc[1]);
            break;
        }
        meet();
    }
}

// (B^K in 128 registers at most; eight slots of partial logits in LDS)
bool rope_keys_ok(const xkv_shape &s) { return s.r_k <= 512 && s.H_q / s.H_kv <= 8; }

// Where two halves pay with these keys beyond where they do with the KEYS form (rope_kept_pays; below 2^18 rows that line is kept for
// both: where it says two halves they are 0.99 to 1.9 times as fast with these keys): from 2^18 rows on.  One launch / two halves, us, 8 KV
// heads, bf16, four query heads: ranks 512, 8 sequences x 4096 rows 129 / 122 (from 32768 tokens), 132 / 127 (65536), 135 / 134
// (131072), with eight heads 130 / 125, 132 / 132, 134 / 137; 8 x 4128 136 / 128, 16 x 4096 240 / 223, 4 x 8192 124 / 116; ranks 384, 8 x
// 4096 116 / 101; ranks 256 80 / 73; ranks 128 65 / 51.  (8 x 4096 is where the one launch has nothing to pad and its rounds are
// full; there its time varies by 10 % from one card to another, and ranks 512 were 0.91 to 1.09 times as fast in two halves on different ones.)
// Quantised, 8 x 4096 from 131072 tokens: ranks 256 62.8 / 60.0 in 4 bits, 62.1 / 60.5 in 3, with eight heads 64.7 / 64.2 and 63.2 /
// 63.3; ranks 512 113.8 / 98.9.  Below: 4 x 4096 in bf16 71 / 74 (ranks 512), 42.5 / 44.4 (256), but 65 / 60 (384).
// But not bf16 rows of more than 384 and 512 ranks where the one launch is a single round of workgroups with at least 9 of 10 places filled
// and the rows are few of the tokens, so that the heads share little of what the caches hold, which the second pass over the list
// feels: 8 x 4096 rows of ranks 512 from 32768 tokens 120 / 115, 65536 123 / 124, 98304 127 / 128, 131072 127 / 130, 196608 126 / 133; eight
// heads 120 / 118, 125 / 128, 126 / 131, 127 / 133 and 128 / 137; 4 x 8192 from 131072 118 / 118, eight heads 118 / 122; 8 x 5000 149 / 150 and
// 153 / 156, 8 x 4128 (8 of 10 places) 142 / 136 and 143 / 140; 8 x 4096 of ranks 448 121 / 118.
bool rope_keys_pays(const xkv_shape &s, const Plan &p, int qbits)
{
    if (!p.absorb || s.r_v > 512 || p.n_rep > 8 || (long long)p.rows * s.k < 1 << 18) return false;
    const long long places = (long long)p.rows * p.sr_splits * p.sr_chunk;
    const bool one_round = p.rows * p.sr_splits <= 256 && 10LL * p.rows * s.k >= 9 * places;
    return qbits != 0 || s.r_k <= 384 || s.r_v != 512 || !one_round || (p.n_rep > 4 ? 16LL : 24LL) * s.k > s.L;
}

hipError_t launch_rope_keys(const xkv_shape &s, const Plan &p, const PackArgs &pa, const void *A_k, const void *B_packed, int layer,
                            const int32_t *idx, const int32_t *counts, float rope_theta, int qbits, float *logits, hipStream_t st)
{
    const size_t per_head = (size_t)(pa.F8k + pa.F8v) * 256;  // pieces of 16 B
    const u32x4_t *bsrc = B_packed ? (const u32x4_t *)B_packed + (size_t)layer * s.H_kv * per_head : (const u32x4_t *)pa.pack;
    const size_t seq_stride = (B_packed ? (size_t)s.G : 1) * s.H_kv * per_head;
    RopeFactors rope;
    for (int j = 0; j < 64; ++j) {
        const double f = std::pow((double)rope_theta, -(double)j / 64.0) / 6.283185307179586476925286766559;
        const double f256 = 256.0 * f;
        rope.f0[j] = (float)f;
        rope.f1[j] = (float)(f256 - std::floor(f256));
    }
    // two workgroups per compute unit, in whole rounds; the start of one (B^K into registers) counts as four tiles
    const int tiles = (s.k + kRows - 1) / kRows, rows = p.rows;
    int splits = 1, per = tiles;
    long long best = 0;
    const int first = (rows + 511) / 512;
    for (int rounds = first; rounds < first + 8; ++rounds) {
        long long n = 512LL * rounds / rows;
        const long long fewest = (tiles + kMaxRunTiles - 1) / kMaxRunTiles;
        n = n < fewest ? fewest : n;
        n = n > tiles ? tiles : n;
        const int each = (int)((tiles + n - 1) / n), used = (tiles + each - 1) / each;
        const long long time = ((long long)rows * used + 511) / 512 * (each + 4);
        if (best > 0 && time >= best) continue;
        best = time, splits = used, per = each;
    }
    const dim3 grid((unsigned)((long long)splits * rows));
    const int hp = head_pitch_of(p.n_rep);
#define XKV_RK(NF, QB)                                                                                                            \
    do {                                                                                                                          \
        static DynamicLdsOnce attr;                                                                                               \
        if (hipError_t e = attr.ensure((const void *)rope_keys_kernel<NF, QB>, rope_keys_lds<NF>()); e != hipSuccess) return e;   \
        hipLaunchKernelGGL((rope_keys_kernel<NF, QB>), grid, dim3(256), rope_keys_lds<NF>(), st, A_k, bsrc, seq_stride, per_head, \
                           (const u32x4_t *)pa.pack_q, idx, counts, s.L, s.r_k, s.H_kv, s.k, splits, per, p.scale, rope, logits, hp); \
    } while (0)
#define XKV_RK_Q(NF)       \
    do {                   \
        if (qbits == 4)    \
            XKV_RK(NF, 4); \
        else if (qbits == 3) \
            XKV_RK(NF, 3); \
        else               \
            XKV_RK(NF, 0); \
    } while (0)
    if (s.r_k <= 128)
        XKV_RK_Q(8);
    else if (s.r_k <= 256)
        XKV_RK_Q(16);
    else if (s.r_k <= 384)
        XKV_RK_Q(24);
    else
        XKV_RK_Q(32);
#undef XKV_RK_Q
#undef XKV_RK
    return hipGetLastError();
}

}  // namespace xkv
