// factorize.hip -- Cross-Layer Factorization (Sec. 3.1, Eq. 1) on the GPU: the caches of the G layers of a
// group, concatenated along the feature axis into X_cat [L][n] (n = G * H_kv * d_h), are replaced by a shared
// token basis A [L][r] and per-layer reconstruction matrices B_l [r][d] with A [B_1 .. B_G] the best rank-r
// approximation of X_cat.
//
// How it is computed here.  n is a few thousand while L is tens of thousands, so the right singular subspace
// is taken from the n x n Gram matrix C = X_cat^T X_cat, which is built once on the matrix cores and then
// stays in cache:
//   1. X_cat is rewritten channel-major (Xt [n][Lp], tokens contiguous, zero-padded to a multiple of 64) so
//      that both operands of the Gram product are contiguous along the summation index;
//   2. C = Xt Xt^T (lower tiles, split over the tokens, fp32 accumulation), mirrored to the full matrix;
//   3. block power iteration on C: V <- orth(C V) for a random start V [r][n], `iters` times.  The product
//      runs on the fp32 matrix cores; orth() is a Cholesky-QR in fp64 (Gram matrix of the r vectors,
//      inverse of its Cholesky factor, product with it), which keeps r directions apart whose lengths differ by many
//      orders of magnitude after the multiplication by C;
//   4. B = V rounded to the storage type (rows of B are an orthonormal basis of the dominant right singular
//      subspace), A = X_cat B^T (matrix cores again).
// A B is then X_cat projected onto the span of B's rows.  The factors differ from (U Sigma, V^T) of Eq. 1 by an
// r x r rotation inside that span, which leaves every product A B_l, and with it every quantity the decode path
// computes, unchanged.  (Randomised subspace iteration with Cholesky-QR is also what App. B.3 describes for
// the paper's own implementation; working on the Gram matrix instead of X_cat is this implementation's choice.)
#include "xkv_common.h"

#include <algorithm>
#include <type_traits>

namespace xkv {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 fz_bf16x8_t;
typedef __attribute__((ext_vector_type(16))) float fz_f32x16_t;
typedef __attribute__((ext_vector_type(4))) uint32_t fz_u32x4_t;
typedef __attribute__((ext_vector_type(4))) float fz_f32x4_t;
typedef __attribute__((address_space(3))) void fz_lds_void_t;

// ------------------------------------------------------------------------------------------------
// (1) X [G*H_kv][L][d_h] (one sequence, every layer and head of the group) -> Xt [n][Lp], row
//     cb * d_h + j = channel j of column block cb, zero beyond token L.  64 x 64 tiles through LDS.
// ------------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void xt_pack_kernel(const T *__restrict__ X, T *__restrict__ Xt, int L, int Lp, int d_h,
                                                      long long x_seq, long long xt_seq)
{
    X += (size_t)blockIdx.z * x_seq;
    Xt += (size_t)blockIdx.z * xt_seq;
    constexpr int V = 16 / sizeof(T);  // elements per 16 B
    constexpr int PPR = 64 / V;        // 16 B pieces per tile row
    __shared__ __attribute__((aligned(16))) T tile[64][64 + V];
    const int t0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    const int cb = n0 / d_h, c0 = n0 % d_h;
    const T *src = X + (size_t)cb * L * d_h + c0;
    for (int i = threadIdx.x; i < 64 * PPR; i += 256) {
        const int tt = i / PPR, p = i % PPR;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (t0 + tt < L) v = *reinterpret_cast<const uint4 *>(src + (size_t)(t0 + tt) * d_h + p * V);
        *reinterpret_cast<uint4 *>(&tile[tt][p * V]) = v;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 64 * PPR; i += 256) {
        const int c = i / PPR, p = i % PPR;
        __attribute__((aligned(16))) T vals[V];
#pragma unroll
        for (int e = 0; e < V; ++e) vals[e] = tile[p * V + e][c];
        *reinterpret_cast<uint4 *>(Xt + (size_t)(n0 + c) * Lp + t0 + p * V) = *reinterpret_cast<const uint4 *>(vals);
    }
}

// ------------------------------------------------------------------------------------------------
// (2) out[m][n] = sum_k P[m][k] Q[n][k] on the matrix cores, both operands contiguous along k.
//
// Element (row, k) of an operand lives at base + (k / kbw) * kblk + row * pitch + k % kbw: a plain row-major
// matrix has kbw = K, and a cache stored as [column block][token][d_h] is read as X_cat [token][n] with
// kbw = d_h, kblk = L * d_h, pitch = d_h.  K is consumed in slabs of 128 B per row (64 bf16 or 32 fp32
// values); kbw is a multiple of the slab.
//
// Workgroup: 8 wavefronts, a 256 x 256 output tile, wavefront (wm, wn) owns rows 64 wm .. +63 and columns
// 128 wn .. +127 as 2 x 4 accumulator tiles of 32 x 32.  A slab of the 256 + 256 operand rows (64 KiB) is
// copied global -> LDS directly, two stages: one copy instruction moves 8 rows x 128 B, lane l fetching the 16 B
// piece (l % 8) ^ (row / 2) % 8 of row l / 8, so that a row's pieces sit in LDS xor-swizzled by (row / 2) % 8 and
// the fragment reads (consecutive rows, same piece) spread over all 64 banks.  Rows beyond the operand's end are
// clamped to its last row; what they produce is never stored.
// Output: fp32 partial planes out_f32[split][m][n] (summed by a second kernel), or, with one split, the
// final matrix in fp32 or bf16.  With lower_only (P == Q) only tiles on or below the diagonal are computed.
// ------------------------------------------------------------------------------------------------
struct GemmOperand {
    const void *base;
    long long pitch, kblk;  // elements
    int kbw, rows;
    long long seq;  // elements between the matrices of consecutive sequences (blockIdx.z)
};
struct GemmArgs {
    GemmOperand P, Q;
    int n_slabs, splits, lower_only, tiles_n, tiles;  // tiles: output tiles per split (lower_only: on or below the diagonal)
    float *out_f32;
    bf16_t *out_bf16;
    long long ldo, plane, out_seq;
};

constexpr int kGemmThreads = 512, kGemmTile = 256, kGemmStages = 2, kGemmStage = 512 * 128, kGemmLds = kGemmStages * kGemmStage;

// Decoding of a linear index into a pair (bi, bj), bj <= bi, enumerated row by row.
__device__ __forceinline__ void fz_lower_pair(int t, int &bi, int &bj)
{
    int m = (int)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
    while ((m + 1) * (m + 2) / 2 <= t) ++m;
    while (m * (m + 1) / 2 > t) --m;
    bi = m;
    bj = t - m * (m + 1) / 2;
}

// The t-th tile on or below the diagonal of a T x T tile grid, counted patch by patch (patches of 4 x 4 tiles,
// row by row; inside a patch row by row).
__device__ __forceinline__ void fz_lower_patch_tile(int t, int T, int &tm, int &tn)
{
    const int PT = (T + 3) / 4;
    for (int pr = 0; pr < PT; ++pr)
        for (int pc = 0; pc <= pr; ++pc) {
            const int m0 = 4 * pr, n0 = 4 * pc, m1 = (m0 + 4 < T) ? m0 + 4 : T, n1 = (n0 + 4 < T) ? n0 + 4 : T;
            for (int m = m0; m < m1; ++m) {
                const int hi = (n1 - 1 < m) ? n1 - 1 : m, cnt = hi - n0 + 1;  // tiles (m, n0 .. hi)
                if (cnt <= 0) continue;
                if (t < cnt) {
                    tm = m;
                    tn = n0 + t;
                    return;
                }
                t -= cnt;
            }
        }
    tm = tn = 0;  // not reached for t < T (T + 1) / 2
}

// The eight copy instructions of a wavefront for one slab: its 64 operand rows, 8 rows x 128 B each.
__device__ __forceinline__ void fz_issue_slab(const unsigned char *const (&rowp)[8], size_t off, uint32_t dst)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) copy16_global_to_lds(rowp[j] + off, dst + j * 1024);
}

// One k-step of a wavefront: its 2 + 4 operand fragments (32 rows each, the lane's 16 B piece), and the 8 products.
__device__ __forceinline__ void fz_read_frags(fz_u32x4_t (&af)[2], fz_u32x4_t (&qf)[4], const fz_u32x4_t *st, int arow, int qrow,
                                              int slot)
{
#pragma unroll
    for (int i = 0; i < 2; ++i) af[i] = st[arow + i * 256 + slot];
#pragma unroll
    for (int j = 0; j < 4; ++j) qf[j] = st[qrow + j * 256 + slot];
}

template <typename T>
__device__ __forceinline__ void fz_multiply(fz_f32x16_t (&acc)[2][4], const fz_u32x4_t (&af)[2], const fz_u32x4_t (&qf)[4])
{
    if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(fz_bf16x8_t, af[i]),
                                                                    __builtin_bit_cast(fz_bf16x8_t, qf[j]), acc[i][j], 0, 0, 0);
    } else {
        // a 16 B piece holds 4 consecutive k of the lane's row; step e pairs k = 8 s + e (lanes 0-31) with
        // k = 8 s + 4 + e (lanes 32-63) on both operands
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(fz_f32x4_t, af[i])[e],
                                                                     __builtin_bit_cast(fz_f32x4_t, qf[j])[e], acc[i][j], 0, 0, 0);
    }
}

template <typename T>
__global__ __launch_bounds__(kGemmThreads) void gemm_nt_kernel(const GemmArgs a)
{
    constexpr int E = 128 / (int)sizeof(T);  // elements per slab row
    extern __shared__ __attribute__((aligned(16))) unsigned char fz_smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = wave_id();
    const int m32 = lane & 31, h = lane >> 5;

    // Work item -> compute-unit die.  Workgroups go to the 8 dies (each with its own L2) round-robin by their
    // linear id, so die x = blockIdx.x % 8 takes the x-th eighth of the item list, in order: the items a die
    // works on at the same time are neighbours in the list, and the list is ordered so that neighbours share
    // operand rows (same range of k; tiles in 4 x 4 patches, or side by side along n).
    const int items = a.tiles * a.splits, per_die = (items + 7) / 8;
    const int q = (int)(blockIdx.x & 7) * per_die + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per_die || q >= items) return;
    const int split = q / a.tiles, t = q % a.tiles;
    int tm, tn;
    if (a.lower_only) {
        fz_lower_patch_tile(t, a.tiles_n, tm, tn);
    } else {
        tm = t / a.tiles_n;
        tn = t % a.tiles_n;
    }
    const int sb_begin = (int)((long long)a.n_slabs * split / a.splits);
    const int sb_end = (int)((long long)a.n_slabs * (split + 1) / a.splits);

    // ---- copy side: wavefronts 0-3 bring in P rows 64 w .. +63 of the tile, wavefronts 4-7 the Q rows
    const bool is_p = w < 4;
    const unsigned char *op_base = reinterpret_cast<const unsigned char *>(is_p ? a.P.base : a.Q.base) +
                                   (size_t)blockIdx.z * (size_t)(is_p ? a.P.seq : a.Q.seq) * sizeof(T);
    const long long op_pitch = is_p ? a.P.pitch : a.Q.pitch, op_kblk = is_p ? a.P.kblk : a.Q.kblk;
    const int op_kbw = is_p ? a.P.kbw : a.Q.kbw, op_rows = is_p ? a.P.rows : a.Q.rows;
    const int origin = (is_p ? tm : tn) * kGemmTile + (w & 3) * 64;
    const unsigned char *rowp[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        int R = origin + 8 * j + (lane >> 3);
        R = R < op_rows ? R : op_rows - 1;
        const int piece = (lane & 7) ^ ((4 * j + (lane >> 4)) & 7);  // slot ^ (stage row / 2) % 8
        rowp[j] = op_base + (size_t)((long long)R * op_pitch) * sizeof(T) + piece * 16;
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(fz_lds_void_t *)fz_smem + (uint32_t)(w * 8 * 1024);
    // Byte offset of the next slab to request within an operand row, advanced without divisions: slabs are
    // requested in order, and past the last one the last one again.
    const long long kk0 = (long long)sb_begin * E;
    int kin = (int)(kk0 % op_kbw);
    size_t slab_off = (size_t)((kk0 / op_kbw) * op_kblk + kin) * sizeof(T);
    const size_t blk_jump = (size_t)(op_kblk - op_kbw) * sizeof(T);
    int to_advance = sb_end - sb_begin - 1;  // how many more times the offset moves on
    auto next_slab = [&]() __attribute__((always_inline)) {
        const size_t cur = slab_off;
        if (to_advance > 0) {
            --to_advance;
            kin += E;
            slab_off += E * sizeof(T);
            if (kin >= op_kbw) {
                kin = 0;
                slab_off += blk_jump;
            }
        }
        return cur;
    };

    // ---- compute side
    const int wm = w & 3, wn = w >> 2;
    fz_f32x16_t acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    // 16 B index of (row, piece c) in a stage: row * 8 + (c ^ (row / 2) % 8); (row / 2) % 8 == (m32 / 2) % 8 for every row
    // read here.  With 64 banks of 4 B, 16 consecutive rows x one piece then cover every bank exactly once.
    const int arow = (64 * wm + m32) * 8, qrow = (256 + 128 * wn + m32) * 8, sw = (m32 >> 1) & 7;

    // Two stages of 128 B per row (a whole cache line per row and request: row-scattered 64 B pieces reach only about
    // 60 % of the L2 -> LDS rate of whole lines): the next slab is requested right after the barrier that retires
    // the previous one, while the current one is multiplied.  Within a slab the fragments of a step are read during
    // the products of the step before (the scheduling fences keep that order).
    const int n_sb = sb_end - sb_begin;
    fz_issue_slab(rowp, next_slab(), lds0);
    fz_u32x4_t a0[2], q0[4], a1[2], q1[4];
    for (int i = 0; i < n_sb; ++i) {
        XKV_WAIT_VMCNT(0);   // slab i is in LDS
        lds_barrier();   // ... for every wavefront; and nobody reads the other stage any more
        if (i + 1 < n_sb) fz_issue_slab(rowp, next_slab(), lds0 + (uint32_t)(((i + 1) & 1) * kGemmStage));
        const fz_u32x4_t *st = reinterpret_cast<const fz_u32x4_t *>(fz_smem + (i & 1) * kGemmStage);
        fz_read_frags(a0, q0, st, arow, qrow, h ^ sw);
        __builtin_amdgcn_sched_barrier(0);
        fz_read_frags(a1, q1, st, arow, qrow, (2 + h) ^ sw);
        __builtin_amdgcn_sched_barrier(0);
        fz_multiply<T>(acc, a0, q0);
        __builtin_amdgcn_sched_barrier(0);
        fz_read_frags(a0, q0, st, arow, qrow, (4 + h) ^ sw);
        __builtin_amdgcn_sched_barrier(0);
        fz_multiply<T>(acc, a1, q1);
        __builtin_amdgcn_sched_barrier(0);
        fz_read_frags(a1, q1, st, arow, qrow, (6 + h) ^ sw);
        __builtin_amdgcn_sched_barrier(0);
        fz_multiply<T>(acc, a0, q0);
        __builtin_amdgcn_sched_barrier(0);
        fz_multiply<T>(acc, a1, q1);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- store: accumulator register v of a 32 x 32 tile is row 8 (v / 4) + 4 h + v % 4, column m32
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int col = tn * kGemmTile + 128 * wn + 32 * j + m32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = tm * kGemmTile + 64 * wm + 32 * i + 8 * (v / 4) + 4 * h + (v % 4);
                if (row < a.P.rows && col < a.Q.rows) {
                    const size_t o = (size_t)blockIdx.z * a.out_seq + (size_t)row * a.ldo + col;
                    if (a.out_bf16)
                        a.out_bf16[o] = f32_to_bf16(acc[i][j][v]);
                    else
                        a.out_f32[(size_t)split * a.plane + o] = acc[i][j][v];
                }
            }
        }
}

// (2b) C = sum of the split planes of the lower 64 x 64 blocks, mirrored into the upper triangle.  Memory bound: n = 4096, three planes,
// 164 MB in 34 us (64 with four bytes per request and one plane's value after the other).
__global__ __launch_bounds__(256) void gram_finish_kernel(const float *__restrict__ part, float *__restrict__ C, int n,
                                                          int splits, long long plane, long long part_seq)
{
    part += (size_t)blockIdx.z * part_seq;
    C += (size_t)blockIdx.z * n * n;
    const int bm = blockIdx.y, bn = blockIdx.x;
    if (bn > bm) return;
    __shared__ float tile[64][65];
    const int c4 = (threadIdx.x & 15) * 4, r0 = threadIdx.x >> 4;  // (n is a multiple of 64)
    fz_f32x4_t v[4] = {};
    for (int s = 0; s < splits; ++s)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] += *reinterpret_cast<const fz_f32x4_t *>(part + (size_t)s * plane + (size_t)(bm * 64 + r0 + 16 * u) * n + bn * 64 + c4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        *reinterpret_cast<fz_f32x4_t *>(C + (size_t)(bm * 64 + r0 + 16 * u) * n + bn * 64 + c4) = v[u];
#pragma unroll
        for (int e = 0; e < 4; ++e) tile[r0 + 16 * u][c4 + e] = v[u][e];
    }
    __syncthreads();
    if (bn == bm) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) {  // rows of the upper block
        fz_f32x4_t x;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = tile[c4 + e][r0 + 16 * u];
        *reinterpret_cast<fz_f32x4_t *>(C + (size_t)(bn * 64 + r0 + 16 * u) * n + bm * 64 + c4) = x;
    }
}

// (2c) out = sum of `splits` planes of `count` floats.
__global__ __launch_bounds__(256) void sum_planes_kernel(const float *__restrict__ part, float *__restrict__ out,
                                                         long long count, int splits, long long plane, long long part_seq)
{
    part += (size_t)blockIdx.z * part_seq;
    out += (size_t)blockIdx.z * count;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    float v = 0.0f;
    for (int s = 0; s < splits; ++s) v += part[(size_t)s * plane + i];
    out[i] = v;
}

// (3a) Start block of the iteration: r x n values in (-1, 1) from a counter hash of (seed, index).
__global__ __launch_bounds__(256) void init_v_kernel(float *__restrict__ Vt, long long count, uint32_t seed)
{
    Vt += (size_t)blockIdx.z * count;
    seed += 0x9E37u * blockIdx.z;
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    uint32_t x = (uint32_t)i * 0x9E3779B9u + seed * 0x85EBCA6Bu + (uint32_t)(i >> 32) * 0xC2B2AE35u + 0x27D4EB2Fu;
    x ^= x >> 16; x *= 0x7FEB352Du; x ^= x >> 15; x *= 0x846CA68Bu; x ^= x >> 16;
    Vt[i] = ((float)(x >> 8) + 0.5f) * (2.0f / 16777216.0f) - 1.0f;
}

// fp64 matrix-core instruction v_mfma_f64_16x16x4_f64: D[16][16] += A[16][4] B[4][16], one double per lane for A
// (row lane % 16, k = lane / 16) and for B (column lane % 16, k = lane / 16); lane l holds D[l / 16 + 4 v][l % 16]
// in element v of its four results.
typedef __attribute__((ext_vector_type(2))) double fz_f64x2_t;
typedef __attribute__((ext_vector_type(4))) double fz_f64x4_t;

__device__ __forceinline__ void fz_gram_fetch(float (&fa)[8][2], float (&fb)[8][2], const float *__restrict__ Xn,
                                              const float *__restrict__ Wn, int n0, int n_begin, int n_end, int r,
                                              const int (&ci)[2], const int (&cj)[2], int kk)
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int row = n0 + 4 * q + kk;
        const bool ok = row < n_end;
        const size_t at = (size_t)(ok ? row : n_begin) * r;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            fa[q][u] = (ok && ci[u] < r) ? Xn[at + ci[u]] : 0.0f;
            fb[q][u] = (ok && cj[u] < r) ? Wn[at + cj[u]] : 0.0f;
        }
    }
}

// (3b) Products of r vectors with r vectors, products and sums in fp64: G[i][j] = sum_n X[n][i] W[n][j].  One wavefront
// per 32 x 32 block and per range of n (one partial plane per range, added up in a fixed order by the next kernel); a
// step multiplies 4 rows, widened to fp64 as they are loaded.  LOWER: X = W, the blocks on or below the diagonal (the
// Gram matrix of the orthonormalisation); otherwise all of them (the Rayleigh-Ritz matrix, X = V: 59 us at r = 512, n =
// 4096 where one workgroup per block without matrix instructions took 466).
template <bool LOWER>
__global__ __launch_bounds__(256) void gram_f64_kernel(const float *__restrict__ Xn, long long x_seq,
                                                       const float *__restrict__ Wn, double *__restrict__ planes, int n,
                                                       int r, int splits, int n_pairs)
{
    Xn += (size_t)blockIdx.z * x_seq;
    Wn += (size_t)blockIdx.z * n * r;
    planes += (size_t)blockIdx.z * splits * r * r;
    const int pair = blockIdx.x * 4 + wave_id();
    if (pair >= n_pairs) return;
    int bi, bj;
    if (LOWER) {
        fz_lower_pair(pair, bi, bj);
    } else {
        const int gb = (r + 31) / 32;
        bi = pair / gb;
        bj = pair % gb;
    }
    const int split = blockIdx.y, lane = lane_id(), col = lane & 15, kk = lane >> 4;
    const int n_begin = (int)((long long)n * split / splits), n_end = (int)((long long)n * (split + 1) / splits);
    fz_f64x4_t acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
    int ci[2], cj[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        ci[u] = bi * 32 + 16 * u + col;
        cj[u] = bj * 32 + 16 * u + col;
    }
    // eight steps (32 rows of W) at a time; the loads of the next eight are requested before the 32 products of
    // the current ones
    float fa[8][2], fb[8][2];
    fz_gram_fetch(fa, fb, Xn, Wn, n_begin, n_begin, n_end, r, ci, cj, kk);
    for (int n0 = n_begin; n0 < n_end; n0 += 32) {
        double da[8][2], db[8][2];
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                da[q][u] = (double)fa[q][u];
                db[q][u] = (double)fb[q][u];
            }
        if (n0 + 32 < n_end) fz_gram_fetch(fa, fb, Xn, Wn, n0 + 32, n_begin, n_end, r, ci, cj, kk);
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 2; ++v)
                    acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(da[q][u], db[q][v], acc[u][v], 0, 0, 0);
    }
    double *out = planes + (size_t)split * r * r;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = bi * 32 + 16 * u + kk + 4 * e, j = bj * 32 + 16 * v + col;
                if (i < r && j < r) out[(size_t)i * r + j] = acc[u][v][e];
            }
}

__global__ __launch_bounds__(256) void gram_sum_kernel(const double *__restrict__ planes, double *__restrict__ G,
                                                       double *__restrict__ diag0, int r, int splits)
{
    planes += (size_t)blockIdx.z * splits * r * r;
    G += (size_t)blockIdx.z * r * r;
    diag0 += (size_t)blockIdx.z * r;
    const int i = blockIdx.y, j = blockIdx.x * 256 + threadIdx.x;
    if (j >= r || (j >> 5) > (i >> 5)) return;
    const size_t idx = (size_t)i * r + j;
    double v = 0.0;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) v += planes[(size_t)s * r * r + idx];
    G[idx] = v;
    if (i == j) diag0[i] = v;
}

// (3c) The inverse Li of the Cholesky factor Lc of G + shift I, right-looking in panels of 32 columns: the factor's columns are eliminated from
// the trailing matrix and, the same way, from the rows of an identity that becomes the inverse.  A launch has three kinds of
// workgroups, for the panel c0 .. c0 + 31, whose diagonal block of Li is there:
//   * 32 x 32 blocks of the trailing matrix, on or below the diagonal.  The panel entries Lc[j'][c0 .. c0 + 32) of its rows and of its
//     columns are G[j'][panel] times the transposed diagonal block of Li (fp64 matrix cores, 16 rows a step) and stay in LDS; their
//     product is subtracted;
//   * 32 x 32 blocks of the unfinished inverse X: rows below the panel, columns up to its end.  The panel's rows of X times the diagonal
//     block of Li are the final rows of Li (written by the first block of each column); with the panel entries of the block's rows
//     they are subtracted.  X lies transposed above the diagonal of G, which the factorization does not use;
//   * workgroup 0 prepares the next panel: it brings the next diagonal block up to date by itself (its 32 panel rows and one
//     outer product), factors and inverts it and leaves the inverse in Li.  The first launch, c0 = -32, has only this
//     workgroup; in the last, the last panel's, it has nothing to do.
// The elimination runs in one wavefront without a barrier, 16 columns at a time: a lane holds a row of the block or a column of an
// identity, and step c is the same for both: t = x[c] / sqrt(pivot), x[j] -= (t of lane j) t for j > c.  What t leaves in
// the lanes are column c of the factor and row c of its inverse.  Between the two halves of a block of 32 the lower right quarter and
// the start of the inverse's lower left quarter are brought up to date with eight matrix instructions.
// shift = 1e-13 * max diagonal of the original G (diag0) keeps the factor defined when the r vectors are
// numerically dependent (an X_cat of rank below r): such directions come out short instead of normalised and
// contribute nothing to A B.
// What bounds it: the chain of its launches, 17 at r = 512, each of which takes as long as its workgroup 0 (the last has none): 12 us
// in general, 9.3 where r is a multiple of 32: few wavefronts do all the work, so instructions count, and there every row comes in 16-byte
// runs and without bounds checks; the maximum of the diagonal is found once (11.4 -> 9.3 us).  32 steps on rows of 32 elements with scalar
// broadcasts of t took 21.5 us per launch (13 of them the steps); 16 + 16 steps 17, with workgroups of 32 whole rows, 25 us in the first
// launches and 14 in the last; blocks of 32 x 32 12 in all of them.  Panels of 16 columns, twice as many launches, take longer at every
// rank (factorisation at r = 1024, one and four sequences: 14.3 and 29.2 ms, with 32 columns 13.7 and 26.9).
constexpr int kCholRB = 32, kCholThreads = 512, kCholPitch = 36;  // panels and blocks; doubles per row of the panel in LDS
// 64 rows of the panel; workgroup 0: its rows and three blocks
constexpr size_t kCholLds = 8 * std::max<size_t>(2 * kCholRB * kCholPitch, kCholRB * kCholPitch + 3 * kCholRB * (kCholRB + 1));

// 1 / sqrt(x): the hardware's estimate y (better than 2^-20) and one third-order step, y (1 + e / 2 + 3 e^2 / 8) with
// e = 1 - x y^2: a chain of four dependent operations where two Newton steps are eight.
__device__ __forceinline__ double fz_rsqrt(double x)
{
    const double y = __builtin_amdgcn_rsq(x), e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// The value of lane N of the same 16.
template <int N> __device__ __forceinline__ double fz_lane_of_16(double x)
{
    return __builtin_amdgcn_update_dpp(0.0, x, 0x150 + N, 0xF, 0xF, false);  // row_newbcast
}

// f(I), f(I + 1) .. with the index as a type
template <int I, int END, typename F> __device__ __forceinline__ void fz_for(F f)
{
    if constexpr (I < END) {
        f(std::integral_constant<int, I>{});
        fz_for<I + 1, END>(f);
    }
}

// Products over 16 or 32 positions in steps of 4: in step s, lane group kk takes position fz_run_k(s, kk), so that what a lane needs of
// a row are runs of four.
__device__ __forceinline__ constexpr int fz_run_k(int s, int kk) { return 16 * (s >> 2) + 4 * kk + (s & 3); }

// The elements fz_run_k(0 .. N - 1, kk) of a row.
template <int N> __device__ __forceinline__ void fz_run_row(const double *row, int kk, double (&v)[N])
{
#pragma unroll
    for (int h = 0; h < N / 2; ++h) {
        const fz_f64x2_t t = *reinterpret_cast<const fz_f64x2_t *>(row + 16 * (h >> 1) + 4 * kk + 2 * (h & 1));
        v[2 * h] = t[0];
        v[2 * h + 1] = t[1];
    }
}

template <bool FULL>  // FULL: r a multiple of 32
__global__ __launch_bounds__(kCholThreads) void chol_panel_kernel(double *__restrict__ G, double *__restrict__ Li,
                                                                  double *__restrict__ diag0, int r, int c0)
{
    constexpr int PB = kCholRB, KS = PB / 4, CT = PB / 16, PITCH = kCholPitch, LP = PB + 1, WAVES = kCholThreads / 64;
    G += (size_t)blockIdx.z * r * r;
    Li += (size_t)blockIdx.z * r * r;
    diag0 += (size_t)blockIdx.z * r;
    extern __shared__ __attribute__((aligned(16))) unsigned char fz_smem[];
    double *P = reinterpret_cast<double *>(fz_smem);  // [rows][PITCH] panel entries of Lc
    const int tid = threadIdx.x, lane = tid & 63, w = wave_id(), l16 = lane & 15, kk = lane >> 4;
    const int d0 = c0 + PB;  // first row below the diagonal block

    // Sixteen rows (lane l16 holds fz_run_k(.., kk) of row l16) times columns 16 ct .. of the transposed inverse of the panel's diagonal
    // block -> rows `at` .. of P
    auto times_inverse = [&](const double (&ga)[KS], int ct, int at) __attribute__((always_inline)) {
        double lb[KS];
        const int ir = c0 + 16 * ct + l16;
        if constexpr (FULL) {
            fz_run_row(Li + (size_t)ir * r + c0, kk, lb);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                lb[ks] = (ir < r && c0 + fz_run_k(ks, kk) < r) ? Li[(size_t)ir * r + c0 + fz_run_k(ks, kk)] : 0.0;
        }
        fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[ks], lb[ks], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) P[(at + kk + 4 * v) * PITCH + 16 * ct + l16] = acc[v];
    };
    auto panel_tile = [&](int row0, int ct, int at) __attribute__((always_inline)) {  // rows of the factor
        const int row = row0 + l16;
        double ga[KS];
        if constexpr (FULL) {
            fz_run_row(G + (size_t)row * r + c0, kk, ga);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) ga[ks] = row < r ? G[(size_t)row * r + c0 + fz_run_k(ks, kk)] : 0.0;
        }
        times_inverse(ga, ct, at);
    };
    auto inverse_tile = [&](int col0, int ct, int at) __attribute__((always_inline)) {  // columns of the panel's rows of the inverse
        const int col = col0 + l16;
        double ga[KS];
        if (FULL && col0 < c0) {
            fz_run_row(G + (size_t)col * r + c0, kk, ga);
        } else {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int k = fz_run_k(ks, kk);
                ga[ks] = !FULL && col < c0 ? (c0 + k < r ? G[(size_t)col * r + c0 + k] : 0.0) : col == c0 + k ? 1.0 : 0.0;
            }
        }
        times_inverse(ga, ct, at);
    };
    auto outer = [&](int rs, int cs) __attribute__((always_inline)) {  // tile of 16 x 16 of the panel's outer product
        double a[KS], b[KS];
        fz_run_row(P + (rs + l16) * PITCH, kk, a);
        fz_run_row(P + (cs + l16) * PITCH, kk, b);
        fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ks], b[ks], acc, 0, 0, 0);
        return acc;
    };

    if (blockIdx.x > 0) {
        const int nb = (r - d0 + kCholRB - 1) / kCholRB, n_tri = nb > 0 ? nb * (nb + 1) / 2 : 0;
        const bool inverse = (int)blockIdx.x - 1 >= n_tri;
        int bi, bj;
        if (inverse) {
            const int x = (int)blockIdx.x - 1 - n_tri, n_cb = (d0 + kCholRB - 1) / kCholRB;
            bi = x / n_cb;
            bj = x % n_cb;
        } else {
            fz_lower_pair((int)blockIdx.x - 1, bi, bj);
        }
        const int i0 = d0 + kCholRB * bi, j0 = (inverse ? 0 : d0) + kCholRB * bj, own_end = (i0 + kCholRB) < r ? (i0 + kCholRB) : r;
        // tile (w / 2 % 2, w % 2) of the block for wavefronts 0 .. 3, requested first: rows i0 .., columns j0 .. of the trailing matrix, or
        // columns j0 .., rows i0 .. of the inverse, which lies transposed above the diagonal
        const int rt = (w >> 1) & 1, ctile = w & 1, jc = j0 + 16 * ctile + l16;
        const bool rows = !FULL || i0 < r;  // (the last launch has rows of the inverse to write, and no blocks below them)
        double old[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (FULL) {
                if (!rows || w >= 4 || (inverse && j0 >= c0))
                    old[v] = 0.0;
                else if (inverse)
                    old[v] = G[(size_t)(j0 + 16 * ctile + kk + 4 * v) * r + i0 + 16 * rt + l16];
                else
                    old[v] = G[(size_t)(i0 + 16 * rt + kk + 4 * v) * r + jc];
            } else if (inverse) {
                const int col = j0 + 16 * ctile + kk + 4 * v, irow = i0 + 16 * rt + l16;
                old[v] = (w < 4 && irow < own_end && col < c0) ? G[(size_t)col * r + irow] : 0.0;
            } else {
                const int irow = i0 + 16 * rt + kk + 4 * v;
                old[v] = (w < 4 && irow < own_end && jc <= irow) ? G[(size_t)irow * r + jc] : 0.0;
            }
        }
        // panel entries of the block's 32 rows; of its 32 columns
        const bool square = !inverse && bi == bj;
        for (int item = w; item < (square ? 2 : 4) * CT; item += WAVES) {
            const int half = item / (2 * CT), rest = item % (2 * CT), ct = rest % CT, at = 16 * (rest / CT);
            if (half == 0) {
                if (rows) panel_tile(i0 + at, ct, at);
            } else if (inverse)
                inverse_tile(j0 + at, ct, kCholRB + at);
            else
                panel_tile(j0 + at, ct, kCholRB + at);
        }
        __syncthreads();
        if (inverse && bi == 0)  // the panel's rows of the inverse are final (its diagonal block is there already)
            for (int t = tid; t < PB * kCholRB; t += kCholThreads) {
                const int row = c0 + t / kCholRB, col = j0 + t % kCholRB;
                if (row < r && col < c0) Li[(size_t)row * r + col] = P[(kCholRB + col - j0) * PITCH + row - c0];
            }
        if (w < 4 && rows && !(square && ctile > rt)) {
            if (inverse) {
                const fz_f64x4_t acc = outer(kCholRB + 16 * ctile, 16 * rt);
                const int irow = i0 + 16 * rt + l16;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int col = j0 + 16 * ctile + kk + 4 * v;
                    if (FULL || (irow < own_end && col < d0)) G[(size_t)col * r + irow] = old[v] - acc[v];
                }
            } else {
                const fz_f64x4_t acc = outer(16 * rt, (square ? 0 : kCholRB) + 16 * ctile);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int irow = i0 + 16 * rt + kk + 4 * v;
                    // (the next diagonal block is workgroup 0's: it reads what this launch began with)
                    if ((FULL || irow < own_end) && jc <= irow && irow >= d0 + PB) G[(size_t)irow * r + jc] = old[v] - acc[v];
                }
            }
        }
        return;
    }
    if (d0 >= r) return;  // (the last launch: the last panel's rows of the inverse)

    // ---- workgroup 0: the next diagonal block, rows and columns d0 .. d0 + pwc - 1
    double *D = P + PB * PITCH, *LF = D + PB * LP, *LI = LF + PB * LP;  // [PB][LP] block, its factor, the inverse
    __shared__ double red[WAVES];
    const int pwc = FULL || (r - d0) >= PB ? PB : r - d0;
    double mx = c0 < 0 ? 0.0 : diag0[0];  // the first launch leaves the largest element of the diagonal there
    double g0[4];  // this wavefront's tile (w / CT, w % CT) of the block
    const int tr = w / CT, tc = w % CT;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = 16 * tr + kk + 4 * v, j = 16 * tc + l16;
        g0[v] = (w < CT * CT && (FULL || (i < pwc && j <= i))) ? G[(size_t)(d0 + i) * r + d0 + j] : 0.0;
    }
    if (c0 < 0) {
        for (int i = tid; i < r; i += kCholThreads) mx = fmax(mx, diag0[i]);
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        if (lane == 0) red[w] = mx;
    } else if (w < CT * CT) {
        panel_tile(d0 + 16 * tr, tc, 16 * tr);  // (rows beyond the matrix are zero)
    }
    __syncthreads();
    if (c0 < 0) {
        mx = red[0];
#pragma unroll
        for (int ww = 1; ww < WAVES; ++ww) mx = fmax(mx, red[ww]);
        if (tid == 0) diag0[0] = mx;
    }
    const double shift = fmax(1e-13 * mx, 1e-300);
    if (w < CT * CT) {
        fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
        if (c0 >= 0) acc = outer(16 * tr, 16 * tc);
#pragma unroll
        for (int v = 0; v < 4; ++v) {  // (rows beyond the matrix are identity rows)
            const int i = 16 * tr + kk + 4 * v, j = 16 * tc + l16;
            D[i * LP + j] = (i < pwc && j <= i) ? g0[v] - acc[v] + (i == j ? shift : 0.0) : i == j ? 1.0 : 0.0;
        }
    }
    __syncthreads();
    if (w == 0) {
        // 16 columns at a time.  Every 16 lanes hold the block's lower triangle, lane l16 row l16 (x), and beside it (y) the lanes kk = 1
        // column l16 of an identity, kk = 2 row l16 of the block's lower left quarter, then column l16 of what the inverse's lower left
        // quarter comes from
        double x[16], y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            x[j] = D[l16 * LP + j];
            y[j] = kk == 1 ? (l16 == j ? 1.0 : 0.0) : kk == 2 ? D[(PB - 16 + l16) * LP + j] : 0.0;
        }
        double *out = kk == 0 ? LF + l16 * LP : kk == 1 ? LI + l16 : kk == 2 ? LF + (PB - 16 + l16) * LP : LI + PB - 16 + l16;
        int step = kk & 1 ? LP : 1;
        bool store = true;
#pragma unroll 1
        for (int half = 0; half < CT; ++half) {
            fz_for<0, 16>([&](auto cc) __attribute__((always_inline)) {
                constexpr int c = decltype(cc)::value;
                double piv = fz_lane_of_16<c>(x[c]);
                piv = piv > shift * 1e-3 ? piv : shift * 1e-3;
                const double rs = fz_rsqrt(piv), t = l16 < c ? 0.0 : x[c] * rs, ty = y[c] * rs;
                if (store) out[c * step] = kk == 0 ? t : ty;
                fz_for<c + 1, 16>([&](auto jj) __attribute__((always_inline)) {
                    constexpr int j = decltype(jj)::value;
                    const double tj = fz_lane_of_16<j>(t);
                    x[j] = fma(tj, -t, x[j]);
                    y[j] = fma(tj, -ty, y[j]);
                });
            });
            if (half + 1 == CT) break;
            // lower right quarter minus the product of the lower left quarter of the factor with itself; and minus its product with the
            // inverse of the upper left one
            __builtin_amdgcn_wave_barrier();
            double *F = LF + 16 * LP, *Q = D + 16 * LP;  // (Q: the quarters of D that were read above)
            fz_f64x4_t s0 = fz_f64x4_t{0.0, 0.0, 0.0, 0.0}, s1 = s0;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const double f = F[l16 * LP + 4 * ks + kk], v = LI[(4 * ks + kk) * LP + l16];
                s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(f, f, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(f, v, s1, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Q[(kk + 4 * v) * LP + 16 + l16] -= s0[v];
                Q[(kk + 4 * v) * LP + l16] = -s1[v];
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                x[j] = Q[l16 * LP + 16 + j];
                y[j] = kk == 1 ? (l16 == j ? 1.0 : 0.0) : kk == 2 ? Q[j * LP + l16] : 0.0;
            }
            out = kk == 0 ? LF + (16 + l16) * LP + 16 : LI + 16 * LP + (kk == 1 ? 16 : 0) + l16;
            step = kk == 0 ? 1 : LP;
            store = kk < 3;
        }
    }
    __syncthreads();
    if constexpr (FULL) {
        const int row = tid / (PB / 2), col = tid % (PB / 2) * 2;
        static_assert(kCholThreads == PB * PB / 2, "two elements each");
        *reinterpret_cast<fz_f64x2_t *>(Li + (size_t)(d0 + row) * r + d0 + col) = fz_f64x2_t{LI[row * LP + col], LI[row * LP + col + 1]};
        return;
    }
    for (int t = tid; t < PB * PB; t += kCholThreads) {
        const int row = t / PB, col = t % PB;
        if (row < pwc && col < pwc) Li[(size_t)(d0 + row) * r + d0 + col] = LI[row * LP + col];
    }
}

// (3d) V = Lc^-1 W: Vt[i][n] = sum over c <= i of Li[i][c] Wn[n][c] on the fp64 matrix cores, written as fp32.  A wavefront makes tiles of 32
// x 32, the four of a workgroup next to each other in n; it takes a block of 32 rows of Vt from the bottom, whose sums are long, and
// one from the top, so that all are equally long.  Of 16 values of c a lane asks for four in a row, two such steps ahead.
// What bounds it: the matrix cores (16 us of products at r = 512, n = 4096).  Forward substitution in blocks of 16, the factor instead of
// its inverse, took 121 us: 32 dependent steps of two barriers.
template <bool VEC>  // r a multiple of four
__global__ __launch_bounds__(256) void orth_apply_kernel(const float *__restrict__ Wn, const double *__restrict__ Li, float *__restrict__ Vt,
                                                         int n, int r)
{
    Wn += (size_t)blockIdx.z * n * r;
    Li += (size_t)blockIdx.z * r * r;
    Vt += (size_t)blockIdx.z * n * r;
    const int lane = lane_id(), w = wave_id(), l16 = lane & 15, kk = lane >> 4;
    const int n0 = blockIdx.x * 128 + 32 * w, n_blocks = (r + 31) / 32;
    if (n0 >= n) return;
    struct Step {
        double a[2][4];
        float b[2][4];
    };
    for (int turn = 0; turn < 2; ++turn) {
        const int blk = turn == 0 ? n_blocks - 1 - (int)blockIdx.y : (int)blockIdx.y;
        if (turn == 1 && blk == n_blocks - 1 - (int)blockIdx.y) break;
        const int i0 = 32 * blk, c_end = i0 + 32 < r ? i0 + 32 : r, steps = (c_end + 15) / 16;
        auto fetch = [&](Step &x, int step) __attribute__((always_inline)) {
            const int c = 16 * step + 4 * kk;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int i = i0 + 16 * u + l16;
                const double *pa = Li + (size_t)(i < r ? i : 0) * r + c;
                const float *pb = Wn + (size_t)(n0 + 16 * u + l16) * r + c;
                if constexpr (VEC) {
                    const bool in = c < c_end;  // (whole quads)
                    const fz_f64x2_t lo = in && i < r ? *reinterpret_cast<const fz_f64x2_t *>(pa) : fz_f64x2_t{0.0, 0.0};
                    const fz_f64x2_t hi = in && i < r ? *reinterpret_cast<const fz_f64x2_t *>(pa + 2) : fz_f64x2_t{0.0, 0.0};
                    const fz_f32x4_t v = in ? *reinterpret_cast<const fz_f32x4_t *>(pb) : fz_f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
                    x.a[u][0] = lo[0], x.a[u][1] = lo[1], x.a[u][2] = hi[0], x.a[u][3] = hi[1];
#pragma unroll
                    for (int q = 0; q < 4; ++q) x.b[u][q] = v[q];
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        x.a[u][q] = c + q < c_end && i < r ? pa[q] : 0.0;
                        x.b[u][q] = c + q < c_end ? pb[q] : 0.0f;
                    }
                }
            }
        };
        fz_f64x4_t acc[2][2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v) acc[u][v] = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
        auto multiply = [&](const Step &x) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 2; ++v)
                        acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a[u][q], (double)x.b[v][q], acc[u][v], 0, 0, 0);
        };
        Step s0, s1;
        fetch(s0, 0);
        fetch(s1, steps > 1 ? 1 : 0);
        for (int step = 0; step < steps; step += 2) {
            multiply(s0);
            if (step + 2 < steps) fetch(s0, step + 2);
            if (step + 1 < steps) multiply(s1);
            if (step + 3 < steps) fetch(s1, step + 3);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 2; ++v)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = i0 + 16 * u + kk + 4 * e;
                    if (i < r) Vt[(size_t)i * n + n0 + 16 * v + l16] = (float)acc[u][v][e];
                }
    }
}

// ------------------------------------------------------------------------------------------------
// (5) Rotation to singular vectors (Sec. 3.1 Eq. 1: A = U Sigma, B = V^T).  The iteration leaves an orthonormal basis
// V of the dominant subspace; within it the Rayleigh-Ritz matrix M = V C V^T (= A^T A for A = X_cat V^T) is
// diagonalised, M = R Lambda R^T, and V is replaced by R^T V with the eigenvalues in descending order, after which
// A^T A = Lambda is diagonal and descending and any leading block of rows of B spans the best subspace of that size
// that the basis contains.  M is r x r, symmetric positive semi-definite, fp64.
//
// Eigen-solver: two-sided Jacobi in blocks.  Plane rotations T make M' = T M T^T more and more diagonal; their product
// is J^T (stored as such: row c = eigenvector c in the basis V), the diagonal ends as the eigenvalues.  The r columns
// are cut into blocks of 16; a round of a round-robin tournament between blocks rotates, for every pair of blocks,
// every pair of columns between the two blocks once (in a sweep's first round also the pairs inside each block), so that
// every pair of columns meets exactly once per sweep.  The rotations of a pair of blocks depend on its 32 x 32 diagonal
// block of M alone; applying them is two 32 x 32 x 32 products per block of M and one per block of J^T.  A round is one
// launch: it applies its rotations and finds those of the next round, for which each pair of blocks brings its diagonal
// block up to date by itself.  Launch boundaries are the only synchronisation.
// What bounds it: the chain of launches, and in a launch the 16 dependent inner rounds of the rotations.  One launch takes
// 12.4 us (r = 512; 5.2 us the inner rounds, 1.6 us one that returns at once), eight sweeps run: 3.25 ms.  The rest is instructions of one
// wavefront per SIMD, so there are few of them: no division in the tournament's schedule, 16-byte requests, and no bounds checks where
// every block lies inside the matrix (15.8 -> 13.2 us); and no compute unit of a finding workgroup is shared while 256 are
// enough (J^T in 128 instead of 64 positions: 216 workgroups instead of 280 at r = 512, 12.9 -> 12.4 us).  One-sided Jacobi on whole columns of 512, three dot
// products of columns per rotation, took 63 us per launch; every workgroup finding the rotations
// of its own two pairs 16 us with one sequence, but all 200 workgroups of a sequence then hold a compute unit for the 16
// inner rounds; two launches per round 18 us.
// The launches of kJacobiSweeps sweeps are all enqueued up front (no value is read back by the host); a sequence is
// finished early on the device: every sweep counts, per sequence, the rotations whose element alpha was above
// kJacobiSettled sqrt(beta gamma), and the workgroups of the sweeps after one with a count of zero return at once.  Convergence is
// quadratic by then: what a sweep without such a rotation leaves behind is of the order of the square of that bound.
// ------------------------------------------------------------------------------------------------

// (4z) Vn[c][i] = Vt[i][c]: the basis in the layout in which the fp64 products read it.
__global__ __launch_bounds__(256) void transpose_v_kernel(const float *__restrict__ Vt, float *__restrict__ Vn, long long vn_seq, int n,
                                                          int r)
{
    __shared__ float tile[32][33];
    Vt += (size_t)blockIdx.z * r * n;
    Vn += (size_t)blockIdx.z * vn_seq;
    const int c0 = blockIdx.x * 32, i0 = blockIdx.y * 32, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int i = i0 + ty + 8 * u, c = c0 + tx;
        tile[ty + 8 * u][tx] = (i < r && c < n) ? Vt[(size_t)i * n + c] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int c = c0 + ty + 8 * u, i = i0 + tx;
        if (c < n && i < r) Vn[(size_t)c * r + i] = tile[tx][ty + 8 * u];
    }
}

constexpr int kJacobiSweeps = 10;        // most sweeps of the block Jacobi eigen-solver (each: every pair of column blocks once)
constexpr double kJacobiSettled = 1e-7;  // a sweep whose elements all stayed below this cosine was the last one needed

// (5b) M = (S + S^T) / 2 with S the sum of its planes, Jt = identity, rotation counts zero.  A workgroup makes a block of 32 x 32 and its
// mirror image, so that the transposed one is read in rows too (r = 512, 16 planes: 36 -> 12 us).
__global__ __launch_bounds__(256) void jacobi_init_kernel(const double *__restrict__ planes, double *__restrict__ M,
                                                          double *__restrict__ Jt, int *__restrict__ rotations, int r,
                                                          int splits)
{
    if (blockIdx.x == 0 && threadIdx.x < kJacobiSweeps) rotations[blockIdx.z * kJacobiSweeps + threadIdx.x] = 0;
    planes += (size_t)blockIdx.z * splits * r * r;
    M += (size_t)blockIdx.z * r * r;
    Jt += (size_t)blockIdx.z * r * r;
    // block (bi, bj), bi >= bj, of 32 x 32 and its mirror image
    __shared__ double low[32][33], up[32][33];
    int bi, bj;
    fz_lower_pair((int)blockIdx.x, bi, bj);
    const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    double x[4] = {}, y[4] = {};
    for (int s = 0; s < splits; ++s) {
        const double *p = planes + (size_t)s * r * r;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = r0 + 8 * u;
            x[u] += (32 * bi + k < r && 32 * bj + c < r) ? p[(size_t)(32 * bi + k) * r + 32 * bj + c] : 0.0;
            y[u] += (32 * bj + k < r && 32 * bi + c < r) ? p[(size_t)(32 * bj + k) * r + 32 * bi + c] : 0.0;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        low[r0 + 8 * u][c] = x[u];
        up[r0 + 8 * u][c] = y[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int k = r0 + 8 * u, i = 32 * bi + k, j = 32 * bj + c, it = 32 * bj + k, jt = 32 * bi + c;
        if (i < r && j < r) {
            M[(size_t)i * r + j] = 0.5 * (x[u] + up[c][k]);
            Jt[(size_t)i * r + j] = i == j ? 1.0 : 0.0;
        }
        if (bi != bj && it < r && jt < r) {
            M[(size_t)it * r + jt] = 0.5 * (low[c][k] + y[u]);
            Jt[(size_t)it * r + jt] = 0.0;
        }
    }
}

// The value of the next lane of the same 16 (the last lane takes the first one's).
__device__ __forceinline__ double fz_next_of_16(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x12F, 0xF, 0xF, false);  // row_ror:15
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x12F, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double fz_from_lane(double v, int l)
{
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(4 * l, __double2hiint(v)), __builtin_amdgcn_ds_bpermute(4 * l, __double2loint(v)));
}

// The rotation that makes [[beta, alpha], [alpha, gamma]] diagonal: new a = cs a - sn b, new b = sn a + cs b, |angle| <=
// 45 degrees.  cos 2t = |gamma - beta| / h, sin 2t = +-2 alpha / h, then the half angle; two reciprocal square roots and
// no division.  An element that is zero to working accuracy stays as it is.
__device__ __forceinline__ void fz_rotation(double alpha, double beta, double gamma, double &cs, double &sn)
{
    const double dif = gamma - beta, a2 = 2.0 * alpha;
    const double rh = fz_rsqrt(fma(dif, dif, a2 * a2));
    const double u = fma(0.5 * fabs(dif), rh, 0.5), rc = fz_rsqrt(u);
    const bool on = alpha * alpha > 1e-30 * fabs(beta * gamma);
    cs = on ? u * rc : 1.0;
    sn = on ? (dif >= 0.0 ? alpha : -alpha) * rh * rc : 0.0;
}

// (5c) round k of the tournament: M' = T M T^T and J^T' = T J^T with the rotations T that the launch before found, and
// beside them the rotations of round k + 1.  Workgroups x < pairs find rotations; the next pairs (pairs + 1) / 2 make block
// (p, q), p >= q, of M' and its mirror image, in the other buffer; the others the rows of J^T of one pair, 128 positions.
// The first launch, k = -1, only finds the rotations of round 0.
constexpr int kJacNC = 32, kJacBS = 16, kJacLP = 34, kJacTile = kJacNC * kJacLP;
constexpr int kJacLds = 2 * kJacTile + 2 * 256 * 2 + 2 * 16 * 4;  // doubles

// Row `row` of M in the columns of a pair of blocks, in that order; FULL: every block lies inside the matrix, otherwise zeros beyond it.
template <bool FULL>
__device__ __forceinline__ void fz_jac_m_row(const double *M, int row, const int (&b)[2], int kk, int r, double (&v)[8])
{
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int col = b[h >> 1] + 4 * kk + 2 * (h & 1);
        if constexpr (FULL) {
            const fz_f64x2_t t = *reinterpret_cast<const fz_f64x2_t *>(M + (size_t)row * r + col);
            v[2 * h] = t[0];
            v[2 * h + 1] = t[1];
        } else {
            v[2 * h] = (row < r && col < r) ? M[(size_t)row * r + col] : 0.0;
            v[2 * h + 1] = (row < r && col + 1 < r) ? M[(size_t)row * r + col + 1] : 0.0;
        }
    }
}

// First columns of the two blocks of pair number x in round t, 0 <= t < m - 1, of the round-robin tournament of m = n_blocks players:
// the last player meets t, and t + x meets t - x modulo m - 1.
__device__ __forceinline__ void fz_pair_of_blocks(int x, int t, int n_blocks, int (&b)[2])
{
    const int m1 = n_blocks - 1, u = t + x >= m1 ? t + x - m1 : t + x, v = x == 0 ? m1 : t < x ? t - x + m1 : t - x;
    b[0] = (u < v ? u : v) * kJacBS;
    b[1] = (u < v ? v : u) * kJacBS;
}

__device__ __forceinline__ int fz_pair_column(const int (&b)[2], int c) { return (c < kJacBS ? b[0] : b[1]) + (c & 15); }

// Which pair of round t a block is in, and as which half (inverse of fz_pair_of_blocks).
__device__ __forceinline__ void fz_pair_of_block(int b, int t, int n_blocks, int &x, int &half)
{
    const int m1 = n_blocks - 1;
    int other;
    if (b == m1 || b == t) {
        x = 0;
        other = b == t ? m1 : t;
    } else {
        const int up = b < t ? b - t + m1 : b - t, o = 2 * t - b;  // -m1 < o < 2 m1
        x = up < m1 - up ? up : m1 - up;
        other = o < 0 ? o + m1 : o >= m1 ? o - m1 : o;
    }
    half = b > other ? 1 : 0;
}

// The rotations of pair of blocks x in round `round`, from its 32 x 32 diagonal block of M' (M as it is where T_old is null,
// otherwise the three 16 x 16 blocks of T_old M T_old^T that make it up).
// Thread = one 2 x 2 block of pairs, rows x columns.  The 16 x 16 rotations between the two halves, inner round t:
// a = w meets b = 16 + (w + t) % 16.  A thread keeps the elements of its pairs in registers; from one inner round to the
// next the b side moves on by one pair, along the columns with a lane permutation, along the rows through LDS.  One
// barrier per inner round.  Rows and columns beyond the matrix are zero and are not rotated.
template <bool FULL>
__device__ __forceinline__ void fz_find_rotations(const double *__restrict__ M, const double *T_old, double *T, int *count, int r,
                                                  int n_blocks, int round, int x, double *sm)
{
    // LDS: the diagonal block; T in the sweep's first round, the elements on the move and alpha, beta, gamma of the next
    // inner round's pairs -- before any of these the intermediate of the three parts
    double *G = sm, *Ts = sm + kJacTile;
    auto mv = reinterpret_cast<fz_f64x2_t (*)[16][16]>(Ts + kJacTile);  // [2]
    auto dg = reinterpret_cast<double (*)[16][4]>(Ts + kJacTile + 2 * 256 * 2);  // [2]
    __shared__ int big_rotations;
    T += (size_t)x * kJacNC * kJacNC;  // row c = coefficients of new column c in the old ones
    const int tid = threadIdx.x, lane = lane_id(), pr = tid >> 4, pc = tid & 15;
    int blk[2];
    fz_pair_of_blocks(x, round, n_blocks, blk);
    if (T_old) {
        constexpr int KS = kJacNC / 4, YP = 18;
        auto Y = reinterpret_cast<double (*)[kJacNC * YP]>(Ts);  // [3]
        static_assert(3 * kJacNC * YP <= kJacLds - kJacTile, "in the place of what comes later");
        const int w = wave_id(), l16 = lane & 15, kk = lane >> 4, before = round == 0 ? n_blocks - 2 : round - 1;
        int px[2], half[2], pb[2][2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            fz_pair_of_block(blk[h] / kJacBS, before, n_blocks, px[h], half[h]);
            fz_pair_of_blocks(px[h], before, n_blocks, pb[h]);
        }
        // parts 0, 1, 2 = (a, c) = (0, 0), (1, 1), (0, 1)
        double ma[2][KS], tc[2][KS], ta0[KS];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int item = w + 4 * u, part = item >> 1, mt = item & 1, a = part == 1 ? 1 : 0, c = part == 0 ? 0 : 1;
            const int row = (mt ? (a ? pb[1][1] : pb[0][1]) : (a ? pb[1][0] : pb[0][0])) + l16;
            const double *Tc = T_old + (size_t)(c ? px[1] : px[0]) * kJacNC * kJacNC + (16 * (c ? half[1] : half[0]) + l16) * kJacNC;
            const int pbc[2] = {c ? pb[1][0] : pb[0][0], c ? pb[1][1] : pb[0][1]};
            if (u == 0 || w < 2) {
                fz_jac_m_row<FULL>(M, row, pbc, kk, r, ma[u]);
                fz_run_row(Tc, kk, tc[u]);
            }
        }
        const int sa = w == 1 ? 1 : 0, sc0 = w == 0 ? 0 : 1;  // wavefronts 0 .. 2: the part they finish
        const double *Ta = T_old + (size_t)(sa ? px[1] : px[0]) * kJacNC * kJacNC + (16 * (sa ? half[1] : half[0]) + l16) * kJacNC;
        fz_run_row(Ta, kk, ta0);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int item = w + 4 * u;
            if (item < 6) {
                fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ma[u][ks], tc[u][ks], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) Y[item >> 1][(16 * (item & 1) + kk + 4 * v) * YP + l16] = acc[v];
            }
        }
        lds_barrier();
        if (w < 3) {
            fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ta0[ks], Y[w][fz_run_k(ks, kk) * YP + l16], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                G[(16 * sa + kk + 4 * v) * kJacLP + 16 * sc0 + l16] = acc[v];
                if (w == 2) G[(16 + l16) * kJacLP + kk + 4 * v] = acc[v];
            }
        }
    } else {
        const int lj = tid & 31, li = tid >> 5, cj = fz_pair_column(blk, lj);
        double g[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ri = fz_pair_column(blk, li + 8 * u);
            g[u] = FULL || (ri < r && cj < r) ? M[(size_t)ri * r + cj] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) G[(li + 8 * u) * kJacLP + lj] = g[u];
    }
    if (tid == 0) big_rotations = 0;
    lds_barrier();

    int big = 0;
    auto note = [&](double al, double be, double ga) __attribute__((always_inline)) {
        if (pr == pc && al * al > kJacobiSettled * kJacobiSettled * fabs(be * ga)) ++big;
    };
    double ta[2], tb[2];  // rows a, b of pair pc of T, columns 2 pr and 2 pr + 1
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        ta[u] = pc == 2 * pr + u ? 1.0 : 0.0;
        tb[u] = 16 + pc == 2 * pr + u ? 1.0 : 0.0;
    }
    if (round == 0) {
        // once per sweep, every block being in exactly one pair of the round: the pairs inside the two blocks, as halves
        // of 8, then of 4, 2 and 1 that meet each other
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            Ts[pc * kJacLP + 2 * pr + u] = ta[u];
            Ts[(16 + pc) * kJacLP + 2 * pr + u] = tb[u];
        }
        for (int h = 8; h >= 1; h >>= 1)
            for (int t = 0; t < h; ++t) {
                const int ar = pr / h * 2 * h + pr % h, br = pr / h * 2 * h + h + (pr + t) % h;
                const int ac = pc / h * 2 * h + pc % h, bc = pc / h * 2 * h + h + (pc + t) % h;
                lds_barrier();
                double cc, sc;
                fz_rotation(G[ac * kJacLP + bc], G[ac * kJacLP + ac], G[bc * kJacLP + bc], cc, sc);
                const double cr = fz_from_lane(cc, (lane & 48) | pr), sr = fz_from_lane(sc, (lane & 48) | pr);
                note(G[ac * kJacLP + bc], G[ac * kJacLP + ac], G[bc * kJacLP + bc]);
                const double aa = G[ar * kJacLP + ac], ab = G[ar * kJacLP + bc], ba = G[br * kJacLP + ac], bb = G[br * kJacLP + bc];
                const double x0 = cr * aa - sr * ba, x1 = cr * ab - sr * bb, y0 = sr * aa + cr * ba, y1 = sr * ab + cr * bb;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const double x = Ts[ac * kJacLP + 2 * pr + u], y = Ts[bc * kJacLP + 2 * pr + u];
                    Ts[ac * kJacLP + 2 * pr + u] = cc * x - sc * y;
                    Ts[bc * kJacLP + 2 * pr + u] = sc * x + cc * y;
                }
                lds_barrier();
                G[ar * kJacLP + ac] = cc * x0 - sc * x1;
                G[ar * kJacLP + bc] = pr == pc ? 0.0 : sc * x0 + cc * x1;
                G[br * kJacLP + ac] = pr == pc ? 0.0 : cc * y0 - sc * y1;
                G[br * kJacLP + bc] = sc * y0 + cc * y1;
            }
        lds_barrier();
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            ta[u] = Ts[pc * kJacLP + 2 * pr + u];
            tb[u] = Ts[(16 + pc) * kJacLP + 2 * pr + u];
        }
    }
    double aa = G[pr * kJacLP + pc], ab = G[pr * kJacLP + 16 + pc], ba = G[(16 + pr) * kJacLP + pc], bb = G[(16 + pr) * kJacLP + 16 + pc];
    double al = G[pc * kJacLP + 16 + pc], be = G[pc * kJacLP + pc], ga = G[(16 + pc) * kJacLP + 16 + pc];
    for (int t = 0; t < kJacBS; ++t) {
        const int par = t & 1;
        double cc, sc;
        fz_rotation(al, be, ga, cc, sc);
        // (every 16 lanes compute the rotations of all pairs, for their columns; the one of their row is among them)
        const double cr = fz_from_lane(cc, (lane & 48) | pr), sr = fz_from_lane(sc, (lane & 48) | pr);
        note(al, be, ga);
        const double x0 = cc * aa - sc * ab, x1 = sc * aa + cc * ab, y0 = cc * ba - sc * bb, y1 = sc * ba + cc * bb;
        aa = cr * x0 - sr * y0;
        ab = fz_next_of_16(pr == pc ? 0.0 : cr * x1 - sr * y1);
        ba = pr == pc ? 0.0 : sr * x0 + cr * y0;
        bb = fz_next_of_16(sr * x1 + cr * y1);
        mv[par][pr][pc] = fz_f64x2_t{ba, bb};
        if (pr == pc) *reinterpret_cast<fz_f64x2_t *>(dg[par][pc]) = fz_f64x2_t{ab, aa};
        if (pr == ((pc + 1) & 15)) dg[par][pc][2] = bb;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const double x = ta[u], y = tb[u];
            ta[u] = cc * x - sc * y;
            tb[u] = fz_next_of_16(sc * x + cc * y);
        }
        lds_barrier();
        const fz_f64x2_t m = mv[par][(pr + 1) & 15][pc], c2 = *reinterpret_cast<const fz_f64x2_t *>(dg[par][pc]);
        ba = m[0];
        bb = m[1];
        al = c2[0];
        be = c2[1];
        ga = dg[par][pc][2];
    }
    *reinterpret_cast<fz_f64x2_t *>(T + pc * kJacNC + 2 * pr) = fz_f64x2_t{ta[0], ta[1]};
    *reinterpret_cast<fz_f64x2_t *>(T + (16 + pc) * kJacNC + 2 * pr) = fz_f64x2_t{tb[0], tb[1]};
    if (big > 0) atomicAdd(&big_rotations, big);
    lds_barrier();
    if (tid == 0 && big_rotations > 0) atomicAdd(count, big_rotations);
}

template <bool FULL>
__global__ __launch_bounds__(256) void jacobi_round_kernel(const double *__restrict__ Ma, double *__restrict__ Mb,
                                                           double *__restrict__ Jt, const double *__restrict__ T,
                                                           double *__restrict__ T_next, long long t_seq, int *rotations, int r,
                                                           int n_blocks, int sweep, int round)
{
    // rotations[sequence][sweep]: written by the workgroups that find the rotations of that sweep; final before a launch
    // that applies the sweep's last ones, and a sweep without any ends the work of all later launches
    rotations += blockIdx.z * kJacobiSweeps;
    Ma += (size_t)blockIdx.z * r * r;
    T += (size_t)blockIdx.z * t_seq;
    __shared__ __attribute__((aligned(16))) double sm[kJacLds];  // both kinds of workgroups: several share a compute unit
    const int n_pairs = n_blocks / 2, n_tri = n_pairs * (n_pairs + 1) / 2, m1 = n_blocks - 1;
    int x = (int)blockIdx.x;
    if (x < n_pairs) {
        const bool next = round + 1 == m1;
        const int s = sweep + next;
        if (s == kJacobiSweeps || (s > 0 && rotations[s - 1] == 0)) return;  // same for the whole workgroup
        fz_find_rotations<FULL>(Ma, round < 0 ? nullptr : T, T_next + (size_t)blockIdx.z * t_seq, rotations + s, r, n_blocks,
                                next ? 0 : round + 1, x, sm);
        return;
    }
    x -= n_pairs;
    if (sweep > 0 && rotations[sweep - 1] == 0) return;
    double *Y = sm;
    Mb += (size_t)blockIdx.z * r * r;
    Jt += (size_t)blockIdx.z * r * r;
    constexpr int KS = kJacNC / 4;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id(), l16 = lane & 15, kk = lane >> 4;
    if (x >= n_tri) {  // wavefront = two times 16 positions
        const int p = (x - n_tri) % n_pairs, i0 = (x - n_tri) / n_pairs * 128 + 32 * w + l16;
        int blk[2];
        fz_pair_of_blocks(p, round, n_blocks, blk);
        const double *Tp = T + (size_t)p * kJacNC * kJacNC;
        double tv[2][KS], ta[2][KS];
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const int c = fz_pair_column(blk, fz_run_k(ks, kk)), i = i0 + 16 * g;
                tv[g][ks] = (FULL || c < r) && i < r ? Jt[(size_t)c * r + i] : 0.0;
            }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt) fz_run_row(Tp + (16 * mt + l16) * kJacNC, kk, ta[mt]);
#pragma unroll
        for (int g = 0; g < 2; ++g)
#pragma unroll
            for (int mt = 0; mt < 2; ++mt) {
                fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(ta[mt][ks], tv[g][ks], acc, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int c = fz_pair_column(blk, 16 * mt + kk + 4 * v), i = i0 + 16 * g;
                    if ((FULL || c < r) && i < r) Jt[(size_t)c * r + i] = acc[v];
                }
            }
        return;
    }
    int p, q, bp[2], bq[2];
    fz_lower_pair(x, p, q);
    fz_pair_of_blocks(p, round, n_blocks, bp);
    fz_pair_of_blocks(q, round, n_blocks, bq);
    const double *Tp = T + (size_t)p * kJacNC * kJacNC, *Tq = T + (size_t)q * kJacNC * kJacNC;
    const int mt = w >> 1, nt = w & 1;  // wavefront = one tile of 16 x 16
    double xa[KS], tq[KS], tp[KS];
    fz_jac_m_row<FULL>(Ma, bp[mt] + l16, bq, kk, r, xa);
    fz_run_row(Tq + (16 * nt + l16) * kJacNC, kk, tq);
    fz_run_row(Tp + (16 * mt + l16) * kJacNC, kk, tp);
    fz_f64x4_t acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[ks], tq[ks], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) Y[(16 * mt + kk + 4 * v) * kJacLP + 16 * nt + l16] = acc[v];
    __syncthreads();
    acc = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(tp[ks], Y[fz_run_k(ks, kk) * kJacLP + 16 * nt + l16], acc, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v) Y[(16 * mt + kk + 4 * v) * kJacLP + 16 * nt + l16] = acc[v];
    __syncthreads();
    const int j = 2 * l16, li = tid >> 4;
#pragma unroll
    for (int u = 0; u < 2; ++u) {  // rows li + 16 u, columns j and j + 1; M' stays symmetric to the last bit
        const int i = li + 16 * u, ra = bp[u] + li, cb = fz_pair_column(bq, j), rb = bq[u] + li, ca = fz_pair_column(bp, j);
        const double v0 = p == q && i > j ? Y[j * kJacLP + i] : Y[i * kJacLP + j];
        const double v1 = p == q && i > j + 1 ? Y[(j + 1) * kJacLP + i] : Y[i * kJacLP + j + 1];
        if constexpr (FULL) {
            *reinterpret_cast<fz_f64x2_t *>(Mb + (size_t)ra * r + cb) = fz_f64x2_t{v0, v1};
            if (p != q) *reinterpret_cast<fz_f64x2_t *>(Mb + (size_t)rb * r + ca) = fz_f64x2_t{Y[j * kJacLP + i], Y[(j + 1) * kJacLP + i]};
        } else {
            if (ra < r && cb < r) Mb[(size_t)ra * r + cb] = v0;
            if (ra < r && cb + 1 < r) Mb[(size_t)ra * r + cb + 1] = v1;
            if (p != q && rb < r && ca < r) Mb[(size_t)rb * r + ca] = Y[j * kJacLP + i];
            if (p != q && rb < r && ca + 1 < r) Mb[(size_t)rb * r + ca + 1] = Y[(j + 1) * kJacLP + i];
        }
    }
}

// (5d) eigenvalues = |diagonal| of the rotated matrix; order[k] = the column with the k-th largest one (ties: smaller
// index); sigma (nullable) receives the singular values sqrt(lambda) of the leading r_out, in that order.  A sweep is an
// odd number of rounds, each from one buffer to the other, so the matrix lies in Mb after an odd number of sweeps.
__global__ __launch_bounds__(1024) void ritz_order_kernel(const double *__restrict__ Ma, const double *__restrict__ Mb,
                                                          const int *__restrict__ rotations, int *__restrict__ order,
                                                          float *__restrict__ sigma, int r, int r_out)
{
    __shared__ double lam[1024];
    rotations += blockIdx.x * kJacobiSweeps;
    int sweeps = 1;
    while (sweeps < kJacobiSweeps && rotations[sweeps - 1] != 0) ++sweeps;
    const double *M = (sweeps & 1 ? Mb : Ma) + (size_t)blockIdx.x * r * r;
    order += (size_t)blockIdx.x * r;
    const int c = threadIdx.x;
    if (c < r) {
        // (a NaN would compare as neither larger nor equal and leave places of `order` unwritten: it goes last)
        const double v = fabs(M[(size_t)c * r + c]);
        lam[c] = v >= 0.0 ? v : -1.0;
    }
    __syncthreads();
    if (c < r) {
        int rank = 0;
        const double mine = lam[c];
        for (int j = 0; j < r; ++j) rank += (lam[j] > mine || (lam[j] == mine && j < c)) ? 1 : 0;
        order[rank] = c;
        if (sigma && rank < r_out) sigma[(size_t)blockIdx.x * r_out + rank] = (float)sqrt(mine);  // (NaN for the -1)
    }
}

// (5e) the leading r_out rotated basis vectors: Vr[k][c] = sum_j Jt[order[k]][j] Vt[j][c] on the fp64 matrix cores.
// Wavefront = 32 k x 64 positions c, eight products per four j; four steps at a time, their operands requested before the
// products of the four before.  The matrix cores bound it (27 us at r = 512, n = 4096); 69 us, thread = position with vector multiply-adds
// 170 us.
__device__ __forceinline__ void fz_rotate_fetch(double (&ja)[4][2], float (&vb)[4][4], const double *const (&jrow)[2],
                                                const float *__restrict__ Vt, int j0, int r, int n, const int (&cc)[4], int kk)
{
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int j = j0 + 4 * s + kk;
        const bool ok = j < r;
        const int jj = ok ? j : 0;
#pragma unroll
        for (int u = 0; u < 2; ++u) ja[s][u] = ok ? jrow[u][jj] : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) vb[s][v] = Vt[(size_t)jj * n + cc[v]];
    }
}

__global__ __launch_bounds__(256) void rotate_basis_kernel(const double *__restrict__ Jt, const int *__restrict__ order,
                                                           const float *__restrict__ Vt, float *__restrict__ Vr, int n,
                                                           int r, int r_out, long long vr_seq)
{
    Jt += (size_t)blockIdx.z * r * r;
    order += (size_t)blockIdx.z * r;
    Vt += (size_t)blockIdx.z * r * n;
    Vr += (size_t)blockIdx.z * vr_seq;
    const int lane = lane_id(), l16 = lane & 15, kk = lane >> 4, c0 = (blockIdx.x * 4 + wave_id()) * 64, k0 = blockIdx.y * 32;
    if (c0 >= n) return;
    const double *jrow[2];
    int cc[4];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int k = k0 + 16 * u + l16;
        jrow[u] = Jt + (size_t)order[k < r_out ? k : r_out - 1] * r;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) cc[v] = c0 + 16 * v + l16 < n ? c0 + 16 * v + l16 : n - 1;
    fz_f64x4_t acc[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[u][v] = fz_f64x4_t{0.0, 0.0, 0.0, 0.0};
    double ja[4][2];
    float vb[4][4];
    fz_rotate_fetch(ja, vb, jrow, Vt, 0, r, n, cc, kk);
    for (int j0 = 0; j0 < r; j0 += 16) {
        double a[4][2], b[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int u = 0; u < 2; ++u) a[s][u] = ja[s][u];
#pragma unroll
            for (int v = 0; v < 4; ++v) b[s][v] = (double)vb[s][v];
        }
        if (j0 + 16 < r) fz_rotate_fetch(ja, vb, jrow, Vt, j0 + 16, r, n, cc, kk);
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s][u], b[s][v], acc[u][v], 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = k0 + 16 * u + kk + 4 * e;
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (k < r_out && c0 + 16 * v + l16 < n) Vr[(size_t)k * n + c0 + 16 * v + l16] = (float)acc[u][v][e];
        }
}

// (4a) B_out[l][i][c] = Vt[i][l * d + c] in the storage type.
template <typename T>
__global__ __launch_bounds__(256) void write_b_kernel(const float *__restrict__ Vt, long long vt_seq, T *__restrict__ B,
                                                      int G, int r, int d)
{
    Vt += (size_t)blockIdx.z * vt_seq;
    B += (size_t)blockIdx.z * G * r * d;
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)G * r * d) return;
    const int c = (int)(idx % d), i = (int)((idx / d) % r), l = (int)(idx / ((long long)d * r));
    B[idx] = from_f32<T>(Vt[(size_t)i * ((size_t)G * d) + (size_t)l * d + c]);
}

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Sequences are processed `bc` at a time (grid dimension z of every kernel), which is what keeps the many small
// launches of the orthonormalisation busy; the workspace holds the intermediates of one such chunk.
constexpr int kFzChunk = 16;

struct FzLayout {
    int n, Lp, bc, gram_tiles, gram_splits, w_splits, g_splits;
    size_t esz, xt_seq, part_seq, off_xt, off_part, off_c, off_vt, off_wn, off_g, off_lt, off_planes, off_diag, off_order,
        off_rot, total;
};

// Of at most `most` splits of `tiles` output tiles the number with which the rounds of 256 workgroups take least, in shares of a tile:
// ceil(tiles splits / 256) / splits (136 tiles: 2 / 3 with three, 3 / 4 with four).  Fewer, where that is the same: less to add up.
int gram_splits_of(int tiles, int most)
{
    int best = 1;
    for (int s = 2; s <= most; ++s)
        if ((tiles * s + 255) / 256 * best < (tiles * best + 255) / 256 * s) best = s;
    return best;
}

// The same for the fp64 Gram matrix, whose workgroups share a compute unit: at least half of the splits, the more where it is the same.
// (r = 512, n = 4096: 34 workgroups in 16 splits are three on 32 of the compute units, in 15 two on every one: 44.8 -> 36.8 us.)
int g_splits_of(int workgroups, int most)
{
    int best = most;
    for (int s = most - 1; 2 * s >= most && s > 0; --s)
        if ((workgroups * s + 255) / 256 * best < (workgroups * best + 255) / 256 * s) best = s;
    return best;
}

FzLayout fz_layout(const xkv_shape &s, int r)
{
    FzLayout f{};
    f.esz = s.dtype == XKV_F32 ? 4 : 2;
    f.n = s.G * s.H_kv * s.d_h;
    f.Lp = (s.L + 63) / 64 * 64;
    // a row pitch that is a multiple of 4 KiB would put the same piece of every row of a tile on the same cache
    // channel; 64 more (zero) tokens move consecutive rows one 128 B line apart
    if (((size_t)f.Lp * f.esz) % 4096 == 0) f.Lp += 64;
    f.bc = std::max(1, std::min(s.batch, kFzChunk));
    const int t = (f.n + kGemmTile - 1) / kGemmTile;
    f.gram_tiles = t * (t + 1) / 2;
    const int slab = 128 / (int)f.esz, gram_slabs = f.Lp / slab;
    auto splits_for = [&](int wgs_per_seq, int target, int most) {  // enough workgroups to fill the chip twice over
        const int wgs = wgs_per_seq * f.bc;
        return std::max(1, std::min(std::min(16, most), (target + wgs - 1) / wgs));
    };
    f.gram_splits = splits_for(f.gram_tiles, 512, gram_slabs);
    f.w_splits = splits_for(t * ((r + kGemmTile - 1) / kGemmTile), 256, f.n / 32);
    const int gb = (r + 31) / 32;
    f.g_splits = splits_for((gb * (gb + 1) / 2 + 3) / 4, 1024, f.n / 64);
    f.xt_seq = (size_t)f.n * f.Lp;
    f.part_seq = std::max((size_t)f.gram_splits * f.n * f.n, (size_t)f.w_splits * f.n * r);
    const size_t bc = (size_t)f.bc;
    size_t o = 0;
    f.off_xt = o;     o += align256(bc * f.xt_seq * f.esz);
    f.off_part = o;   o += align256(bc * f.part_seq * 4);
    f.off_c = o;      o += align256(bc * f.n * f.n * 4);
    f.off_vt = o;     o += align256(bc * r * f.n * 4);
    f.off_wn = o;     o += align256(bc * f.n * r * 4);
    f.off_g = o;      o += align256(bc * r * r * 8);
    f.off_lt = o;     o += align256(bc * r * r * 8);
    f.off_planes = o; o += align256(bc * f.g_splits * r * r * 8);
    f.off_diag = o;   o += align256(bc * r * 8);
    f.off_order = o;  o += align256(bc * ((r + 15) / 16) * 256 * 8);
    f.off_rot = o;    o += align256(bc * 16 * 4);
    f.total = o;
    return f;
}

template <typename T> hipError_t launch_gemm(const GemmArgs &a, int tiles, int nseq, hipStream_t st)
{
    static DynamicLdsOnce attr;
    if (hipError_t e0 = attr.ensure((const void *)gemm_nt_kernel<T>, kGemmLds); e0 != hipSuccess) return e0;
    GemmArgs b = a;
    b.tiles = tiles;
    const int per_die = (tiles * a.splits + 7) / 8;
    hipLaunchKernelGGL(gemm_nt_kernel<T>, dim3(8 * per_die, 1, nseq), dim3(kGemmThreads), kGemmLds, st, b);
    return hipGetLastError();
}

inline unsigned blocks256(long long count) { return (unsigned)((count + 255) / 256); }

template <typename T>
hipError_t factorize_typed(const xkv_shape &s, const FzLayout &f, const void *X, int r, int r_out, int iters, uint32_t seed,
                           void *A_out, void *B_out, float *sigma_out, unsigned char *ws, hipStream_t st)
{
    const int n = f.n, d = s.H_kv * s.d_h, tn = (n + kGemmTile - 1) / kGemmTile, tr = (r + kGemmTile - 1) / kGemmTile;
    constexpr int E = 128 / (int)sizeof(T);
    T *Xt = reinterpret_cast<T *>(ws + f.off_xt);
    float *part = reinterpret_cast<float *>(ws + f.off_part), *C = reinterpret_cast<float *>(ws + f.off_c);
    float *Vt = reinterpret_cast<float *>(ws + f.off_vt), *Wn = reinterpret_cast<float *>(ws + f.off_wn);
    double *Gm = reinterpret_cast<double *>(ws + f.off_g), *Lt = reinterpret_cast<double *>(ws + f.off_lt);
    double *planes = reinterpret_cast<double *>(ws + f.off_planes), *diag0 = reinterpret_cast<double *>(ws + f.off_diag);
    int *order = reinterpret_cast<int *>(ws + f.off_order);
    int *rotations = reinterpret_cast<int *>(ws + f.off_rot);
    static_assert(kJacobiSweeps <= 16, "the rotation counters have 16 slots per sequence");
    static_assert(kCholLds <= 64 * 1024 - 256, "no raised LDS limit needed");
    hipError_t e = hipSuccess;
    const long long vcount = (long long)r * n, x_seq = (long long)n * s.L;
    for (int b0 = 0; b0 < s.batch && e == hipSuccess; b0 += f.bc) {
        const int nb = std::min(f.bc, s.batch - b0);  // sequences of this chunk
        const T *Xb = reinterpret_cast<const T *>(X) + (size_t)b0 * x_seq;
        hipLaunchKernelGGL(xt_pack_kernel<T>, dim3(f.Lp / 64, n / 64, nb), dim3(256), 0, st, Xb, Xt, s.L, f.Lp, s.d_h, x_seq,
                           (long long)f.xt_seq);
        {  // C = Xt Xt^T
            GemmArgs a{};
            a.P = GemmOperand{Xt, f.Lp, 0, f.Lp, n, (long long)f.xt_seq};
            a.Q = a.P;
            a.n_slabs = f.Lp / E; a.splits = gram_splits_of(f.gram_tiles * nb, f.gram_splits); a.lower_only = 1; a.tiles_n = tn;
            a.out_f32 = part; a.out_bf16 = nullptr; a.ldo = n; a.plane = (long long)n * n; a.out_seq = (long long)f.part_seq;
            profile_begin(3, st);
            e = launch_gemm<T>(a, f.gram_tiles, nb, st);
            profile_end(3, st);
            if (e != hipSuccess) break;
            const int n64 = (n + 63) / 64;
            hipLaunchKernelGGL(gram_finish_kernel, dim3(n64, n64, nb), dim3(256), 0, st, part, C, n, a.splits, a.plane,
                               (long long)f.part_seq);
        }
        hipLaunchKernelGGL(init_v_kernel, dim3(blocks256(vcount), 1, nb), dim3(256), 0, st, Vt, vcount,
                           seed + 0x9E37u * (uint32_t)b0);
        // Vt <- orthonormal basis of the columns of Wn (Cholesky-QR: r x r Gram matrix, inverse of its Cholesky factor, product; fp64)
        auto orthonormalise = [&]() {
            const int gb = (r + 31) / 32, pairs = gb * (gb + 1) / 2, g_splits = g_splits_of((pairs + 3) / 4 * nb, f.g_splits);
            hipLaunchKernelGGL(gram_f64_kernel<true>, dim3((pairs + 3) / 4, g_splits, nb), dim3(256), 0, st, Wn, vcount, Wn,
                               planes, n, r, g_splits, pairs);
            hipLaunchKernelGGL(gram_sum_kernel, dim3((r + 255) / 256, r, nb), dim3(256), 0, st, planes, Gm, diag0, r,
                               g_splits);
            const auto panel_kernel = r % kCholRB == 0 ? chol_panel_kernel<true> : chol_panel_kernel<false>;
            for (int c0 = -kCholRB; c0 < r; c0 += kCholRB) {
                const int blocks = c0 < 0 ? 0 : std::max(0, (r - c0 - 1) / kCholRB);
                const int columns = c0 < 0 ? 0 : std::max(1, blocks) * (c0 / kCholRB + 1);
                hipLaunchKernelGGL(panel_kernel, dim3(1 + blocks * (blocks + 1) / 2 + columns, 1, nb), dim3(kCholThreads), kCholLds, st, Gm,
                                   Lt, diag0, r, c0);
            }
            const dim3 grid((n + 127) / 128, ((r + 31) / 32 + 1) / 2, nb);
            if (r % 4 == 0)
                hipLaunchKernelGGL(orth_apply_kernel<true>, grid, dim3(256), 0, st, Wn, Lt, Vt, n, r);
            else
                hipLaunchKernelGGL(orth_apply_kernel<false>, grid, dim3(256), 0, st, Wn, Lt, Vt, n, r);
        };
        for (int it = 0; it < iters; ++it) {
            GemmArgs a{};  // Wn [n][r] = C Vt^T
            a.P = GemmOperand{C, n, 0, n, n, (long long)n * n};
            a.Q = GemmOperand{Vt, n, 0, n, r, vcount};
            a.n_slabs = n / 32; a.splits = f.w_splits; a.lower_only = 0; a.tiles_n = tr;
            a.out_f32 = f.w_splits > 1 ? part : Wn; a.out_bf16 = nullptr; a.ldo = r; a.plane = vcount;
            a.out_seq = f.w_splits > 1 ? (long long)f.part_seq : vcount;
            if ((e = launch_gemm<float>(a, tn * tr, nb, st)) != hipSuccess) break;
            if (f.w_splits > 1)
                hipLaunchKernelGGL(sum_planes_kernel, dim3(blocks256(vcount), 1, nb), dim3(256), 0, st, part, Wn, vcount,
                                   f.w_splits, vcount, (long long)f.part_seq);
            orthonormalise();
        }
        if (e != hipSuccess) break;
        // Cholesky-QR once more on the basis itself: after the last multiplication by C the weakest directions are
        // orthonormal only to fp32 rounding times the spread of the spectrum; a second pass on a matrix that is already
        // nearly orthonormal brings them to fp32 rounding
        hipLaunchKernelGGL(transpose_v_kernel, dim3((n + 31) / 32, (r + 31) / 32, nb), dim3(256), 0, st, Vt, Wn, vcount, n, r);
        orthonormalise();
        if (e != hipSuccess) break;
        // ---- rotation to singular vectors (5): Wn = C Vt^T once more, M = Vt Wn, eigenvectors of M by block Jacobi
        {
            GemmArgs a{};
            a.P = GemmOperand{C, n, 0, n, n, (long long)n * n};
            a.Q = GemmOperand{Vt, n, 0, n, r, vcount};
            a.n_slabs = n / 32; a.splits = f.w_splits; a.lower_only = 0; a.tiles_n = tr;
            a.out_f32 = f.w_splits > 1 ? part : Wn; a.out_bf16 = nullptr; a.ldo = r; a.plane = vcount;
            a.out_seq = f.w_splits > 1 ? (long long)f.part_seq : vcount;
            if ((e = launch_gemm<float>(a, tn * tr, nb, st)) != hipSuccess) break;
            if (f.w_splits > 1)
                hipLaunchKernelGGL(sum_planes_kernel, dim3(blocks256(vcount), 1, nb), dim3(256), 0, st, part, Wn, vcount,
                                   f.w_splits, vcount, (long long)f.part_seq);
        }
        double *Ma = Gm, *Mb = planes, *Jt = Lt;  // r x r each per sequence
        // the rotations of two rounds, 32 x 32 per pair of blocks, where C (no longer needed) and the transposed basis are: at
        // most (r + 31) / 32 pairs, and n^2 / 2 doubles are 1024 for each of n / 32 pairs or more, n a multiple of 64, n >= r
        const long long tj_seq = (long long)n * n / 2;
        double *Tj[2] = {reinterpret_cast<double *>(part), reinterpret_cast<double *>(C)};
        const int gb = (r + 31) / 32;
        hipLaunchKernelGGL(transpose_v_kernel, dim3((n + 31) / 32, gb, nb), dim3(256), 0, st, Vt, part, (long long)f.part_seq, n, r);
        hipLaunchKernelGGL(gram_f64_kernel<false>, dim3((gb * gb + 3) / 4, f.g_splits, nb), dim3(256), 0, st, part,
                           (long long)f.part_seq, Wn, planes, n, r, f.g_splits, gb * gb);
        hipLaunchKernelGGL(jacobi_init_kernel, dim3(gb * (gb + 1) / 2, 1, nb), dim3(256), 0, st, planes, Ma, Jt,
                           rotations, r, f.g_splits);
        {
            const int n_blocks = std::max(2, ((r + kJacBS - 1) / kJacBS + 1) / 2 * 2);  // an even number of column blocks
            const int n_pairs = n_blocks / 2, grid = n_pairs * (n_pairs + 1) / 2 + n_pairs * ((r + 127) / 128);
            const auto round_kernel = r == n_blocks * kJacBS ? jacobi_round_kernel<true> : jacobi_round_kernel<false>;
            for (int k = -1; k < kJacobiSweeps * (n_blocks - 1); ++k) {
                const bool odd = k & 1;
                const int sweep = k < 0 ? 0 : k / (n_blocks - 1), round = k < 0 ? -1 : k % (n_blocks - 1);
                hipLaunchKernelGGL(round_kernel, dim3(k < 0 ? n_pairs : n_pairs + grid, 1, nb), dim3(256), 0, st,
                                   k >= 0 && odd ? Mb : Ma, odd ? Ma : Mb, Jt, Tj[odd], Tj[!odd], tj_seq, rotations, r, n_blocks, sweep,
                                   round);
            }
        }
        hipLaunchKernelGGL(ritz_order_kernel, dim3(nb), dim3(1024), 0, st, Ma, Mb, rotations, order,
                           sigma_out ? sigma_out + (size_t)b0 * r_out : nullptr, r, r_out);
        float *Vr = Wn;  // [r_out][n] per sequence, in the place of W
        hipLaunchKernelGGL(rotate_basis_kernel, dim3((n + 255) / 256, (r_out + 31) / 32, nb), dim3(256), 0, st, Jt, order, Vt,
                           Vr, n, r, r_out, vcount);
        if ((e = hipGetLastError()) != hipSuccess) break;
        T *Bb = reinterpret_cast<T *>(B_out) + (size_t)b0 * s.G * r_out * d;
        T *Ab = reinterpret_cast<T *>(A_out) + (size_t)b0 * s.L * r_out;
        const long long bcount = (long long)s.G * r_out * d;
        const int tro = (r_out + kGemmTile - 1) / kGemmTile;
        hipLaunchKernelGGL(write_b_kernel<T>, dim3(blocks256(bcount), 1, nb), dim3(256), 0, st, Vr, vcount, Bb, s.G, r_out, d);
        {  // A = X_cat B^T
            GemmArgs a{};
            a.P = GemmOperand{Xb, s.d_h, (long long)s.L * s.d_h, s.d_h, s.L, x_seq};
            a.Q = GemmOperand{Bb, d, (long long)r_out * d, d, r_out, bcount};
            a.n_slabs = n / E; a.splits = 1; a.lower_only = 0; a.tiles_n = tro;
            a.out_f32 = sizeof(T) == 4 ? reinterpret_cast<float *>(Ab) : nullptr;
            a.out_bf16 = sizeof(T) == 2 ? reinterpret_cast<bf16_t *>(Ab) : nullptr;
            a.ldo = r_out; a.plane = 0; a.out_seq = (long long)s.L * r_out;
            e = launch_gemm<T>(a, ((s.L + kGemmTile - 1) / kGemmTile) * tro, nb, st);
        }
        if (e == hipSuccess) e = hipGetLastError();
    }
    return e;
}

}  // namespace

bool factorize_shape_ok(const xkv_shape &s, int r)
{
    const long long n = (long long)s.G * s.H_kv * s.d_h;
    return s.d_h % 64 == 0 && r >= 1 && r <= 1024 && r <= n && n <= 16384;
}

size_t factorize_workspace_bytes(const xkv_shape &s, int r) { return fz_layout(s, r).total; }

hipError_t launch_factorize(const xkv_shape &s, const void *X, int r, int r_out, int iters, uint32_t seed, void *A_out,
                            void *B_out, float *sigma_out, void *ws, hipStream_t st)
{
    const FzLayout f = fz_layout(s, r);
    if (s.dtype == XKV_F32)
        return factorize_typed<float>(s, f, X, r, r_out, iters, seed, A_out, B_out, sigma_out,
                                      reinterpret_cast<unsigned char *>(ws), st);
    return factorize_typed<bf16_t>(s, f, X, r, r_out, iters, seed, A_out, B_out, sigma_out,
                                   reinterpret_cast<unsigned char *>(ws), st);
}

}  // namespace xkv
