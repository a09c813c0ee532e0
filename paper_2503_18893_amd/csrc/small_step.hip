// A whole step of a small problem in one launch, single precision: one workgroup per (sequence, KV head) projects its queries,
// scores its tokens, selects, and attends over the selected rows in the regrouped form (logits from the projected queries,
// U_h = w_h^T A^V[I_g], out_h = U_h B^V_g), with the uncompressed tail, if any, in the same softmax.
//
// Such a step is launches and load latencies: five kernels of 3 to 14 us for 512 tokens of rank 32.  One compute unit reads a mebibyte
// in less than these launches wait, so that is where the line lies (small_step_ok); where it scores and selects longer than the launches for
// that would take, those come first and the rest follows here (small_step_whole).  A layer in a graph, us, five kernels / now: 512 tokens of rank
// 32, 32 selected 31 / 15; 128 selected and a tail of 33 75 / 22; 4096 tokens of rank 48, 1024 selected 67 / 47; 3000 of rank 64, 64
// selected 37 / 29; with 512 pairs of sequence and head 83 / 34, 164 / 50, 940 / 262, 226 / 106 (4096 pairs 385 / 248 for the first).
// The stage call for selected rows takes the second half (WHOLE false) at the same sizes, so that the chained stages and the
// step give the same bits.
#include <type_traits>

#include "row_select.h"

namespace xkv {

constexpr int kSmPart = 8192, kSmRank = 2048, kSmMap = 256;  // words: partial sums, P (once more in double precision) and U, bitmap
constexpr int kSmLists = 2 * kRowWaves * kRowList;           // ... lists, afterwards ids and weights
constexpr int kSmWords = kSmLists + kRowBins + kSmMap + kSmPart + 3 * kSmRank;
// !WHOLE: words of ids and weights, of P or U, and of all; small enough for two workgroups per compute unit in most cases
__host__ __device__ inline int rows_words(int n_rep, int n, int k) { return (k + n_rep * n + 3) / 4 * 4; }
__host__ __device__ inline int rank_words(int n_rep, int r_k, int r_v) { return (n_rep * (r_k > r_v ? r_k : r_v) + 3) / 4 * 4; }

struct SmallArgs {
    const float *A_k, *A_v, *B_k, *B_v, *q, *K_tail, *V_tail;
    float *out, *score_out;
    int32_t *idx_out;
    const int32_t *idx;  // !WHOLE
    int G, layer, L, r_k, r_v, H_kv, H_q, d_h, k, T;
    float scale;
};

// Exchanges on the vector ALU.  swap16(x, y) trades the odd rows (16 lanes) of x for the even rows of y, swap32 the upper half of x
// for the lower half of y; rot<CTRL> moves within a row.
__device__ __forceinline__ void swap16(float &x, float &y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
}

__device__ __forceinline__ void swap32(float &x, float &y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    x = __uint_as_float(r[0]);
    y = __uint_as_float(r[1]);
}

__device__ __forceinline__ void swap16(double &x, double &y)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(y), false, false);
    x = __hiloint2double((int)hi[0], (int)lo[0]);
    y = __hiloint2double((int)hi[1], (int)lo[1]);
}

__device__ __forceinline__ void swap32(double &x, double &y)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(y), false, false);
    x = __hiloint2double((int)hi[0], (int)lo[0]);
    y = __hiloint2double((int)hi[1], (int)lo[1]);
}

template <int CTRL> __device__ __forceinline__ float rot(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xF, 0xF, true));
}

template <int CTRL> __device__ __forceinline__ double rot(double x)
{
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xF, 0xF, true),
                            __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xF, 0xF, true));
}

// Sums of four values over the wavefront: row i of the result holds that of v[i], added up in the order of an exchange with lane ^ 32,
// ^ 16, ... ^ 1.  (A value at a time through LDS, the sixteen wavefronts' exchanges were 5 us of the kernel's 20.)
template <typename V> __device__ __forceinline__ V wave_sum4(V (&v)[4])
{
    swap32(v[0], v[2]);
    swap32(v[1], v[3]);
    V a = v[0] + v[2], b = v[1] + v[3];  // halves: values 0, 2 and 1, 3
    swap16(a, b);
    a += b;
    a += rot<0x128>(a);  // row_ror:8, :4, :2, :1
    a += rot<0x124>(a);
    a += rot<0x122>(a);
    a += rot<0x121>(a);
    return a;
}

// Scaled logits of one row for heads h0 .. h0 + 3 (those beyond nh repeat the first): P [heads][r_k] in LDS.
__device__ __forceinline__ void row_logits(const float *__restrict__ row, const float *P, int r_k, int h0, int nh, bool vec, float scale, float (&z)[4])
{
    const float *Ph[4];
    float acc[4];
#pragma unroll
    for (int hh = 0; hh < 4; ++hh) {
        Ph[hh] = P + (h0 + (hh < nh ? hh : 0)) * r_k;
        acc[hh] = 0.0f;
    }
    if (vec) {
#pragma unroll 8
        for (int i = 0; i < r_k; i += 4) {
            const float4 x = *reinterpret_cast<const float4 *>(row + i);
#pragma unroll
            for (int hh = 0; hh < 4; ++hh) {
                const float4 p = *reinterpret_cast<const float4 *>(Ph[hh] + i);
                acc[hh] = fmaf(x.w, p.w, fmaf(x.z, p.z, fmaf(x.y, p.y, fmaf(x.x, p.x, acc[hh]))));
            }
        }
    } else {
#pragma unroll 8
        for (int i = 0; i < r_k; ++i)
#pragma unroll
            for (int hh = 0; hh < 4; ++hh) acc[hh] = fmaf(row[i], Ph[hh][i], acc[hh]);
    }
#pragma unroll
    for (int hh = 0; hh < 4; ++hh) z[hh] = scale * acc[hh];
}

template <bool WHOLE, int THREADS>
__global__ __launch_bounds__(THREADS) void small_step_kernel(SmallArgs a)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    __shared__ RowShared sh;
    __shared__ float head_den[16];
    const int n_rep = a.H_q / a.H_kv;
    uint32_t *lists = smem, *bins = lists + kSmLists, *map = bins + kRowBins;
    float *part = reinterpret_cast<float *>(WHOLE ? map + kSmMap : lists + rows_words(n_rep, a.k + a.T, a.k)), *P = part + kSmPart;
    double *Pd = reinterpret_cast<double *>(P + (WHOLE ? kSmRank : rank_words(n_rep, a.r_k, a.r_v)));
    const int g = blockIdx.x % a.H_kv, b = blockIdx.x / a.H_kv;
    const int tid = threadIdx.x, lane = lane_id(), w = wave_id();
    constexpr int WAVES = THREADS / kWave;
    static_assert(!WHOLE || THREADS == kRowThreads, "the selection's threads");
    const int L = a.L, r_k = a.r_k, r_v = a.r_v, d_h = a.d_h, d = a.H_kv * d_h, k = a.k, T = a.T;
    const float *A_k = a.A_k + (size_t)b * L * r_k, *A_v = a.A_v + (size_t)b * L * r_v;
    const float *B_k = a.B_k + ((size_t)b * a.G + a.layer) * r_k * d + (size_t)g * d_h;
    const float *B_v = a.B_v + ((size_t)b * a.G + a.layer) * r_v * d + (size_t)g * d_h;
    const float *q = a.q + ((size_t)b * a.H_q + (size_t)g * n_rep) * d_h;
    const float *K_t = T > 0 ? a.K_tail + ((size_t)b * a.H_kv + g) * T * d_h : nullptr, *V_t = T > 0 ? a.V_tail + ((size_t)b * a.H_kv + g) * T * d_h : nullptr;
    [[maybe_unused]] const int words = (L + 63) / 64 * 2;

    if constexpr (WHOLE) {
        bins[2 * tid] = 0;
        bins[2 * tid + 1] = 0;
        for (int i = tid; i < words; i += kRowThreads) map[i] = 0;
    }
    // ---- projected queries, a rank per wavefront at a time, lanes over the head dimension: in single precision with the operations of
    // the score stage, and in double precision for the logits of the selected rows (sums of a few dozen products taken one
    // after the other: the attention was twice as far from the exact one with single-precision logits)
    for (int i = w; i < r_k; i += WAVES)
        for (int h0 = 0; h0 < n_rep; h0 += 4) {
            const int nh = n_rep - h0 < 4 ? n_rep - h0 : 4;
            float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            double accd[4] = {0.0, 0.0, 0.0, 0.0};
            for (int j = lane; j < d_h; j += kWave) {
                const float bv = B_k[(size_t)i * d + j];
#pragma unroll
                for (int hh = 0; hh < 4; ++hh) {
                    const float qv = q[(size_t)(h0 + (hh < nh ? hh : 0)) * d_h + j];
                    if (WHOLE) acc[hh] = fmaf(bv, qv, acc[hh]);
                    accd[hh] = fma((double)bv, (double)qv, accd[hh]);
                }
            }
            const int hh = lane >> 4;
            const double pd = wave_sum4(accd);
            const float pf = WHOLE ? wave_sum4(acc) : 0.0f;
            if ((lane & 15) == 0 && hh < nh) {
                if (WHOLE) P[(h0 + hh) * r_k + i] = pf;
                Pd[(h0 + hh) * r_k + i] = pd;
            }
        }
    __syncthreads();
    const bool vec = r_k % 4 == 0 && ((uintptr_t)A_k & 15u) == 0;
    const int n = k + T;
    int32_t *ids = reinterpret_cast<int32_t *>(lists);
    float *wt = reinterpret_cast<float *>(lists + k);  // [n_rep][k + T]
    if constexpr (WHOLE) {
        // ---- scores, a token per thread; the pooled ones are the wavefront's list
        uint32_t *list = lists + w * 2 * kRowList;
        for (int t0 = 0; t0 < L; t0 += kRowThreads) {
            const int t = t0 + tid, at = t0 / kRowWaves + lane;
            if (t >= L) break;
            float best = -INFINITY;
            for (int h0 = 0; h0 < n_rep; h0 += 4) {
                const int nh = n_rep - h0 < 4 ? n_rep - h0 : 4;
                float z[4];
                row_logits(A_k + (size_t)t * r_k, P, r_k, h0, nh, vec, a.scale, z);
#pragma unroll
                for (int hh = 0; hh < 4; ++hh)
                    if (hh < nh) best = fmaxf(best, z[hh]);
            }
            if (a.score_out) a.score_out[((size_t)b * a.H_kv + g) * L + t] = best;
            list[at] = __float_as_uint(best);
            list[at + kRowList] = (uint32_t)t;
        }
        // tokens of this wavefront: rounds of 64, the last one in part
        const int full = L / kRowThreads, rest = L - full * kRowThreads - 64 * w;
        const uint32_t count = (uint32_t)(64 * full + (rest < 0 ? 0 : rest < 64 ? rest : 64));
        // ---- the k largest (the lists hold the whole row)
        (void)select_from_lists(lists, count, (uint32_t)k, 0u, 0xFFFFFFFFu, bins, map, words, sh);
        write_map(map, words, (uint32_t)k, sh, ids);
        __syncthreads();
    } else {
        for (int j = tid; j < k; j += THREADS) {
            const int t = a.idx[((size_t)b * a.H_kv + g) * k + j];
            ids[j] = t < 0 ? 0 : (t >= L ? L - 1 : t);
        }
        __syncthreads();
    }
    if (WHOLE && a.idx_out)
        for (int j = tid; j < k; j += kRowThreads) a.idx_out[((size_t)b * a.H_kv + g) * k + j] = ids[j];
    // the first values that the thread takes below are requested here, behind the logits' rows  (the sums' parts don't depend on how many
    // threads share them)
    const int parts = kRowThreads / r_v < kSmPart / (n_rep * r_v) ? kRowThreads / r_v : kSmPart / (n_rep * r_v);
    const int grp = tid / r_v, col = tid - grp * r_v;
    const bool sums = grp < parts;
    const float x = sums && grp < k ? A_v[(size_t)ids[grp] * r_v + col] : 0.0f;
    // ---- logits of the selected rows, a thread per row and head, and of the tail
    for (int i = tid; i < n_rep * k; i += THREADS) {
        const int hh = i / k, j = i - hh * k;
        const float *row = A_k + (size_t)ids[j] * r_k;
        const double *ph = Pd + hh * r_k;
        double z = 0.0;
#pragma unroll 8
        for (int c = 0; c < r_k; ++c) z = fma((double)row[c], ph[c], z);
        wt[hh * n + j] = (float)((double)a.scale * z);
    }
    for (int t = w; t < T; t += WAVES)
        for (int hh = 0; hh < n_rep; ++hh) {
            float part = 0.0f;
            for (int j = lane; j < d_h; j += kWave) part = fmaf(K_t[(size_t)t * d_h + j], q[(size_t)hh * d_h + j], part);
            part = wave_sum(part);
            if (lane == 0) wt[hh * n + k + t] = a.scale * part;
        }
    __syncthreads();
    // ---- weights, a wavefront per head
    for (int hh = w; hh < n_rep; hh += WAVES) {
        float m = -INFINITY, den = 0.0f;
        for (int j = lane; j < n; j += kWave) {
            m = fmaxf(m, wt[hh * n + j]);
        }
        m = wave_max(m);
        for (int j = lane; j < n; j += kWave) {
            const float e = expf(wt[hh * n + j] - m);
            wt[hh * n + j] = e;
            den += e;
        }
        den = wave_sum(den);
        if (lane == 0) head_den[hh] = den;
    }
    __syncthreads();
    // ---- U = w A^V[rows]: `parts` groups of threads share the rows, a thread per rank and four heads at a time
    float *U = P;
    auto sum_part = [&](int grp, int col, auto first) __attribute__((always_inline)) {  // first: the value that is there already
        for (int h0 = 0; h0 < n_rep; h0 += 4) {
            const int nh = n_rep - h0 < 4 ? n_rep - h0 : 4;
            float u[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
            for (int j = grp; j < k; j += parts) {
                const float v = first && j == grp ? x : A_v[(size_t)ids[j] * r_v + col];
#pragma unroll
                for (int hh = 0; hh < 4; ++hh) u[hh] = fmaf(wt[(h0 + (hh < nh ? hh : 0)) * n + j], v, u[hh]);
            }
#pragma unroll
            for (int hh = 0; hh < 4; ++hh)
                if (hh < nh) part[(grp * n_rep + h0 + hh) * r_v + col] = u[hh];
        }
    };
    if (sums) sum_part(grp, col, std::true_type());
    if constexpr (THREADS < kRowThreads)
        for (int vt = tid + THREADS; vt < parts * r_v; vt += THREADS) sum_part(vt / r_v, vt % r_v, std::false_type());
    __syncthreads();
    for (int i = tid; i < n_rep * r_v; i += THREADS) {
        float u = 0.0f;
        for (int p = 0; p < parts; ++p) u += part[p * n_rep * r_v + i];
        U[i] = u;
    }
    __syncthreads();
    // ---- out = (U B^V + w V_tail) / den: the ranks and the tail's tokens in `cuts` parts
    const int cols = n_rep * d_h;
    int cuts = kRowThreads / cols;
    cuts = cuts < 1 ? 1 : cuts;
    for (int i = tid; i < cols * cuts; i += THREADS) {
        const int cut = i / cols, hj = i - cut * cols, hh = hj / d_h, j = hj - hh * d_h;
        float o = 0.0f;
#pragma unroll 8
        for (int c = cut; c < r_v; c += cuts) o = fmaf(U[hh * r_v + c], B_v[(size_t)c * d + j], o);
#pragma unroll 4
        for (int t = cut; t < T; t += cuts) o = fmaf(wt[hh * n + k + t], V_t[(size_t)t * d_h + j], o);
        part[i] = o;
    }
    __syncthreads();
    for (int hj = tid; hj < cols; hj += THREADS) {
        float o = 0.0f;
        for (int cut = 0; cut < cuts; ++cut) o += part[cut * cols + hj];
        a.out[((size_t)b * a.H_q + (size_t)g * n_rep) * d_h + hj] = o / head_den[hj / d_h];
    }
}

// A mebibyte of A, B and the tail per workgroup at most (see above); everything else fits its LDS.
bool small_step_ok(const xkv_shape &s, int T)
{
    if (s.dtype != XKV_F32 || s.H_kv < 1) return false;
    const long long n_rep = s.H_q / s.H_kv, d_h = s.d_h;
    const long long numbers = (long long)s.L * s.r_k + (long long)s.k * s.r_v + (s.r_k + s.r_v + 2LL * T) * d_h;
    return numbers <= 262144 && s.L <= 4096 && n_rep <= 16 && n_rep * s.r_k <= kSmRank && n_rep * s.r_v <= kSmRank &&
           s.r_v <= kRowThreads && n_rep * d_h <= kSmPart && s.k + n_rep * (s.k + T) <= kSmLists;
}

// Scores and selection on one compute unit against two launches and a selection over all of them (staged / whole, in a graph, us, one KV head:
// 2048 tokens of rank 32 23.5 / 21.0, 4096 23.4 / 28.5, 2048 of rank 64 27.4 / 30.5, 1000 of rank 128 43.7 / 42.3, 512 of rank 256 102 / 97, 3000 of
// rank 64 27.1 / 37.5; launched one by one, three launches more cost 3 to 5 us more).  The score kernel takes the KV heads of a sequence one
// after the other: with two 3000 of rank 64 31 / 38, with four about the same, with eight a whole step is 1.1 to 1.7 times as fast.
bool small_step_whole(const xkv_shape &s)
{
    return (long long)s.batch * s.H_kv > 32 || s.H_kv > 2 || (long long)s.L * s.r_k <= 163840;
}

// idx (nullable): attend over these rows only, nothing is scored or selected
hipError_t launch_small_step(const xkv_shape &s, int layer, const void *A_k, const void *A_v, const void *B_k, const void *B_v, const void *q,
                             const void *K_tail, const void *V_tail, int T, void *out, int32_t *idx_out, float *score_out, float scale,
                             const int32_t *idx, hipStream_t st)
{
    static DynamicLdsOnce attr, attr_rows, attr_few;
    const SmallArgs a{(const float *)A_k, (const float *)A_v, (const float *)B_k, (const float *)B_v, (const float *)q, (const float *)K_tail,
                      (const float *)V_tail, (float *)out, score_out, idx_out, idx, s.G, layer, s.L, s.r_k, s.r_v, s.H_kv, s.H_q, s.d_h, s.k, T,
                      scale};
    const dim3 grid(s.H_kv * s.batch);
    if (idx) {
        const int n_rep = s.H_q / s.H_kv;
        const size_t words = rows_words(n_rep, s.k + T, s.k) + kSmPart + 3 * (size_t)rank_words(n_rep, s.r_k, s.r_v);
        // Small ones on more workgroups than compute units: four wavefronts each, several workgroups per compute unit (rows given, 4 heads of 64,
        // ranks 32, 32 of 512 rows, 288 pairs 16.7 -> 14.1 us, 4096 137 -> 76; the general kernels 24 and 168).  Sixteen are faster for more
        // work on few pairs (ranks 128, 64 rows, heads of 128: 288 pairs 47 / 61, 1024 93 / 73; 100 rows 1024 pairs 104 / 135) or for long
        // lists (ranks 64, 256 rows, 1024 pairs 81 / 104).
        const long long pairs = (long long)s.batch * s.H_kv, work = (long long)n_rep * s.r_k * (s.k + s.d_h);
        const bool few = pairs > 256 && (work <= 32768 || (pairs > 512 && s.k <= 128 && work <= 100000));
        auto launch = [&](auto kernel, DynamicLdsOnce &at, int threads) {
            const hipError_t e = at.ensure((const void *)kernel, (size_t)kSmWords * 4);
            if (e != hipSuccess) return e;
            profile_begin(1, st);
            hipLaunchKernelGGL(kernel, grid, dim3(threads), words * 4, st, a);
            profile_end(1, st);
            return hipGetLastError();
        };
        return few ? launch(small_step_kernel<false, 256>, attr_few, 256) : launch(small_step_kernel<false, kRowThreads>, attr_rows, kRowThreads);
    } else {
        const hipError_t e = attr.ensure((const void *)small_step_kernel<true, kRowThreads>, (size_t)kSmWords * 4);
        if (e != hipSuccess) return e;
        profile_begin(0, st);  // (it is the score kernel and the one for the selected rows)
        profile_begin(1, st);
        hipLaunchKernelGGL((small_step_kernel<true, kRowThreads>), grid, dim3(kRowThreads), (size_t)kSmWords * 4, st, a);
        profile_end(1, st);
        profile_end(0, st);
    }
    return hipGetLastError();
}

}  // namespace xkv
