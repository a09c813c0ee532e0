// Dense decode attention on an uncompressed cache (the "Full Attention" baseline of Sec. 5):
//   out_h = softmax(scale * K_{rho(h)} q_h)^T V_{rho(h)}  over all L tokens,
// split over the tokens flash-decoding style, plus the kernel that merges split partials
// (shared with the SR path).
#include "xkv_common.h"
#include "dense_block.h"

namespace xkv {

// ------------------------------------------------------------------------------------------
// General path: lanes run over the head dimension, a wavefront walks TM tokens at a time.
// K, V: [batch][H_kv][L][d_h].
// ------------------------------------------------------------------------------------------
template <typename T, int JP>
__global__ __launch_bounds__(256) void dense_generic_kernel(const T *__restrict__ K, const T *__restrict__ V,
                                                            const T *__restrict__ q, float *__restrict__ part_o,
                                                            float *__restrict__ part_ml, int L, int H_kv, int H_q,
                                                            int d_h, int splits, int chunk, float scale)
{
    constexpr int TM = 4;
    const int split = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    const int n_rep = H_q / H_kv;
    const int lane = lane_id(), w = wave_id();

    float qreg[16][JP], o[16][JP], mx[16], den[16];
#pragma unroll
    for (int hh = 0; hh < 16; ++hh) {
        mx[hh] = -INFINITY;
        den[hh] = 0.0f;
#pragma unroll
        for (int jj = 0; jj < JP; ++jj) {
            const int j = lane + jj * kWave;
            o[hh][jj] = 0.0f;
            qreg[hh][jj] = (hh < n_rep && j < d_h) ? to_f32(q[((size_t)b * H_q + g * n_rep + hh) * d_h + j]) : 0.0f;
        }
    }
    const T *Kg = K + ((size_t)b * H_kv + g) * L * d_h;
    const T *Vg = V + ((size_t)b * H_kv + g) * L * d_h;
    const int t_begin = split * chunk;
    const int t_end = (t_begin + chunk < L) ? t_begin + chunk : L;

    for (int t0 = t_begin + w * TM; t0 < t_end; t0 += 4 * TM) {
        float kr[TM][JP], vr[TM][JP];
#pragma unroll
        for (int mm = 0; mm < TM; ++mm) {
            const int t = (t0 + mm < t_end) ? t0 + mm : t_end - 1;
#pragma unroll
            for (int jj = 0; jj < JP; ++jj) {
                const int j = lane + jj * kWave;
                kr[mm][jj] = j < d_h ? to_f32(Kg[(size_t)t * d_h + j]) : 0.0f;
                vr[mm][jj] = j < d_h ? to_f32(Vg[(size_t)t * d_h + j]) : 0.0f;
            }
        }
#pragma unroll
        for (int mm = 0; mm < TM; ++mm) {
            if (t0 + mm < t_end) {  // wave-uniform
#pragma unroll
                for (int hh = 0; hh < 16; ++hh) {
                    if (hh < n_rep) {
                        float part = 0.0f;
#pragma unroll
                        for (int jj = 0; jj < JP; ++jj) part = fmaf(kr[mm][jj], qreg[hh][jj], part);
                        const float z = scale * wave_sum(part);
                        const float m_new = fmaxf(mx[hh], z);
                        const float alpha = expf(mx[hh] - m_new);
                        const float pw = expf(z - m_new);
                        den[hh] = den[hh] * alpha + pw;
#pragma unroll
                        for (int jj = 0; jj < JP; ++jj) o[hh][jj] = fmaf(pw, vr[mm][jj], o[hh][jj] * alpha);
                        mx[hh] = m_new;
                    }
                }
            }
        }
    }

    const int n_part = splits * 4, part = split * 4 + w;
#pragma unroll
    for (int hh = 0; hh < 16; ++hh) {
        if (hh < n_rep) {
            const size_t slot = ((size_t)b * H_q + g * n_rep + hh) * n_part + part;
#pragma unroll
            for (int jj = 0; jj < JP; ++jj) {
                const int j = lane + jj * kWave;
                if (j < d_h) part_o[slot * d_h + j] = o[hh][jj];
            }
            if (lane == 0) {
                part_ml[slot * 2 + 0] = mx[hh];
                part_ml[slot * 2 + 1] = den[hh];
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Merge the split partials of one (sequence, query head) with the log-sum-exp rule and write
// the normalised output in the storage dtype.  A partial that saw no token has max = -inf.
// Latency is all there is to it, so every load is requested at once: (maximum, sum) of every partial, and the first BATCH
// partials of each of the groups of 2^tpg threads that share the partials between them (thread = VEC columns of one
// group's partials, a group covers all columns, the groups are added up at the end).  One thread per column, four partials
// at a time and the sums loaded after the maxima took 13.5 us with 64 partials (d_h = 128, 32 heads) and
// 4.1 us with 8, now 6.5 and 3.9 us.
// ------------------------------------------------------------------------------------------
template <typename T, int VEC>
__global__ __launch_bounds__(256) void combine_kernel(const float *__restrict__ part_o,
                                                      const float *__restrict__ part_ml, T *__restrict__ out,
                                                      int H_q, int d_h, int n_part,
                                                      const float *__restrict__ part_o2,
                                                      const float *__restrict__ part_ml2, int n_part2, int tpg)
{
    typedef __attribute__((ext_vector_type(VEC))) float vec_t;
    // the second set of partials (n_part2 may be 0) has the same layout; it holds the uncompressed tail tokens
    const int h = blockIdx.x, b = blockIdx.y;
    const size_t base = ((size_t)b * H_q + h) * n_part, base2 = ((size_t)b * H_q + h) * n_part2;
    constexpr int BATCH = VEC == 1 ? 16 : 8, PER = kMaxCombineParts / 256;
    __shared__ float sm_w[kMaxCombineParts], sm_red[2][4];
    __shared__ vec_t sm_acc[256];
    const int n_all = n_part + n_part2, cols = d_h / VEC;
    const int n_grp = (int)blockDim.x >> tpg, grp = (int)threadIdx.x >> tpg, j = (int)threadIdx.x & ((1 << tpg) - 1);
    const int jc = j < cols ? j : cols - 1;
    // partials s1 + grp, s1 + grp + n_grp, .. (a load under a lane's condition would be waited for: lanes beyond the last one
    // read the last one again, and whole steps beyond it are left out)
    auto fetch = [&](int s1, vec_t (&v)[BATCH]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            if (s1 + n_grp * u >= n_all) break;
            const int t = s1 + n_grp * u + grp, s = t < n_all ? t : n_all - 1;
            const float *p = s < n_part ? part_o + (base + s) * d_h : part_o2 + (base2 + (s - n_part)) * d_h;
            v[u] = *reinterpret_cast<const vec_t *>(p + VEC * jc);
        }
    };
    // up to 64 partials: every wavefront holds (maximum, sum) of all of them, a lane each, and needs neither LDS nor a
    // barrier for the weights (lane s: weight of partial s); more: a thread of 256 each, PER at most
    const bool few = n_all <= kWave;
    const int lane = lane_id(), first = few ? lane : (int)threadIdx.x;
    float pm[PER], pl[PER];
    vec_t v[BATCH];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int s = first + 256 * u, sc = s < n_all ? s : n_all - 1;
        const float *p = sc < n_part ? part_ml + (base + sc) * 2 : part_ml2 + (base2 + (sc - n_part)) * 2;
        pm[u] = -INFINITY;
        pl[u] = 0.0f;
        if (256 * u < n_all) {  // (the same in every thread)
            const float m = p[0], l = p[1];
            pm[u] = s < n_all ? m : -INFINITY;
            pl[u] = s < n_all ? l : 0.0f;
        }
    }
    fetch(0, v);
    float M = pm[0], den, weight = 0.0f;
    if (few) {
        for (int off = 1; off < n_all; off <<= 1) M = fmaxf(M, __shfl_xor(M, off, kWave));
        M = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, M)));
        weight = pm[0] == -INFINITY ? 0.0f : expf(pm[0] - M);
        den = weight * pl[0];
        for (int off = 1; off < n_all; off <<= 1) den += __shfl_xor(den, off, kWave);
        den = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, den)));
    } else {
#pragma unroll
        for (int u = 1; u < PER; ++u) M = fmaxf(M, pm[u]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off, kWave));
        if (lane == 0) sm_red[0][wave_id()] = M;
        __syncthreads();
        M = fmaxf(fmaxf(sm_red[0][0], sm_red[0][1]), fmaxf(sm_red[0][2], sm_red[0][3]));
        den = 0.0f;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int s = first + 256 * u;
            if (s < n_all) {
                const float wt = (pm[u] == -INFINITY) ? 0.0f : expf(pm[u] - M);
                sm_w[s] = wt;
                den = fmaf(wt, pl[u], den);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) den += __shfl_xor(den, off, kWave);
        if (lane == 0) sm_red[1][wave_id()] = den;
        __syncthreads();
        den = (sm_red[1][0] + sm_red[1][1]) + (sm_red[1][2] + sm_red[1][3]);
    }
    vec_t num = vec_t(0.0f);
    auto add_up = [&](auto weight_of) __attribute__((always_inline)) {  // (the same number of rounds in every thread: lanes exchange)
        for (int s1 = 0; s1 < n_all; s1 += n_grp * BATCH) {
            if (s1 > 0) fetch(s1, v);
            float wt[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int s = s1 + n_grp * u + grp;
                wt[u] = weight_of(s < n_all ? s : n_all - 1);
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
                if (s1 + n_grp * u + grp < n_all) num += wt[u] * v[u];
        }
    };
    if (few)
        add_up([&](int s) __attribute__((always_inline)) { return __shfl(weight, s, kWave); });
    else
        add_up([&](int s) __attribute__((always_inline)) { return sm_w[s]; });
    const int n_sum = n_all < n_grp ? n_all : n_grp;  // groups that have a partial
    if (n_sum > 1) {
        sm_acc[threadIdx.x] = num;
        __syncthreads();
    }
    if (grp == 0 && j < cols) {
        for (int k = 1; k < n_sum; ++k) num += sm_acc[(k << tpg) + j];
        // a head with no token at all (every list empty, no tail) has den == 0: its output is defined as zero
        T *o = out + ((size_t)b * H_q + h) * d_h + VEC * j;
#pragma unroll
        for (int e = 0; e < VEC; ++e) o[e] = from_f32<T>(den > 0.0f ? num[e] / den : 0.0f);
    }
}

// The matrix-core path (dense_block.h).
__global__ __launch_bounds__(256, 2) void dense_mfma_kernel(DenseArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char smem[dense::kLdsBytes];
    dense::mfma_block(a, blockIdx.x, blockIdx.y, blockIdx.z, smem);
}

DenseArgs dense_args(const xkv_shape &s, const Plan &p, const void *K, const void *V, const void *q, float *part_o, float *part_ml)
{
    return DenseArgs{(const bf16_t *)K, (const bf16_t *)V, (const bf16_t *)q, part_o, part_ml, s.L, s.H_kv, s.H_q, p.dense_splits,
                     p.dense_chunk, s.batch, p.scale};
}

template <typename T>
static hipError_t launch_dense_generic(const xkv_shape &s, const Plan &p, const void *K, const void *V, const void *q,
                                       float *part_o, float *part_ml, hipStream_t st)
{
    dim3 grid(p.dense_splits, s.H_kv, s.batch), block(256);
#define XKV_DENSE_LAUNCH(JP)                                                                                    \
    hipLaunchKernelGGL((dense_generic_kernel<T, JP>), grid, block, 0, st, (const T *)K, (const T *)V,           \
                       (const T *)q, part_o, part_ml, s.L, s.H_kv, s.H_q, s.d_h, p.dense_splits, p.dense_chunk, \
                       p.scale)
    profile_begin(2, st);
    if (s.d_h <= 64)
        XKV_DENSE_LAUNCH(1);
    else if (s.d_h <= 128)
        XKV_DENSE_LAUNCH(2);
    else
        XKV_DENSE_LAUNCH(4);
    profile_end(2, st);
#undef XKV_DENSE_LAUNCH
    return hipGetLastError();
}

bool dense_mfma_shape_ok(const xkv_shape &s) { return s.dtype == XKV_BF16 && s.d_h == 128; }

bool dense_uses_mfma(const Plan &p, const void *K, const void *V, const void *q);

hipError_t launch_dense(const xkv_shape &s, const Plan &p, const void *K, const void *V, const void *q, float *part_o,
                        float *part_ml, hipStream_t st)
{
    if (dense_uses_mfma(p, K, V, q)) {
        dim3 grid(p.dense_splits, s.H_kv, s.batch), block(256);
        profile_begin(2, st);
        hipLaunchKernelGGL(dense_mfma_kernel, grid, block, 0, st, dense_args(s, p, K, V, q, part_o, part_ml));
        profile_end(2, st);
        return hipGetLastError();
    }
    if (s.dtype == XKV_F32) return launch_dense_generic<float>(s, p, K, V, q, part_o, part_ml, st);
    return launch_dense_generic<bf16_t>(s, p, K, V, q, part_o, part_ml, st);
}

hipError_t launch_combine(const xkv_shape &s, int n_part, const float *part_o, const float *part_ml, void *out,
                          hipStream_t st, int n_part2, const float *part_o2, const float *part_ml2)
{
    if (n_part + n_part2 > kMaxCombineParts) return hipErrorInvalidValue;
    const bool vec = s.d_h % 4 == 0;  // four columns per thread (the partials begin on 256-byte boundaries of the workspace)
    // A group of threads covers the columns (d_h <= 256); at most eight groups, no more than there are partials, and whole
    // wavefronts: 256 threads for each of 2048 output rows of 128 columns and two partials cost 1.2 us of 28, groups of 64
    // threads in four rounds 40 of 180 us at 255 columns.  More than 64 partials need the 256 threads for their weights.
    int tpg = 3;
    while ((1 << tpg) < (vec ? s.d_h / 4 : s.d_h)) ++tpg;
    const int n_all = n_part + n_part2, grps = n_all < 8 ? n_all : 8;
    const int threads = n_all > kWave || (grps << tpg) > 256 ? 256 : ((grps << tpg) + 63) / 64 * 64;
    auto launch = [&](auto kernel, auto *o) {
        hipLaunchKernelGGL(kernel, dim3(s.H_q, s.batch), dim3(threads), 0, st, part_o, part_ml, o, s.H_q, s.d_h, n_part, part_o2,
                           part_ml2, n_part2, tpg);
    };
    if (s.dtype == XKV_F32)
        vec ? launch(combine_kernel<float, 4>, (float *)out) : launch(combine_kernel<float, 1>, (float *)out);
    else
        vec ? launch(combine_kernel<bf16_t, 4>, (bf16_t *)out) : launch(combine_kernel<bf16_t, 1>, (bf16_t *)out);
    return hipGetLastError();
}

// Whether launch_dense takes the matrix-core kernel (one partial per split) or the general one (one per wavefront).
bool dense_uses_mfma(const Plan &p, const void *K, const void *V, const void *q)
{
    return p.dense_mfma && ((((uintptr_t)K | (uintptr_t)V | (uintptr_t)q)) & 15u) == 0;
}

}  // namespace xkv
