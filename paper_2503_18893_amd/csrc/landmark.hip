// landmark.hip -- the paper's own token selector for Selective Reconstruction (App. B.1): landmark construction
// at prefill (Alg. 1) and the pieces of the landmark-guided chunk selection at decode (Alg. 2) that are not
// already kernels of the factor-scoring path.
//
// At decode, scoring chunks against landmarks is the same computation as scoring tokens against the key factors
// with the landmarks of one KV head in the place of A^K (n_c rows of d_h values), the head's queries in the place
// of the projected queries, and an identity matrix in the place of B^K: the score kernels, the GQA max-pool and
// the radix top-k are used unchanged on that reshaped problem.  What is new here: the chunk means and the
// within-chunk minimum cosine (Alg. 1), the union of the top chunks with the static outliers and its expansion
// to token rows (Alg. 2, last two steps).
#include "xkv_common.h"
#include "expand_block.h"

namespace xkv {
namespace {

// One wavefront per chunk: lane l holds channels l, l + 64, ... of the d_h <= 256 channels.  Landmark = mean of the
// chunk's keys (a shorter last chunk: mean over the tokens it has), rounded once to the storage type; the cosine
// of every key with the fp32 mean, its minimum over the chunk negated into neg_min_cos (so that the chunks with
// the smallest minimum are the top of ArgTopK(-m, o), Alg. 1).  A zero key or a zero mean counts as cosine 0.
template <typename T>
__global__ __launch_bounds__(256) void landmark_kernel(const T *__restrict__ K, T *__restrict__ Lm, float *__restrict__ neg_m,
                                                       int L, int d_h, int c, int n_c)
{
    const int j = blockIdx.x * 4 + wave_id(), row = blockIdx.y;  // chunk, (sequence, KV head)
    if (j >= n_c) return;
    const int lane = lane_id();
    const int t0 = j * c, t1 = (t0 + c < L) ? t0 + c : L;
    const T *Kr = K + (size_t)row * L * d_h;
    float mean[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int t = t0; t < t1; ++t)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ch = lane + 64 * u;
            if (ch < d_h) mean[u] += to_f32(Kr[(size_t)t * d_h + ch]);
        }
    const float inv = 1.0f / (float)(t1 - t0);
    float mm = 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        mean[u] *= inv;
        mm += mean[u] * mean[u];
        const int ch = lane + 64 * u;
        if (ch < d_h) Lm[((size_t)row * n_c + j) * d_h + ch] = from_f32<T>(mean[u]);
    }
    mm = wave_sum(mm);
    float worst = INFINITY;
    for (int t = t0; t < t1; ++t) {
        float xm = 0.0f, xx = 0.0f;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int ch = lane + 64 * u;
            const float x = ch < d_h ? to_f32(Kr[(size_t)t * d_h + ch]) : 0.0f;
            xm += x * mean[u];
            xx += x * x;
        }
        xm = wave_sum(xm);
        xx = wave_sum(xx);
        const float den = sqrtf(xx) * sqrtf(mm);
        worst = fminf(worst, den > 0.0f ? xm / den : 0.0f);
    }
    if (lane == 0 && neg_m) neg_m[(size_t)row * n_c + j] = -worst;
}

// The same for bf16 keys of 128 channels and chunks of 4, 8, 12 or 16 tokens, read once and line-wise.  A wavefront takes
// four chunks, one per row of 16 lanes: lane l holds the 16 B piece l % 16 of every key of chunk l / 16, so that a request
// covers two whole lines of four keys, sums over a chunk's keys stay in the lane and only sums over channels run across the
// 16 lanes, as operand modifiers of additions.  Root and quotient are taken once per key, by lane i of the chunk's 16 for its
// key i.  The stream of keys bounds it as long as little else is done per key (keys across the rows of lanes, exchanges
// through LDS and a root and a quotient in every lane: 36 us for 8 x 50001 keys in chunks of 8, now 19.7; 102 MB, 16 us
// to read).
typedef __attribute__((ext_vector_type(4))) uint32_t lm_u32x4_t;
template <int CTRL> __device__ __forceinline__ float lm_dpp(float x)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(x), CTRL, 0xF, 0xF, true));
}
// over the 16 lanes of a row, neighbours first: lanes 1 0 3 2, then 2 3 0 1, then the two mirrored orders
__device__ __forceinline__ float lm_row_sum(float v)
{
    v += lm_dpp<0xB1>(v);
    v += lm_dpp<0x4E>(v);
    v += lm_dpp<0x141>(v);
    v += lm_dpp<0x140>(v);
    return v;
}

template <int C>
__global__ __launch_bounds__(256) void landmark_bf16_128_kernel(const bf16_t *__restrict__ K, bf16_t *__restrict__ Lm,
                                                                float *__restrict__ neg_m, int L, int n_c)
{
    const int j0 = (blockIdx.x * 4 + wave_id()) * 4, row = blockIdx.y;
    if (j0 >= n_c) return;
    const int lane = lane_id(), pc = lane & 15;
    const int j = j0 + (lane >> 4) < n_c ? j0 + (lane >> 4) : n_c - 1;  // (lanes beyond the last chunk repeat it)
    const int t0 = j * C, nt = L - t0 < C ? L - t0 : C;                  // first key of the chunk, keys that it has
    const lm_u32x4_t *Kc = reinterpret_cast<const lm_u32x4_t *>(K + ((size_t)row * L + t0) * 128) + pc;
    lm_u32x4_t xs[C];
#pragma unroll
    for (int i = 0; i < C; ++i) xs[i] = __builtin_nontemporal_load(Kc + 16 * (i < nt ? i : nt - 1));
    if (nt < C) {
#pragma unroll
        for (int i = 1; i < C; ++i)
            if (i >= nt) xs[i] = lm_u32x4_t{0u, 0u, 0u, 0u};
    }
    const float inv = 1.0f / (float)nt;
    float mean[8], mm = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float s4[4];  // (keys i, i + 4, .. first)
#pragma unroll
        for (int i = 0; i < C; ++i) {
            const float x = __uint_as_float(e & 1 ? xs[i][e >> 1] & 0xFFFF0000u : xs[i][e >> 1] << 16);
            s4[i & 3] = i < 4 ? x : s4[i & 3] + x;
        }
        mean[e] = ((s4[0] + s4[1]) + (s4[2] + s4[3]) + 0.0f) * inv;  // (+ 0: the mean of negative zeros is zero)
        mm += mean[e] * mean[e];
    }
    mm = lm_row_sum(mm);
    lm_u32x4_t pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (uint32_t)f32_to_bf16(mean[2 * e]) | ((uint32_t)f32_to_bf16(mean[2 * e + 1]) << 16);
    reinterpret_cast<lm_u32x4_t *>(Lm + ((size_t)row * n_c + j) * 128)[pc] = pk;
    float xm_l = 0.0f, xx_l = 0.0f;  // of the key that this lane stands for
#pragma unroll
    for (int i = 0; i < C; ++i) {
        float xm = 0.0f, xx = 0.0f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x0 = __uint_as_float(xs[i][e] << 16), x1 = __uint_as_float(xs[i][e] & 0xFFFF0000u);
            xm += x0 * mean[2 * e] + x1 * mean[2 * e + 1];
            xx += x0 * x0 + x1 * x1;
        }
        xm = lm_row_sum(xm);
        xx = lm_row_sum(xx);
        xm_l = pc == i ? xm : xm_l;
        xx_l = pc == i ? xx : xx_l;
    }
    const float den = sqrtf(xx_l) * sqrtf(mm);
    const float cs = den > 0.0f ? xm_l / den : 0.0f;
    float worst = pc < nt ? fminf(INFINITY, cs) : INFINITY;
    worst = fminf(worst, lm_dpp<0xB1>(worst));
    worst = fminf(worst, lm_dpp<0x4E>(worst));
    worst = fminf(worst, lm_dpp<0x141>(worst));
    worst = fminf(worst, lm_dpp<0x140>(worst));
    if (pc == 0 && neg_m) neg_m[(size_t)row * n_c + j] = -worst;
}

// `copies` identity matrices [d_h][d_h] in the storage type.
template <typename T> __global__ __launch_bounds__(256) void identity_kernel(T *__restrict__ B, int d_h, long long count)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= count) return;
    const int col = (int)(i % d_h), rw = (int)((i / d_h) % d_h);
    B[i] = from_f32<T>(rw == col ? 1.0f : 0.0f);
}

// The union of chunks and outliers as a launch of its own, one workgroup per (sequence, KV head).
__global__ __launch_bounds__(256) void expand_chunks_kernel(const int32_t *__restrict__ chunks, int k_ch, ExpandArgs e)
{
    extern __shared__ int32_t lds_i[];
    const int row = blockIdx.x;
    for (int a = threadIdx.x; a < k_ch; a += 256) {
        const int v = chunks[(size_t)row * k_ch + a];
        lds_i[a] = v < 0 ? 0 : (v >= e.n_c ? e.n_c - 1 : v);
    }
    expand_block(lds_i, k_ch, e, row, lds_i + k_ch, 256);
}

}  // namespace

hipError_t launch_landmarks(const xkv_shape &s, const void *K_rope, int c, void *landmarks, float *neg_min_cos,
                            hipStream_t st)
{
    const int n_c = (s.L + c - 1) / c;
    dim3 grid((n_c + 3) / 4, s.batch * s.H_kv);
    if (s.dtype == XKV_BF16 && s.d_h == 128 && c % 4 == 0 && c <= 16 && (((uintptr_t)K_rope | (uintptr_t)landmarks) & 15u) == 0) {
        const dim3 grid4((n_c + 15) / 16, s.batch * s.H_kv);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, grid4, dim3(256), 0, st, (const bf16_t *)K_rope, (bf16_t *)landmarks, neg_min_cos, s.L, n_c);
        };
        c == 4 ? launch(landmark_bf16_128_kernel<4>) : c == 8 ? launch(landmark_bf16_128_kernel<8>)
            : c == 12 ? launch(landmark_bf16_128_kernel<12>) : launch(landmark_bf16_128_kernel<16>);
        return hipGetLastError();
    }
    if (s.dtype == XKV_F32)
        hipLaunchKernelGGL(landmark_kernel<float>, grid, dim3(256), 0, st, (const float *)K_rope, (float *)landmarks,
                           neg_min_cos, s.L, s.d_h, c, n_c);
    else
        hipLaunchKernelGGL(landmark_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t *)K_rope, (bf16_t *)landmarks,
                           neg_min_cos, s.L, s.d_h, c, n_c);
    return hipGetLastError();
}

hipError_t launch_identity(const xkv_shape &s, void *B, int copies, hipStream_t st)
{
    const long long count = (long long)copies * s.d_h * s.d_h;
    const unsigned blocks = (unsigned)((count + 255) / 256);
    if (s.dtype == XKV_F32)
        hipLaunchKernelGGL(identity_kernel<float>, dim3(blocks), dim3(256), 0, st, (float *)B, s.d_h, count);
    else
        hipLaunchKernelGGL(identity_kernel<bf16_t>, dim3(blocks), dim3(256), 0, st, (bf16_t *)B, s.d_h, count);
    return hipGetLastError();
}

hipError_t launch_expand_chunks(int rows, const int32_t *chunks, int k_ch, const ExpandArgs &e, hipStream_t st)
{
    hipLaunchKernelGGL(expand_chunks_kernel, dim3(rows), dim3(256), ((size_t)k_ch + expand_lds_words(k_ch, e.o)) * sizeof(int32_t), st,
                       chunks, k_ch, e);
    return hipGetLastError();
}

}  // namespace xkv
