// The policy that consumes the depth stack in place (Section 4.2 "Approach:
// End-to-End RL"; the SimpleCNN visual encoder of the appendix on model
// sizes: three convolutions without padding or dilation, 8x8 stride 4, 4x4
// stride 2, 3x3 stride 1, each with ReLU, then a fully connected layer), with
// a Gaussian actor and a critic linear in the 512 features and the 7 joint
// angles.  BF16 weights and activations, FP32 accumulation on the matrix
// cores, FP32 heads.
//
// The convolutions are in k_policy_enc.hip and k_policy_bwd.hip; here are the
// heads, the fully connected layer's split, the PPO loss and the sums.
#include "gal_internal.h"
#include "gal_mlp.h"
#include "gal_policy.h"

#include <algorithm>

namespace gal {

namespace {

__device__ __forceinline__ uint16_t f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// The heads of env e (one wave): f = [h (BF16 features), q (joint angles)];
// mean_a = b_a + sum_k W_a[k] f_k, value = b_v + sum_k w_v[k] f_k (FP32,
// lane-strided partial sums combined by a fixed butterfly); the action
// mean + std * noise and its Gaussian log-density sum_a (-noise_a^2 / 2 -
// log_std_a) - A log(2 pi) / 2 (noise null: the mean, no log-density).
__global__ __launch_bounds__(256) void k_policy_heads(const uint16_t *__restrict__ h, const float *__restrict__ state,
                                                      const float *__restrict__ aw, const float *__restrict__ ab,
                                                      const float *__restrict__ vw, const float *__restrict__ vb,
                                                      const float *__restrict__ log_std, int A, int n_envs,
                                                      const float *__restrict__ noise, float *__restrict__ actions,
                                                      float *__restrict__ value, float *__restrict__ logp)
{
    const int lane = threadIdx.x & 63;
    const int e = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)threadIdx.x / 64);
    if (e >= n_envs) return;
    constexpr int F = kPolicyFeat + kPolicyProprio;
    float f[(F + 63) / 64];
#pragma unroll
    for (int i = 0; i < (F + 63) / 64; ++i) {
        const int k = lane + 64 * i;
        f[i] = k < kPolicyFeat ? bf2f(h[(size_t)e * kPolicyFeat + k])
                               : (k < F ? state[(size_t)e * 10 + 3 + (k - kPolicyFeat)] : 0.0f);
    }
    float lp = 0.0f;
    for (int a = 0; a <= A; ++a) {
        const float *w = a < A ? aw + (size_t)a * F : vw;
        float s = 0.0f;
#pragma unroll
        for (int i = 0; i < (F + 63) / 64; ++i) {
            const int k = lane + 64 * i;
            if (k < F) s += w[k] * f[i];
        }
        for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
        if (a < A) {
            const float mean = s + ab[a];
            float act = mean;
            if (noise) {
                const float z = noise[(size_t)e * A + a];
                act = mean + expf(log_std[a]) * z;
                lp += -0.5f * z * z - log_std[a];
            }
            if (lane == 0) actions[(size_t)e * A + a] = act;
        } else if (lane == 0 && value) {
            value[e] = s + vb[0];
        }
    }
    if (lane == 0 && noise && logp) logp[e] = lp - 0.9189385332046727f * (float)A;
}

// ---------------------------------------------------------------- backward

// out[i] = sum over splits of part[z][i].  A workgroup sums 64 outputs, its
// wave w the splits w, w + 4, ... in order, then the four waves' sums in order:
// with one thread per output, a gradient of 35 thousand values in 256 slabs kept
// half the chip's CUs on chains of 256 dependent loads (65 us; 10 us like this).
__global__ __launch_bounds__(256) void k_sum_parts(const float *__restrict__ part, int splits, int64_t n,
                                                   float *__restrict__ out)
{
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 64 + lane;
    float v = 0.0f;
    if (i < n) {
#pragma unroll 8
        for (int z = wave; z < splits; z += 4) v += part[(size_t)z * n + i];
    }
    red[wave][lane] = v;
    __syncthreads();
    if (wave == 0 && i < n) out[i] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// The PPO loss of sample s (one wave): the heads from h4 and the joint angles,
// logp of the taken action, the ratio to the behaviour policy's, the clipped
// surrogate and the value error.  Writes per sample: gm [A] = dL/dmean,
// gls [A] = dL/dlog_std (without the entropy term), gv = dL/dV, the loss terms
// [3] (policy, value, 0), and d4 = bf16([h4 > 0] (gm W_a + gv w_v)) over the
// 512 features.  L is the mean over S samples.
__global__ __launch_bounds__(256) void k_ppo_heads(const uint16_t *__restrict__ h, const float *__restrict__ state,
                                                   const float *__restrict__ aw, const float *__restrict__ ab,
                                                   const float *__restrict__ vw, const float *__restrict__ vb,
                                                   const float *__restrict__ log_std, int A, int S,
                                                   const float *__restrict__ actions, const float *__restrict__ old_logp,
                                                   const float *__restrict__ adv, const float *__restrict__ ret,
                                                   float clip, float vcoef, float *__restrict__ gm,
                                                   float *__restrict__ gls, float *__restrict__ gv,
                                                   float *__restrict__ terms, uint16_t *__restrict__ d4)
{
    const int lane = threadIdx.x & 63;
    const int e = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)threadIdx.x / 64);
    if (e >= S) return;
    constexpr int F = kPolicyFeat + kPolicyProprio;
    constexpr int NF = (F + 63) / 64;
    float f[NF];
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const int k = lane + 64 * i;
        f[i] = k < kPolicyFeat ? bf2f(h[(size_t)e * kPolicyFeat + k])
                               : (k < F ? state[(size_t)e * 10 + 3 + (k - kPolicyFeat)] : 0.0f);
    }
    float zs[kPolicyMaxAct];
    float logp = 0.0f, V = 0.0f;
    for (int a = 0; a <= A; ++a) {
        const float *w = a < A ? aw + (size_t)a * F : vw;
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const int k = lane + 64 * i;
            if (k < F) sum += w[k] * f[i];
        }
        for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
        if (a < A) {
            const float mean = sum + ab[a];
            const float z = (actions[(size_t)e * A + a] - mean) / expf(log_std[a]);
            zs[a] = z;
            logp += -0.5f * z * z - log_std[a];
        } else {
            V = sum + vb[0];
        }
    }
    logp -= 0.9189385332046727f * (float)A;
    const float r = expf(logp - old_logp[e]);
    const float Ad = adv[e];
    const float rc = fminf(fmaxf(r, 1.0f - clip), 1.0f + clip);
    const float s1 = r * Ad, s2 = rc * Ad;
    const bool use1 = s1 <= s2;
    const float invS = 1.0f / (float)S;
    const float dlogp = use1 ? -Ad * r * invS : 0.0f;
    const float dv = vcoef * 2.0f * (V - ret[e]) * invS;
    float g_mean[kPolicyMaxAct];
    for (int a = 0; a < A; ++a) {
        g_mean[a] = dlogp * zs[a] / expf(log_std[a]);
        if (lane == 0) {
            gm[(size_t)e * A + a] = g_mean[a];
            gls[(size_t)e * A + a] = dlogp * (zs[a] * zs[a] - 1.0f);
        }
    }
    if (lane == 0) {
        gv[e] = dv;
        terms[(size_t)e * 3 + 0] = -(use1 ? s1 : s2);
        terms[(size_t)e * 3 + 1] = (V - ret[e]) * (V - ret[e]);
        terms[(size_t)e * 3 + 2] = r;
    }
#pragma unroll
    for (int i = 0; i < NF; ++i) {
        const int k = lane + 64 * i;
        if (k < kPolicyFeat) {
            float df = dv * vw[k];
            for (int a = 0; a < A; ++a) df += g_mean[a] * aw[(size_t)a * F + k];
            d4[(size_t)e * kPolicyFeat + k] = f2bf(f[i] > 0.0f ? df : 0.0f);
        }
    }
}

// Gradients of the heads as sums over the samples, in chunks of kHeadChunk
// samples (one thread per output and chunk, the chunks then added in chunk
// order: deterministic).  Output i of a chunk: i < (A + 1) F the actor's
// W [A][F] then the critic's w [F] (gradient of the output times the
// feature), then the actor bias [A], log_std [A] (without the entropy term),
// the critic bias, and the three loss terms (policy, value, ratio).
constexpr int kHeadChunk = 512;
__global__ void k_ppo_head_part(const uint16_t *__restrict__ h, const float *__restrict__ state,
                                const float *__restrict__ gm, const float *__restrict__ gls,
                                const float *__restrict__ gv, const float *__restrict__ terms, int A, int S,
                                int nout, float *__restrict__ part)
{
    constexpr int F = kPolicyFeat + kPolicyProprio;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nout) return;
    const int e0 = blockIdx.y * kHeadChunk, e1 = min(S, e0 + kHeadChunk);
    const int nw = (A + 1) * F;
    float acc = 0.0f;
    if (i < nw) {
        const int a = i / F, k = i - a * F;
        for (int e = e0; e < e1; ++e) {
            const float fk = k < kPolicyFeat ? bf2f(h[(size_t)e * kPolicyFeat + k])
                                             : state[(size_t)e * 10 + 3 + (k - kPolicyFeat)];
            acc += (a < A ? gm[(size_t)e * A + a] : gv[e]) * fk;
        }
    } else if (i < nw + A) {
        const int a = i - nw;
        for (int e = e0; e < e1; ++e) acc += gm[(size_t)e * A + a];
    } else if (i < nw + 2 * A) {
        const int a = i - nw - A;
        for (int e = e0; e < e1; ++e) acc += gls[(size_t)e * A + a];
    } else if (i == nw + 2 * A) {
        for (int e = e0; e < e1; ++e) acc += gv[e];
    } else {
        const int t = i - nw - 2 * A - 1;
        for (int e = e0; e < e1; ++e) acc += terms[(size_t)e * 3 + t];
    }
    part[(size_t)blockIdx.y * nout + i] = acc;
}

// The summed head outputs into the gradient vector and the statistics [4] =
// mean policy loss, mean value error, entropy, mean ratio.
__global__ void k_ppo_head_finish(const float *__restrict__ sum, const float *__restrict__ log_std, int A, int S,
                                  float ecoef, float *__restrict__ g_aw, float *__restrict__ g_ab,
                                  float *__restrict__ g_vw, float *__restrict__ g_vb, float *__restrict__ g_ls,
                                  float *__restrict__ stats)
{
    constexpr int F = kPolicyFeat + kPolicyProprio;
    const int nw = (A + 1) * F;
    for (int i = threadIdx.x; i < nw + 2 * A + 1; i += blockDim.x) {
        const float v = sum[i];
        if (i < A * F) g_aw[i] = v;
        else if (i < nw) g_vw[i - A * F] = v;
        else if (i < nw + A) g_ab[i - nw] = v;
        else if (i < nw + 2 * A) g_ls[i - nw - A] = v - ecoef;
        else g_vb[0] = v;
    }
    if (threadIdx.x == 0 && stats) {
        float ent = 0.0f;
        for (int a = 0; a < A; ++a) ent += log_std[a] + 1.4189385332046727f;
        const float *t = sum + nw + 2 * A + 1;
        stats[0] = t[0] / (float)S;
        stats[1] = t[1] / (float)S;
        stats[2] = ent;
        stats[3] = t[2] / (float)S;
    }
}

// Column sums of a BF16 [rows][D] matrix in chunks of `per` rows: part
// [chunk][D] (one thread per column; the chunks are summed in order after).
__global__ void k_colsum_chunks(const uint16_t *__restrict__ g, int rows, int D, int per, float *__restrict__ part)
{
    const int c = threadIdx.x, chunk = blockIdx.x;
    if (c >= D) return;
    const int r0 = chunk * per, r1 = min(rows, r0 + per);
    float acc = 0.0f;
    for (int r = r0; r < r1; ++r) acc += bf2f(g[(size_t)r * D + c]);
    part[(size_t)chunk * D + c] = acc;
}

// The fully connected layer from split-K partial products: out[m][n] =
// bf16(relu(sum over splits in order of part[z][m][n] + b[n])).
__global__ void k_fc_finish(const float *__restrict__ part, int splits, int M, int N, const float *__restrict__ bias,
                            uint16_t *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t n_all = (int64_t)M * N;
    if (i >= n_all) return;
    float v = part[i];
    for (int z = 1; z < splits; ++z) v += part[(size_t)z * n_all + i];
    v += bias[i % N];
    out[i] = f2bf(v > 0.f ? v : 0.f);
}

// Generalised advantage estimation, one thread per env, backwards in time.
__global__ void k_gae(const float *__restrict__ rew, const float *__restrict__ val, const uint8_t *__restrict__ done,
                      const float *__restrict__ last, int T, int N, float gamma, float lam, float *__restrict__ adv,
                      float *__restrict__ ret)
{
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float nv = last[n], na = 0.0f;
    for (int t = T - 1; t >= 0; --t) {
        const size_t i = (size_t)t * N + n;
        const float live = done[i] ? 0.0f : 1.0f;
        const float delta = (rew[i] + gamma * nv * live) - val[i];
        na = delta + gamma * lam * live * na;
        adv[i] = na;
        ret[i] = na + val[i];
        nv = val[i];
    }
}

}  // namespace

hipError_t sum_parts(const float *part, int splits, int64_t n, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_sum_parts, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, s, part, splits, n, out);
    return hipGetLastError();
}

hipError_t colsum(const uint16_t *g, int rows, int D, float *part, size_t part_floats, float *out, hipStream_t s)
{
    if (rows <= 0) return hipMemsetAsync(out, 0, sizeof(float) * D, s);
    // about 256 chunks of at least 64 rows
    const int per = std::max(64, (rows + 255) / 256);
    const int chunks = (rows + per - 1) / per;
    if ((size_t)chunks * D > part_floats || D > 1024) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_colsum_chunks, dim3(chunks), dim3((D + 63) / 64 * 64), 0, s, g, rows, D, per, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return sum_parts(part, chunks, D, out, s);
}

hipError_t ppo_heads(const uint16_t *h, const float *state, const float *aw, const float *ab, const float *vw,
                     const float *vb, const float *log_std, int A, int S, const float *actions, const float *old_logp,
                     const float *adv, const float *ret, float clip, float vcoef, float *gm, float *gls, float *gv,
                     float *terms, uint16_t *d4, hipStream_t s)
{
    if (S <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ppo_heads, dim3((S + 3) / 4), dim3(256), 0, s, h, state, aw, ab, vw, vb, log_std, A, S,
                       actions, old_logp, adv, ret, clip, vcoef, gm, gls, gv, terms, d4);
    return hipGetLastError();
}

hipError_t ppo_head_grads(const uint16_t *h, const float *state, const float *gm, const float *gls, const float *gv,
                          const float *terms, const float *log_std, int A, int S, float ecoef, float *g_aw,
                          float *g_ab, float *g_vw, float *g_vb, float *g_ls, float *stats, float *part,
                          size_t part_floats, hipStream_t s)
{
    if (S <= 0) return hipErrorInvalidValue;
    const int nout = (A + 1) * (kPolicyFeat + kPolicyProprio) + 2 * A + 1 + 3;
    const int chunks = (S + kHeadChunk - 1) / kHeadChunk;
    if ((size_t)(chunks + 1) * nout > part_floats) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ppo_head_part, dim3((nout + 255) / 256, chunks), dim3(256), 0, s, h, state, gm, gls, gv,
                       terms, A, S, nout, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    float *sum = part + (size_t)chunks * nout;
    if ((e = sum_parts(part, chunks, nout, sum, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_ppo_head_finish, dim3(1), dim3(256), 0, s, sum, log_std, A, S, ecoef, g_aw, g_ab, g_vw,
                       g_vb, g_ls, stats);
    return hipGetLastError();
}

hipError_t gae(const float *rew, const float *val, const uint8_t *done, const float *last, int T, int N, float gamma,
               float lam, float *adv, float *ret, hipStream_t s)
{
    if (N <= 0 || T <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gae, dim3((N + 255) / 256), dim3(256), 0, s, rew, val, done, last, T, N, gamma, lam, adv, ret);
    return hipGetLastError();
}

int fc_splits(int rows, int N, int K)
{
    const int tiles = ((rows + 63) / 64) * ((N + 63) / 64);
    int splits = 512 / std::max(tiles, 1);              // about 512 workgroups
    splits = std::min(splits, K / 512);                 // at least 512 columns of K each
    return std::max(splits, 1);
}

hipError_t fc_forward(const uint16_t *x, const uint16_t *W, const float *bias, int rows, int N, int K, float *ws,
                      size_t ws_floats, uint16_t *out, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    const int splits = fc_splits(rows, N, K);
    if (splits == 1 || !ws || (size_t)splits * rows * N > ws_floats)
        return mlp_gemm(kGemmFwd, x, W, rows, N, K, K, K, bias, nullptr, 0, nullptr, out, N, s);
    hipError_t e = mlp_gemm_parts(x, W, rows, N, K, K, K, splits, ws, s);
    if (e != hipSuccess) return e;
    const int64_t n = (int64_t)rows * N;
    hipLaunchKernelGGL(k_fc_finish, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ws, splits, rows, N, bias, out);
    return hipGetLastError();
}

hipError_t policy_heads(const uint16_t *h, const float *state, const float *aw, const float *ab, const float *vw,
                        const float *vb, const float *log_std, int A, int n_envs, const float *noise,
                        float *actions, float *value, float *logp, hipStream_t s)
{
    if (n_envs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_policy_heads, dim3((n_envs + 3) / 4), dim3(256), 0, s, h, state, aw, ab, vw, vb, log_std,
                       A, n_envs, noise, actions, value, logp);
    return hipGetLastError();
}

}  // namespace gal
