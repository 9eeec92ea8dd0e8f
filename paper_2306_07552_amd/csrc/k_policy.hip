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

constexpr int kF = kPolicyFeat + kPolicyProprio;   // inputs of the heads: features, joint angles
constexpr int kNF = (kF + 63) / 64;                // values of f per lane: k = lane + 64 i

// Lane l of a row of 16 receives lane (l - n) mod 16's value.
template <int kN>
__device__ __forceinline__ float row_rotate(float v)
{
    const int b = __float_as_int(v);
    return __int_as_float(__builtin_amdgcn_update_dpp(b, b, 0x120 + kN, 0xF, 0xF, false));
}

// Sum over the wave in the order of a butterfly (partners 32, 16, 8, 4, 2, 1
// lanes away), in every lane.  Swapping wave halves and rows, then rotating
// within a row, brings the same partners together without LDS: once lanes 8
// apart agree, the lane 4 places round the row holds the sum of the lane 4 away,
// and so on.  (Six LDS shuffles per head were most of a head's time.)
__device__ __forceinline__ float wave_sum(float v)
{
    uint32_t b = __float_as_uint(v);
    const auto h = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    v = __uint_as_float(h[0]) + __uint_as_float(h[1]);
    b = __float_as_uint(v);
    const auto q = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    v = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    return v + row_rotate<1>(v);
}

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// The heads' inputs of sample e: the BF16 features (from the fully connected
// layer's split partial products, added in order with bias and ReLU and written
// to h, or from h itself) and the joint angles.
__device__ __forceinline__ void head_inputs(const FcParts &fc, uint16_t *h, const float *state, int e, int lane,
                                            float (&f)[kNF])
{
    constexpr int kN = kPolicyFeat / 64;
    const size_t at = (size_t)e * kPolicyFeat + lane;
    f[kN] = lane < kPolicyProprio ? state[(size_t)e * 10 + 3 + lane] : 0.0f;
    if (fc.splits == 1) {
#pragma unroll
        for (int i = 0; i < kN; ++i) f[i] = bf2f(h[at + 64 * i]);
        return;
    }
    // all of a split's loads (and two splits') are in flight together
    const float *__restrict__ part = fc.part + at;
#pragma unroll
    for (int i = 0; i < kN; ++i) f[i] = part[64 * i];
#pragma unroll 2
    for (int z = 1; z < fc.splits; ++z) {
        part += fc.stride;
        float v[kN];
#pragma unroll
        for (int i = 0; i < kN; ++i) v[i] = part[64 * i];
#pragma unroll
        for (int i = 0; i < kN; ++i) f[i] += v[i];
    }
    uint16_t b[kN];
#pragma unroll
    for (int i = 0; i < kN; ++i) {
        const float v = f[i] + fc.bias[lane + 64 * i];
        b[i] = f2bf(v > 0.f ? v : 0.f);
        f[i] = bf2f(b[i]);
    }
#pragma unroll
    for (int i = 0; i < kN; ++i) h[at + 64 * i] = b[i];
}

// out[s] of lane a (0..A): head a's sum over k of w[k] f_k for sample s (FP32,
// lane-strided partial sums, then wave_sum), the critic as head A; four heads at
// a time, so that their loads and sums overlap.
template <int kS>
__device__ __forceinline__ void head_sums(const float *__restrict__ aw, const float *__restrict__ vw, int A,
                                          const float (&f)[kS][kNF], int lane, float (&out)[kS])
{
#pragma unroll
    for (int s = 0; s < kS; ++s) out[s] = 0.0f;
    for (int a0 = 0; a0 <= A; a0 += 4) {
        float sum[4][kS], w[4][kNF];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int a = min(a0 + j, A);
            const float *wa = a < A ? aw + (size_t)a * kF : vw;
#pragma unroll
            for (int i = 0; i < kNF; ++i) w[j][i] = wa[min(lane + 64 * i, kF - 1)];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < kS; ++s) {
                float v = 0.0f;
#pragma unroll
                for (int i = 0; i < kNF; ++i) {
                    const float t = w[j][i] * f[s][i];
                    v += i < kNF - 1 || lane < kPolicyProprio ? t : 0.0f;
                }
                sum[j][s] = v;
            }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < kS; ++s) {
                const float v = wave_sum(sum[j][s]);
                if (lane == a0 + j) out[s] = v;
            }
    }
}

// The heads of env e (one wave): mean_a = b_a + sum_k W_a[k] f_k, value = b_v +
// sum_k w_v[k] f_k; the action mean + std * noise and its Gaussian log-density
// sum_a (-noise_a^2 / 2 - log_std_a) - A log(2 pi) / 2 (noise null: the mean, no
// log-density).  Lane a holds head a.
__global__ __launch_bounds__(256) void k_policy_heads(FcParts fc, uint16_t *__restrict__ h,
                                                      const float *__restrict__ state,
                                                      const float *__restrict__ aw, const float *__restrict__ ab,
                                                      const float *__restrict__ vw, const float *__restrict__ vb,
                                                      const float *__restrict__ log_std, int A, int n_envs,
                                                      const float *__restrict__ noise, float *__restrict__ actions,
                                                      float *__restrict__ value, float *__restrict__ logp)
{
    const int lane = threadIdx.x & 63;
    const int e = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + (int)threadIdx.x / 64);
    if (e >= n_envs) return;
    float f[1][kNF], sum[1];
    head_inputs(fc, h, state, e, lane, f[0]);
    head_sums<1>(aw, vw, A, f, lane, sum);
    float term = 0.0f;
    if (lane < A) {
        const float mean = sum[0] + ab[lane];
        float act = mean;
        if (noise) {
            const float z = noise[(size_t)e * A + lane], ls = log_std[lane];
            act = mean + expf(ls) * z;
            term = -0.5f * z * z - ls;
        }
        actions[(size_t)e * A + lane] = act;
    } else if (lane == A && value) {
        value[e] = sum[0] + vb[0];
    }
    if (noise && logp) {
        float lp = 0.0f;
        for (int a = 0; a < A; ++a) lp += lane_value(term, a);
        if (lane == 0) logp[e] = lp - 0.9189385332046727f * (float)A;
    }
}

// ---------------------------------------------------------------- backward

// out[i] = sum over splits of part[z][i].  A workgroup sums 64 outputs, its
// wave w the splits w, w + 4, ... in order, then the four waves' sums in order:
// with one thread per output, a gradient of 35 thousand values in 256 slabs kept
// half the chip's CUs on chains of 256 dependent loads (65 us; 7 us like this).
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

// The PPO loss of kHeadSamples samples per wave (each weight is loaded once for
// all of them): the heads from the features and the joint angles, logp of the
// taken action, the ratio to the behaviour policy's, the clipped surrogate and
// the value error.  Writes per sample a row of 2 A + 4 values (dL/dmean [A],
// dL/dlog_std [A] without the entropy term, dL/dV, the loss terms: policy, value,
// ratio) and d4 = bf16([h4 > 0] (gm W_a + gv w_v)) over the 512 features.  L is
// the mean over S samples.  Measured, 32,768 samples: 140 us at one sample per
// wave with LDS shuffles, 50 us at four like this.
template <int kHeadSamples>
__global__ __launch_bounds__(256) void k_ppo_heads(FcParts fc, uint16_t *__restrict__ h,
                                                   const float *__restrict__ state,
                                                   const float *__restrict__ aw, const float *__restrict__ ab,
                                                   const float *__restrict__ vw, const float *__restrict__ vb,
                                                   const float *__restrict__ log_std, int A, int S,
                                                   const float *__restrict__ actions, const float *__restrict__ old_logp,
                                                   const float *__restrict__ adv, const float *__restrict__ ret,
                                                   float clip, float vcoef, float *__restrict__ rows,
                                                   uint16_t *__restrict__ d4)
{
    const int lane = threadIdx.x & 63;
    const int e0 = __builtin_amdgcn_readfirstlane(((int)blockIdx.x * 4 + (int)threadIdx.x / 64) * kHeadSamples);
    if (e0 >= S) return;
    float f[kHeadSamples][kNF], sum[kHeadSamples];
#pragma unroll
    for (int s = 0; s < kHeadSamples; ++s) head_inputs(fc, h, state, min(e0 + s, S - 1), lane, f[s]);
    head_sums<kHeadSamples>(aw, vw, A, f, lane, sum);
    const bool head = lane < A;
    const float ls = head ? log_std[lane] : 0.0f, std = expf(ls), bias = head ? ab[lane] : 0.0f;
    const float invS = 1.0f / (float)S;
    float g_mean[kHeadSamples], dv[kHeadSamples];
#pragma unroll
    for (int s = 0; s < kHeadSamples; ++s) {
        const int e = min(e0 + s, S - 1);
        const float z = head ? (actions[(size_t)e * A + lane] - (sum[s] + bias)) / std : 0.0f;
        const float term = -0.5f * z * z - ls;
        float logp = 0.0f;
        for (int a = 0; a < A; ++a) logp += lane_value(term, a);
        logp -= 0.9189385332046727f * (float)A;
        const float V = lane_value(sum[s], A) + vb[0];
        const float r = expf(logp - old_logp[e]);
        const float Ad = adv[e];
        const float rc = fminf(fmaxf(r, 1.0f - clip), 1.0f + clip);
        const float s1 = r * Ad, s2 = rc * Ad;
        const bool use1 = s1 <= s2;
        const float dlogp = use1 ? -Ad * r * invS : 0.0f;
        dv[s] = vcoef * 2.0f * (V - ret[e]) * invS;
        g_mean[s] = dlogp * z / std;
        if (e0 + s < S) {
            float *row = rows + (size_t)e * (2 * A + 4);
            if (head) {
                row[lane] = g_mean[s];
                row[A + lane] = dlogp * (z * z - 1.0f);
            } else if (lane == A) {
                row[2 * A] = dv[s];
                row[2 * A + 1] = -(use1 ? s1 : s2);
                row[2 * A + 2] = (V - ret[e]) * (V - ret[e]);
                row[2 * A + 3] = r;
            }
        }
    }
    float df[kHeadSamples][kPolicyFeat / 64];
#pragma unroll
    for (int i = 0; i < kPolicyFeat / 64; ++i) {
        const float wk = vw[lane + 64 * i];
#pragma unroll
        for (int s = 0; s < kHeadSamples; ++s) df[s][i] = dv[s] * wk;
    }
    for (int a = 0; a < A; ++a) {
        float ga[kHeadSamples];
#pragma unroll
        for (int s = 0; s < kHeadSamples; ++s) ga[s] = lane_value(g_mean[s], a);
#pragma unroll
        for (int i = 0; i < kPolicyFeat / 64; ++i) {
            const float wk = aw[(size_t)a * kF + lane + 64 * i];
#pragma unroll
            for (int s = 0; s < kHeadSamples; ++s) df[s][i] += ga[s] * wk;
        }
    }
#pragma unroll
    for (int s = 0; s < kHeadSamples; ++s)
        if (e0 + s < S) {
#pragma unroll
            for (int i = 0; i < kPolicyFeat / 64; ++i)
                d4[(size_t)(e0 + s) * kPolicyFeat + lane + 64 * i] = f2bf(f[s][i] > 0.0f ? df[s][i] : 0.0f);
        }
}

// Sums over the samples: the heads' weight gradients (head gradient times
// feature), the fully connected layer's bias gradient (d4), and the sums of the
// per-sample rows.  A workgroup takes `per` samples, wave w every fourth of them,
// lane l the features 8 l .. 8 l + 7 of up to kHeadGroup heads (blockIdx.y: which),
// so that a feature is read once for all heads; its four waves' sums are added in
// order into slab blockIdx.x:
//   [A + 1][512] heads x features, [512] fc bias, [A + 1][7] heads x joint angles,
//   [2 A + 4] row sums.
// One thread per output over 512 samples took 366 us for 32,768 samples and 233
// for 2,000 (too few waves, each a chain of dependent loads); this 38 and 14.
constexpr int kHeadGroup = 12;
__host__ __device__ constexpr int head_slab(int A) { return (A + 1) * kF + kPolicyFeat + 2 * A + 4; }

__global__ __launch_bounds__(256) void k_ppo_head_part(const uint16_t *__restrict__ h, const float *__restrict__ state,
                                                       const float *__restrict__ rows,
                                                       const uint16_t *__restrict__ d4, int A, int S, int per,
                                                       float *__restrict__ part)
{
    __shared__ float red[4][kPolicyFeat];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int a0 = blockIdx.y * kHeadGroup, na = min(kHeadGroup, A + 1 - a0);
    const bool first = blockIdx.y == 0;
    const int e0 = blockIdx.x * per, e1 = min(S, e0 + per);
    const int nrow = 2 * A + 4, nq = (A + 1) * kPolicyProprio;
    float acc[kHeadGroup][8], accd[8], accq[4], accr[2];
#pragma unroll
    for (int j = 0; j < kHeadGroup; ++j)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[j][c] = 0.0f;
#pragma unroll
    for (int c = 0; c < 8; ++c) accd[c] = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) accq[c] = 0.0f;
    accr[0] = accr[1] = 0.0f;
#pragma unroll 2
    for (int e = e0 + wave; e < e1; e += 4) {
        const float *row = rows + (size_t)e * nrow;
        const uint4 q = *reinterpret_cast<const uint4 *>(h + (size_t)e * kPolicyFeat + 8 * lane);
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        float f[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) f[c] = __uint_as_float((c & 1) ? w[c >> 1] & 0xFFFF0000u : w[c >> 1] << 16);
#pragma unroll
        for (int j = 0; j < kHeadGroup; ++j) {
            // (past the last head: the critic's again, not stored)
            const float ga = row[a0 + j < A ? a0 + j : 2 * A];
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[j][c] += ga * f[c];
        }
        if (first) {
            const uint4 d = *reinterpret_cast<const uint4 *>(d4 + (size_t)e * kPolicyFeat + 8 * lane);
            const uint32_t v[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int c = 0; c < 8; ++c)
                accd[c] += __uint_as_float((c & 1) ? v[c >> 1] & 0xFFFF0000u : v[c >> 1] << 16);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = lane + 64 * c, a = i / kPolicyProprio;
                if (i < nq) accq[c] += row[a < A ? a : 2 * A] * state[(size_t)e * 10 + 3 + (i - a * kPolicyProprio)];
            }
#pragma unroll
            for (int c = 0; c < 2; ++c)
                if (lane + 64 * c < nrow) accr[c] += row[lane + 64 * c];
        }
    }
    float *slab = part + (size_t)blockIdx.x * head_slab(A);
    // the four waves' sums of n <= 512 values in red
    auto combine = [&](int n, float *dst) {
        __syncthreads();
        for (int i = tid; i < n; i += 256) dst[i] = ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
        __syncthreads();
    };
    auto put8 = [&](const float (&v)[8]) {
#pragma unroll
        for (int c = 0; c < 8; ++c) red[wave][8 * lane + c] = v[c];
    };
#pragma unroll
    for (int j = 0; j < kHeadGroup; ++j)
        if (j < na) {
            put8(acc[j]);
            combine(kPolicyFeat, slab + (size_t)(a0 + j) * kPolicyFeat);
        }
    if (!first) return;
    slab += (A + 1) * kPolicyFeat;
    put8(accd);
    combine(kPolicyFeat, slab);
#pragma unroll
    for (int c = 0; c < 4; ++c) red[wave][lane + 64 * c] = accq[c];
    combine(nq, slab + kPolicyFeat);
#pragma unroll
    for (int c = 0; c < 2; ++c) red[wave][lane + 64 * c] = accr[c];
    combine(nrow, slab + kPolicyFeat + nq);
}

// The slabs' sums (as in k_sum_parts) into the gradient vector and the
// statistics [4] = mean policy loss, mean value error, entropy, mean ratio.
__global__ __launch_bounds__(256) void k_ppo_head_sum(const float *__restrict__ part, int slabs,
                                                      const float *__restrict__ log_std, int A, int S, float ecoef,
                                                      HeadGrads g, float *__restrict__ stats)
{
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = head_slab(A);
    int i = blockIdx.x * 64 + lane;
    float v = 0.0f;
    if (i < n) {
#pragma unroll 8
        for (int z = wave; z < slabs; z += 4) v += part[(size_t)z * n + i];
    }
    red[wave][lane] = v;
    __syncthreads();
    if (wave != 0 || i >= n) return;
    v = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    if (i < (A + 1) * kPolicyFeat) {
        const int a = i / kPolicyFeat, k = i - a * kPolicyFeat;
        (a < A ? g.aw + (size_t)a * kF : g.vw)[k] = v;
        return;
    }
    i -= (A + 1) * kPolicyFeat;
    if (i < kPolicyFeat) {
        g.fcb[i] = v;
        return;
    }
    i -= kPolicyFeat;
    if (i < (A + 1) * kPolicyProprio) {
        const int a = i / kPolicyProprio, k = kPolicyFeat + i - a * kPolicyProprio;
        (a < A ? g.aw + (size_t)a * kF : g.vw)[k] = v;
        return;
    }
    i -= (A + 1) * kPolicyProprio;
    if (i < A) g.ab[i] = v;
    else if (i < 2 * A) g.ls[i - A] = v - ecoef;
    else if (i == 2 * A) g.vb[0] = v;
    else if (stats) {
        stats[i == 2 * A + 3 ? 3 : i - 2 * A - 1] = v / (float)S;
        if (i == 2 * A + 3) {
            float ent = 0.0f;
            for (int a = 0; a < A; ++a) ent += log_std[a] + 1.4189385332046727f;
            stats[2] = ent;
        }
    }
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

hipError_t ppo_heads(const FcParts &fc, uint16_t *h, const float *state, const float *aw, const float *ab,
                     const float *vw, const float *vb, const float *log_std, int A, int S, const float *actions,
                     const float *old_logp, const float *adv, const float *ret, float clip, float vcoef, float *rows,
                     uint16_t *d4, hipStream_t s)
{
    if (S <= 0) return hipSuccess;
    // four samples per wave share the weights' loads; up to 4096 samples one, as
    // the waves would not fill the chip.  From there both are within 0.5 %, four
    // ahead from 12,000.  The whole update with one and four, us: 2,000 samples 351
    // and 358, 4,096 586 and 595, 8,192 1062 and 1063, 12,000 1517 and 1511, 16,384
    // 2023 and 2013.
    const int per = S > 4096 ? 4 : 1;
    hipLaunchKernelGGL(per == 4 ? k_ppo_heads<4> : k_ppo_heads<1>, dim3((S + 4 * per - 1) / (4 * per)), dim3(256), 0, s,
                       fc, h, state, aw, ab, vw, vb, log_std, A, S, actions, old_logp, adv, ret, clip, vcoef, rows, d4);
    return hipGetLastError();
}

hipError_t ppo_head_grads(const uint16_t *h, const float *state, const float *rows, const uint16_t *d4,
                          const float *log_std, int A, int S, float ecoef, const HeadGrads &g, float *stats, float *part,
                          size_t part_floats, hipStream_t s)
{
    if (S <= 0) return hipErrorInvalidValue;
    // at most 256 slabs, of at least 32 samples (8 per wave)
    const int per = std::max(32, (S + 255) / 256);
    const int slabs = (S + per - 1) / per;
    if ((size_t)slabs * head_slab(A) > part_floats) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ppo_head_part, dim3(slabs, (A + kHeadGroup) / kHeadGroup), dim3(256), 0, s, h, state, rows, d4,
                       A, S, per, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ppo_head_sum, dim3((head_slab(A) + 63) / 64), dim3(256), 0, s, part, slabs, log_std, A, S,
                       ecoef, g, stats);
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
                      size_t ws_floats, uint16_t *out, FcParts *parts, hipStream_t s)
{
    *parts = FcParts{nullptr, 1, 0, bias};
    if (rows <= 0) return hipSuccess;
    const int splits = fc_splits(rows, N, K);
    if (splits == 1 || !ws || (size_t)splits * rows * N > ws_floats)
        return mlp_gemm(kGemmFwd, x, W, rows, N, K, K, K, bias, nullptr, 0, nullptr, out, N, s);
    *parts = FcParts{ws, splits, (int64_t)rows * N, bias};
    return mlp_gemm_parts(x, W, rows, N, K, K, K, splits, ws, s);
}

hipError_t policy_heads(const FcParts &fc, uint16_t *h, const float *state, const float *aw, const float *ab,
                        const float *vw, const float *vb, const float *log_std, int A, int n_envs, const float *noise,
                        float *actions, float *value, float *logp, hipStream_t s)
{
    if (n_envs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_policy_heads, dim3((n_envs + 3) / 4), dim3(256), 0, s, fc, h, state, aw, ab, vw, vb, log_std,
                       A, n_envs, noise, actions, value, logp);
    return hipGetLastError();
}

}  // namespace gal
