// The surrogate's training pass around its large GEMMs: everything between the
// first layer's output and the weight gradients, a tile of rows at a time, with
// the activations in LDS: layers 2..4, the logit, the weighted logistic loss and
// the gradients of all four layers' pre-activations.  The weights of the six
// 256 x 256 products stream from L2 into registers, the next product's while the
// current one runs; that stream (786 KB per workgroup, 12 TB/s over the chip for
// 4096 rows) is what bounds it.  As separate launches (three forward GEMMs, head,
// loss, head gradient, three input gradients) the same work took 55 us of kernels
// for 4096 rows, now 16.
//
// A layer's weights are the A operand (rows permuted so that a lane holds 8
// consecutive columns of one row), 16 rows of activations the B operand.  Sums
// run over ascending 32-wide steps of k, as in the GEMMs.
#include "gal_internal.h"
#include "gal_mlp.h"

#include <algorithm>

namespace gal {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t quad __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int D = kMlpHidden;
constexpr int kSteps = D / 32;
constexpr int kPitch = D + 8;    // LDS row pitch (BF16 values)
constexpr int kLayer = D * D;    // one layer's weights
constexpr int kHeadSlab = D + 2; // per workgroup: the logit's weight gradient, bias gradient, loss

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Sum over the wave by a butterfly, in every lane (the inference head's order).
__device__ __forceinline__ float wave_sum(float v)
{
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// The row (output unit of the product) that fragment row r of block j of wave w holds.
__host__ __device__ constexpr int frag_row(int w, int j, int r) { return 32 * w + 8 * (r >> 2) + 4 * j + (r & 3); }

typedef bf16x8 Frags[kSteps][2];   // a wave's 32 output columns of one product

__device__ __forceinline__ void load_frags(const uint16_t *w, int wave, int lane, Frags &f)
{
    // (opaque: a load may not move up over the product before it, where there
    // are no registers for a third set)
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            f[st][j] = __builtin_bit_cast(
                bf16x8, *reinterpret_cast<const quad *>(w + (size_t)(((wave * kSteps + st) * 2 + j) * 64 + lane) * 8));
}

// acc[m][j]: rows 16 m + lane % 16, columns 32 wave + 8 (lane / 16) + 4 j + 0..3
template <int M>
__device__ __forceinline__ void product(const uint16_t (*X)[kPitch], const Frags &f, int lane, floatx4 (&acc)[M][2])
{
    const int r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m][0] = acc[m][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < kSteps; ++st)
#pragma unroll
        for (int m = 0; m < M; ++m) {
            const bf16x8 x = __builtin_bit_cast(bf16x8, *reinterpret_cast<const quad *>(&X[16 * m + r][32 * st + 8 * g]));
            acc[m][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[st][0], x, acc[m][0], 0, 0, 0);
            acc[m][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[st][1], x, acc[m][1], 0, 0, 0);
        }
}

template <int R>
__global__ __launch_bounds__(kThreads, 2) void k_mlp_mid(MlpMidArgs p)
{
    constexpr int M = R / 16;
    __shared__ __attribute__((aligned(16))) uint16_t H[4][R][kPitch];   // h1..h4
    __shared__ __attribute__((aligned(16))) uint16_t G[2][R][kPitch];   // pre-activation gradients
    __shared__ float ys[R], dzs[R], losses[R];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, col = 32 * wave + 8 * (lane >> 4);
    float head = 0.f;   // thread j < 256: the logit's weight gradient j; 256: its bias gradient; 257: the loss
    // loaded before the weight stream: loads complete in order, and a bias read in
    // the middle of it waits for the weights behind which it was issued
    floatx4 bias[3][2];
#pragma unroll
    for (int l = 0; l < 3; ++l)
#pragma unroll
        for (int j = 0; j < 2; ++j) bias[l][j] = *reinterpret_cast<const floatx4 *>(p.b[l] + col + 4 * j);
    float w5[D / 64];
#pragma unroll
    for (int k = 0; k < D / 64; ++k) w5[k] = bf2f(p.w5[lane + 64 * k]);
    const shortx8 w5c = *reinterpret_cast<const shortx8 *>(p.w5 + 8 * (tid & 31));
    const float b5 = p.b5[0];
    const int tiles = (p.rows + R - 1) / R;
    for (int t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int row0 = t * R;
        if (tid < R) ys[tid] = p.y[min(row0 + tid, p.rows - 1)];
        Frags fa, fb;
        load_frags(p.wf, wave, lane, fa);
        // 16-byte pieces of the tile: row i / 32, columns 8 (i % 32) ..
#pragma unroll
        for (int i = tid; i < R * 32; i += kThreads)
            *reinterpret_cast<quad *>(&H[0][i >> 5][8 * (i & 31)]) =
                *reinterpret_cast<const quad *>(p.h1 + (size_t)min(row0 + (i >> 5), p.rows - 1) * D + 8 * (i & 31));
        load_frags(p.wf + kLayer, wave, lane, fb);
        __syncthreads();
        // H[l + 1] = relu(H[l] W^T + b), to memory too where out is given
        auto forward = [&](const Frags &f, int l, uint16_t *out) {
            floatx4 acc[M][2];
            product<M>(H[l], f, lane, acc);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const floatx4 v0 = acc[m][0] + bias[l][0], v1 = acc[m][1] + bias[l][1];
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)fmaxf(e < 4 ? v0[e & 3] : v1[e & 3], 0.f);
                const int r = 16 * m + r16;
                *reinterpret_cast<bf16x8 *>(&H[l + 1][r][col]) = o;
                if (out && row0 + r < p.rows) *reinterpret_cast<bf16x8 *>(out + (size_t)(row0 + r) * D + col) = o;
            }
        };
        // G[b ^ 1] = [H[l] > 0] G[b] W, to memory too
        auto backward = [&](const Frags &f, int b, int l, uint16_t *out) {
            floatx4 acc[M][2];
            product<M>(G[b], f, lane, acc);
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const int r = 16 * m + r16;
                const shortx8 h = *reinterpret_cast<const shortx8 *>(&H[l][r][col]);
                bf16x8 o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (__bf16)(h[e] > 0 ? (e < 4 ? acc[m][0][e & 3] : acc[m][1][e & 3]) : 0.f);
                *reinterpret_cast<bf16x8 *>(&G[b ^ 1][r][col]) = o;
                if (row0 + r < p.rows) *reinterpret_cast<bf16x8 *>(out + (size_t)(row0 + r) * D + col) = o;
            }
        };
        forward(fa, 0, p.h2);
        load_frags(p.wf + 2 * kLayer, wave, lane, fa);
        __syncthreads();
        forward(fb, 1, p.h3);
        load_frags(p.wt + 2 * kLayer, wave, lane, fb);
        __syncthreads();
        forward(fa, 2, nullptr);
        load_frags(p.wt + kLayer, wave, lane, fa);
        __syncthreads();
        // ---- the logit, the loss and its gradient: R / 8 rows per wave
#pragma unroll
        for (int i = 0; i < R / kWaves; ++i) {
            const int r = (R / kWaves) * wave + i;
            float z = 0.f;
#pragma unroll
            for (int k = 0; k < D / 64; ++k) z += bf2f(H[3][r][lane + 64 * k]) * w5[k];
            z = wave_sum(z) + b5;
            float dz = 0.f, l = 0.f;
            if (row0 + r < p.rows) {
                const float y = ys[r];
                const float w = y > 0.5f ? p.pos_w : 1.f;
                const float q = 1.f / (1.f + expf(-z));
                dz = w * (q - y) / (float)p.rows;
                l = w * ((z > 0.f ? z : 0.f) - z * y + log1pf(expf(-fabsf(z)))) / (float)p.rows;
            }
            if (lane == 0) {
                dzs[r] = dz;
                losses[r] = l;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = tid; i < R * 32; i += kThreads) {
            const int r = i >> 5, c = 8 * (i & 31);
            const shortx8 h = *reinterpret_cast<const shortx8 *>(&H[3][r][c]);
            const float dz = dzs[r];
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)(h[e] > 0 ? dz * bf2f((uint16_t)w5c[e]) : 0.f);
            *reinterpret_cast<bf16x8 *>(&G[0][r][c]) = o;
            if (row0 + r < p.rows) *reinterpret_cast<bf16x8 *>(p.dp[3] + (size_t)(row0 + r) * D + c) = o;
        }
        if (tid < D) {
            if (row0 + R <= p.rows) {
#pragma unroll
                for (int r = 0; r < R; ++r) head += dzs[r] * bf2f(H[3][r][tid]);
            } else {   // (rows past the last repeat it, and may be infinite)
                for (int r = 0; row0 + r < p.rows; ++r) head += dzs[r] * bf2f(H[3][r][tid]);
            }
        } else if (tid < D + 2) {
            const float *v = tid == D ? dzs : losses;
            for (int r = 0; r < R; ++r) head += v[r];
        }
        __syncthreads();
        backward(fb, 0, 2, p.dp[2]);
        load_frags(p.wt, wave, lane, fb);
        __syncthreads();
        backward(fa, 1, 1, p.dp[1]);
        __syncthreads();
        backward(fb, 0, 0, p.dp[0]);
        __syncthreads();
    }
    if (tid < kHeadSlab) p.part[(size_t)blockIdx.x * kHeadSlab + tid] = head;
}

// The copies of layers 2..4 that k_mlp_mid reads (w: three row-major [out][in]
// matrices): wf for the forward products, wt (transposed) for the gradients, in
// the order of the fragments, so that a wave's load is one block of 1 KB.
__global__ void k_mid_layout(const uint16_t *__restrict__ w1, const uint16_t *__restrict__ w2,
                             const uint16_t *__restrict__ w3, uint16_t *__restrict__ wf, uint16_t *__restrict__ wt)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;   // one fragment piece of 8 values
    if (i >= 6 * kLayer / 8) return;
    const int dir = i / (3 * kLayer / 8), at = i - dir * (3 * kLayer / 8);
    const int layer = at / (kLayer / 8), q = at - layer * (kLayer / 8);
    const uint16_t *w = layer == 0 ? w1 : layer == 1 ? w2 : w3;
    const int lane = q & 63, j = (q >> 6) & 1, st = (q >> 7) % kSteps, wave = (q >> 7) / kSteps;
    const int n = frag_row(wave, j, lane & 15), k = 32 * st + 8 * (lane >> 4);
    uint16_t v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = dir ? w[(size_t)(k + e) * D + n] : w[(size_t)n * D + k + e];
    quad o;
    memcpy(&o, v, 16);
    *reinterpret_cast<quad *>((dir ? wt : wf) + (size_t)at * 8) = o;
}

// The gradient vector from its sums' parts, four values per thread: [i0, n) the
// splits' slabs of n values in order, then (the last workgroups) the logit's
// slabs; into g and, where given, grads, the loss into loss and loss_out.
__global__ __launch_bounds__(256) void k_grad_sum(const float *__restrict__ part, int splits, int64_t i0, int64_t n,
                                                  int blocks, const float *__restrict__ hpart, int hslabs,
                                                  float *__restrict__ g, float *__restrict__ grads,
                                                  float *__restrict__ loss, float *__restrict__ loss_out)
{
    __shared__ float red[4][64];
    if ((int)blockIdx.x < blocks) {
        const int64_t i = i0 + ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
        if (i >= n) return;
        floatx4 v = *reinterpret_cast<const floatx4 *>(part + i);
        for (int z = 1; z < splits; ++z) v += *reinterpret_cast<const floatx4 *>(part + (size_t)z * n + i);
        *reinterpret_cast<floatx4 *>(g + i) = v;
        if (grads) {
#pragma unroll
            for (int e = 0; e < 4; ++e) grads[i + e] = v[e];
        }
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = ((int)blockIdx.x - blocks) * 64 + lane;
    float v = 0.f;
    if (i < kHeadSlab) {
#pragma unroll 8
        for (int z = wave; z < hslabs; z += 4) v += hpart[(size_t)z * kHeadSlab + i];
    }
    red[wave][lane] = v;
    __syncthreads();
    if (wave != 0 || i >= kHeadSlab) return;
    v = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    if (i <= D) {
        g[n + i] = v;
        if (grads) grads[n + i] = v;
    } else {
        loss[0] = v;
        if (loss_out) loss_out[0] = v;
    }
}

constexpr int kMidGrid = 512;   // workgroups at most (each one slab of the logit's sums)

}  // namespace

size_t mlp_mid_weights() { return (size_t)3 * kLayer; }
size_t mlp_mid_part_floats() { return (size_t)kMidGrid * kHeadSlab; }

hipError_t mlp_mid_layout(const uint16_t *w1, const uint16_t *w2, const uint16_t *w3, uint16_t *wf, uint16_t *wt,
                          hipStream_t s)
{
    hipLaunchKernelGGL(k_mid_layout, dim3(6 * kLayer / 8 / 256), dim3(256), 0, s, w1, w2, w3, wf, wt);
    return hipGetLastError();
}

hipError_t mlp_mid(const MlpMidArgs &a, int *slabs, hipStream_t s)
{
    if (a.rows <= 0) return hipErrorInvalidValue;
    // 16 rows per workgroup up to one workgroup per CU, then 32, which halve the
    // weights streamed per row.  The whole gradient with 16 and 32, us: 1024 rows
    // 41.3 and 45.4, 4096 49.4 and 52.9, 4112 61.5 and 54.7, 8192 71.9 and 62.7.
    const int R = a.rows <= 16 * 256 ? 16 : 32;
    const int grid = std::min((a.rows + R - 1) / R, kMidGrid);
    *slabs = grid;
    hipLaunchKernelGGL(R == 16 ? k_mlp_mid<16> : k_mlp_mid<32>, dim3(grid), dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t mlp_grad_sum(const float *part, int splits, int64_t i0, int64_t n, const float *hpart, int hslabs, float *g,
                        float *grads, float *loss, float *loss_out, hipStream_t s)
{
    if (i0 % 4 || n % 4 || i0 > n) return hipErrorInvalidValue;
    const int blocks = (int)(((n - i0) / 4 + 255) / 256);
    hipLaunchKernelGGL(k_grad_sum, dim3(blocks + (kHeadSlab + 63) / 64), dim3(256), 0, s, part, splits, i0, n, blocks,
                       hpart, hslabs, g, grads, loss, loss_out);
    return hipGetLastError();
}

}  // namespace gal
