// The policy's convolutional encoder (the SimpleCNN of the appendix on model
// sizes: 8x8 stride 4, 4x4 stride 2, 3x3 stride 1, no padding, each with ReLU)
// as one persistent kernel: a workgroup takes one sample at a time through all
// three layers, each layer's map staying in LDS for the next one.
//
// What bounds it: memory traffic on large batches (a sample's 64 KB of depth in,
// 61.5 + 25 + 9 KB of maps out, which the backward pass and the activation
// readout need), the LDS reads of the second layer's windows on small ones.
// Layer by layer (three implicit GEMMs that read each map back) every map
// crossed memory twice and each layer had a launch of its own.  Measured, three
// kernels -> this one: 115 -> 47 us for 1024 samples, 3.65 -> 1.10 ms for 32,768
// (4.8 TB/s), 39 -> 18 us for 30.
//
// A layer is one GEMM per sample with the weights as the A operand of
// v_mfma_f32_16x16x32_bf16 and 16 output pixels as the B operand: a lane then
// holds consecutive output channels of one pixel, so that the ReLU output
// leaves in 16-byte stores (LDS and memory).  The sum over k of every output
// runs over ascending 32-wide steps of (ky, kx, channel) in FP32, bias after.
#include "gal_internal.h"
#include "gal_policy.h"

#include <algorithm>

namespace gal {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512, kWaves = kThreads / 64;
constexpr int kRes = kPolicyRes;
constexpr int kPitch = kRes + 4;             // BF16 image row pitch in LDS
constexpr int kS1 = 31, kS2 = 14, kS3 = 12;  // map edges
constexpr int kC1 = 32, kC2 = 64, kC3 = 32;  // channels
constexpr int kK2 = 16 * kC1, kK3 = 9 * kC2;
constexpr int kQuads = kRes * kRes / 8 / kThreads;   // 16-byte loads per thread of half an image

// LDS of a workgroup.  h1: rows of 32 pixel columns, even columns first (a
// stride-2 window then reads consecutive columns), 4 slots of 8 channels per
// pixel; h2: 8 slots per pixel.  The slot index is XORed with bits of the
// pixel's position, so that lanes reading one slot of consecutive pixels fall in
// different banks.
struct EncLds {
    uint16_t img[kRes * kPitch];
    uint4 h1[kS1 * 32 * 4];
    uint4 h2[kS2 * kS2 * 8];
    uint4 w1[4 * 64];      // layer 1 weight fragments [channel half][k step][lane]
    uint4 w3[2 * 18 * 64]; // layer 3 weight fragments [16 channels][k step][lane]
    float bias[kC1 + kC2 + kC3];
};

// x = d / (2^24 - 1) correctly rounded to FP32, without a division: for
// 1 <= d < 2^24, d / (2^24 - 1) = d 2^-24 (1 + 2^-24 + 2^-48 + ...), and the
// exact value d 2^-24 = m 2^k (m a 24-bit significand) is followed by a
// fraction m / (2^24 - 1) of one unit in the last place that always lies in
// (1/2, 1], so the rounded quotient is d 2^-24 plus one ulp (checked for
// every d against the IEEE division).  The exponent and the ulp are one integer
// addition to the bits of (float)d, which leaves a negative number for d = 0
// alone.  Then rounded to BF16.
__device__ __forceinline__ __bf16 depth_bf16(uint32_t D)
{
    const uint32_t d = D < 16777215u ? D : 16777215u;
    const int x = (int)__float_as_uint((float)d) + (1 - (24 << 23));
    return (__bf16)__int_as_float(x > 0 ? x : 0);
}

// (NaN and -0 become +0)
__device__ __forceinline__ float relu(float v) { return fmaxf(v, 0.f); }

__device__ __forceinline__ bf16x8 frag(const uint4 &q) { return __builtin_bit_cast(bf16x8, q); }

// relu(acc + bias) of 8 consecutive channels, packed
__device__ __forceinline__ uint4 relu8(const floatx4 &a0, const floatx4 &a1, const float4 &c0, const float4 &c1)
{
    bf16x8 o;
    o[0] = (__bf16)relu(a0[0] + c0.x);
    o[1] = (__bf16)relu(a0[1] + c0.y);
    o[2] = (__bf16)relu(a0[2] + c0.z);
    o[3] = (__bf16)relu(a0[3] + c0.w);
    o[4] = (__bf16)relu(a1[0] + c1.x);
    o[5] = (__bf16)relu(a1[1] + c1.y);
    o[6] = (__bf16)relu(a1[2] + c1.z);
    o[7] = (__bf16)relu(a1[3] + c1.w);
    return __builtin_bit_cast(uint4, o);
}

__device__ __forceinline__ floatx4 mfma(const bf16x8 &a, const bf16x8 &b, const floatx4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// LDS slot of h1 pixel column xs (even columns first) and channel slot g
__device__ __forceinline__ int h1_slot(int xs, int g) { return xs * 4 + (g ^ ((xs >> 2) & 3)); }
__device__ __forceinline__ int h2_slot(int y, int x, int s) { return (y * kS2 + x) * 8 + (s ^ ((x + 4 * y) & 7)); }

// Half h (64 rows) of sample s's image: on its way into registers, and from
// there into LDS as BF16.
__device__ __forceinline__ void load_image(const uint32_t *depth, int s, int h, uint4 (&q)[kQuads])
{
    const uint4 *src = reinterpret_cast<const uint4 *>(depth + (size_t)s * kRes * kRes + h * (kRes * kRes / 2));
#pragma unroll
    for (int i = 0; i < kQuads; ++i) q[i] = src[i * kThreads + threadIdx.x];
}

__device__ __forceinline__ void store_image(EncLds &L, int h, const uint4 (&q)[kQuads])
{
    const int t = threadIdx.x;
    uint16_t *dst = &L.img[(h * (kRes / 2) + (t >> 5)) * kPitch + (t & 31) * 4];
#pragma unroll
    for (int i = 0; i < kQuads; ++i) {
        bf16x4 o;
        o[0] = depth_bf16(q[i].x);
        o[1] = depth_bf16(q[i].y);
        o[2] = depth_bf16(q[i].z);
        o[3] = depth_bf16(q[i].w);
        *reinterpret_cast<bf16x4 *>(dst + i * (kThreads / 32) * kPitch) = o;
    }
}

// Layer 1 of the image in LDS into h1 (LDS) and memory: output rows wave,
// wave + 8, ... in pairs, each row as two tiles of 16 pixels (four tiles in
// flight: one at a time a tile was a chain of LDS, matrix and store latencies,
// 580 cycles each).
__device__ __forceinline__ void layer1(EncLds &L, int s, int wave, int lane, uint16_t *__restrict__ out)
{
    const int r16 = lane & 15, g = lane >> 4;
    bf16x8 w[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) w[j][ks] = frag(L.w1[(j * 2 + ks) * 64 + lane]);
    const float4 c0 = *reinterpret_cast<const float4 *>(&L.bias[8 * g]);
    const float4 c1 = *reinterpret_cast<const float4 *>(&L.bias[8 * g + 4]);
    for (int oy = wave; oy < kS1; oy += 2 * kWaves) {
        floatx4 acc[2][2][2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int y = min(oy + r * kWaves, kS1 - 1);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint16_t *src = &L.img[(4 * y + g) * kPitch + 4 * min(16 * h + r16, kS1 - 1)];
                acc[r][h][0] = acc[r][h][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    // k = 32 ks + 8 g ..: window row ky = 4 ks + g, its 8 pixels
                    const uint2 lo = *reinterpret_cast<const uint2 *>(src + 4 * ks * kPitch);
                    const uint2 hi = *reinterpret_cast<const uint2 *>(src + 4 * ks * kPitch + 4);
                    const bf16x8 x = frag(make_uint4(lo.x, lo.y, hi.x, hi.y));
                    acc[r][h][0] = mfma(w[0][ks], x, acc[r][h][0]);
                    acc[r][h][1] = mfma(w[1][ks], x, acc[r][h][1]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int y = oy + r * kWaves;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ox = 16 * h + r16;
                const uint4 o = relu8(acc[r][h][0], acc[r][h][1], c0, c1);
                if (y < kS1 && ox < kS1) {
                    L.h1[y * 128 + h1_slot((ox & 1) * 16 + (ox >> 1), g)] = o;
                    *reinterpret_cast<uint4 *>(out + (((size_t)s * kS1 + y) * kS1 + ox) * kC1 + 8 * g) = o;
                }
            }
        }
    }
}

// Row `kRows` output rows (oy, oy + 1) of layer 2 for this wave's 32 channels.
template <int kRows>
__device__ __forceinline__ void layer2_rows(EncLds &L, const bf16x8 (&w)[2][16], int s, int oy, int cg, int lane,
                                            uint16_t *__restrict__ out)
{
    const int r16 = lane & 15, g = lane >> 4;
    const int i = min(r16, kS2 - 1);
    // columns 2 i + kx of a window row: parity kx & 1, xs = i + (kx >> 1)
    const uint4 *p0 = &L.h1[2 * oy * 128 + h1_slot(i, g)], *p1 = &L.h1[2 * oy * 128 + h1_slot(i + 1, g)];
    floatx4 acc[kRows][2];
#pragma unroll
    for (int r = 0; r < kRows; ++r) acc[r][0] = acc[r][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        const int ky = ks >> 2, kx = ks & 3;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const bf16x8 x = frag(((kx >> 1) ? p1 : p0)[(2 * r + ky) * 128 + (kx & 1) * 64]);
            acc[r][0] = mfma(w[0][ks], x, acc[r][0]);
            acc[r][1] = mfma(w[1][ks], x, acc[r][1]);
        }
    }
    if (r16 < kS2) {
        const float4 c0 = *reinterpret_cast<const float4 *>(&L.bias[kC1 + 32 * cg + 8 * g]);
        const float4 c1 = *reinterpret_cast<const float4 *>(&L.bias[kC1 + 32 * cg + 8 * g + 4]);
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const uint4 o = relu8(acc[r][0], acc[r][1], c0, c1);
            L.h2[h2_slot(oy + r, r16, 4 * cg + g)] = o;
            *reinterpret_cast<uint4 *>(out + ((size_t)s * kS2 * kS2 + (oy + r) * kS2 + r16) * kC2 + 32 * cg + 8 * g) = o;
        }
    }
}

// kTiles 16-pixel tiles t, t + 4, ... of layer 3 for this wave's 16 channels.
template <int kTiles>
__device__ __forceinline__ void layer3_tiles(EncLds &L, int s, int t, int cg, int lane, uint16_t *__restrict__ out)
{
    const int r16 = lane & 15, g = lane >> 4;
    // window pixel (oy + ky, ox + kx), channel half k & 1: the slot is g XOR the
    // pixel's key, and the half and an odd ky both flip bit 2 of it
    const uint4 *p[kTiles][3];
    int flip[kTiles][3];
    floatx4 acc[kTiles];
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
        const int m = 16 * (t + 4 * j) + r16, oy = m / kS3, ox = m - oy * kS3;
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            const int i = h2_slot(oy, ox + kx, g);
            p[j][kx] = &L.h2[i];
            flip[j][kx] = (i & 4) ? -4 : 4;
        }
        acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int ks = 0; ks < 18; ++ks) {
        const int tap = ks >> 1, ky = tap / 3, kx = tap - 3 * ky;
        const bf16x8 w = frag(L.w3[(cg * 18 + ks) * 64 + lane]);
#pragma unroll
        for (int j = 0; j < kTiles; ++j)
            acc[j] = mfma(w, frag(p[j][kx][ky * kS2 * 8 + (((ks ^ ky) & 1) ? flip[j][kx] : 0)]), acc[j]);
    }
    const float4 c = *reinterpret_cast<const float4 *>(&L.bias[kC1 + kC2 + 16 * cg + 4 * g]);
#pragma unroll
    for (int j = 0; j < kTiles; ++j) {
        const int m = 16 * (t + 4 * j) + r16;
        bf16x4 o;
        o[0] = (__bf16)relu(acc[j][0] + c.x);
        o[1] = (__bf16)relu(acc[j][1] + c.y);
        o[2] = (__bf16)relu(acc[j][2] + c.z);
        o[3] = (__bf16)relu(acc[j][3] + c.w);
        *reinterpret_cast<bf16x4 *>(out + ((size_t)s * kS3 * kS3 + m) * kC3 + 16 * cg + 4 * g) = o;
    }
}

// Samples blockIdx.x, + gridDim.x, ...  Two barriers per sample: layer 2 of
// sample s (with the next image on its way, half by half, through registers), then layer 3 of s
// beside layer 1 of the next sample.  The second layer's weights stay in
// registers (128: 32 channels per wave, 4 waves sharing the rows, which halves
// the LDS reads of 16 channels per wave), the others' in LDS.
__global__ __launch_bounds__(kThreads, 2) void k_encoder(const uint32_t *__restrict__ depth, EncoderWeights W, int n,
                                                         uint16_t *__restrict__ o1, uint16_t *__restrict__ o2,
                                                         uint16_t *__restrict__ o3)
{
    __shared__ __attribute__((aligned(16))) EncLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int cg = wave >> 2, mg = wave & 3;
    int s = blockIdx.x;
    // everything the first sample needs is requested before anything is waited for
    uint4 q[kQuads], q1[kQuads];
    load_image(depth, s, 0, q);
    load_image(depth, s, 1, q1);
    // MFMA row r of a pair of 16-channel blocks j = 0, 1 is channel
    // 8 (r / 4) + 4 j + r % 4, so that a lane's rows 4 g + 0..3 of both blocks
    // are channels 8 g .. 8 g + 7
    const int ch = 8 * (r16 >> 2) + (r16 & 3);
    const uint4 f1 = *reinterpret_cast<const uint4 *>(W.w1 + (size_t)(ch + 4 * ((wave >> 1) & 1)) * 64 +
                                                      32 * (wave & 1) + 8 * g);
    uint4 f3[5];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        const int f = min(wave + kWaves * i, 35), c = f / 18;
        f3[i] = *reinterpret_cast<const uint4 *>(W.w3 + (size_t)(16 * c + r16) * kK3 + 32 * (f - 18 * c) + 8 * g);
    }
    const float bias = tid < kC1 ? W.b1[tid] : tid < kC1 + kC2 ? W.b2[tid - kC1] : tid < 128 ? W.b3[tid - kC1 - kC2] : 0.f;
    bf16x8 w2[2][16];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const uint16_t *row = W.w2 + (size_t)(32 * cg + ch + 4 * j) * kK2 + 8 * g;
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) w2[j][ks] = frag(*reinterpret_cast<const uint4 *>(row + 32 * ks));
    }
    store_image(L, 0, q);
    store_image(L, 1, q1);
    if (wave < 4) L.w1[wave * 64 + lane] = f1;
#pragma unroll
    for (int i = 0; i < 5; ++i)
        if (wave + kWaves * i < 36) L.w3[(wave + kWaves * i) * 64 + lane] = f3[i];
    if (tid < kC1 + kC2 + kC3) L.bias[tid] = bias;
    __syncthreads();
    layer1(L, s, wave, lane, o1);
    __syncthreads();
    const int row0 = mg < 2 ? 4 * mg : 8 + 3 * (mg - 2);   // 14 output rows as 4, 4, 3, 3
    for (;;) {
        const int next = s + gridDim.x;
        const bool more = next < n;
        // opaque per sample, so that the LDS addresses of every window are not
        // hoisted out of the loop into registers there are not
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (more) load_image(depth, next, 0, q);
        layer2_rows<2>(L, w2, s, row0, cg, ln, o2);
        if (more) {
            store_image(L, 0, q);
            load_image(depth, next, 1, q);
        }
        if (mg < 2) layer2_rows<2>(L, w2, s, row0 + 2, cg, ln, o2);
        else layer2_rows<1>(L, w2, s, row0 + 2, cg, ln, o2);
        if (more) store_image(L, 1, q);
        __syncthreads();
        if (more) layer1(L, next, wave, ln, o1);
        layer3_tiles<2>(L, s, mg, cg, ln, o3);
        if (mg == 0) layer3_tiles<1>(L, s, 8, cg, ln, o3);
        if (!more) break;
        s = next;
        __syncthreads();
    }
}

}  // namespace

hipError_t encoder_forward(const uint32_t *depth, const EncoderWeights &w, int n, uint16_t *h1, uint16_t *h2,
                           uint16_t *h3, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    // one workgroup per CU (all 160 KB of its LDS, two waves per SIMD); each loops over
    // its samples
    hipLaunchKernelGGL(k_encoder, dim3(std::min(n, kPolicyCUs)), dim3(kThreads), 0, s, depth, w, n, h1, h2, h3);
    return hipGetLastError();
}

}  // namespace gal
