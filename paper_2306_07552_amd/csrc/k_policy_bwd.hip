// Backward pass of the policy's convolutions (the update of Section 4.2) as two
// persistent kernels, a sample at a time through LDS: the third layer (weight
// and input gradient), then the second (both) with the first layer's weight
// gradient.  The first layer's output gradient never leaves LDS.
//
// What bounds them: no one unit.  Of the time of 32,768 samples memory moves 59 KB
// per sample for the third layer and 153 KB for the second and first (3.2 and 3.0
// of 4.7 TB/s), the LDS is busy for 0.39 and 0.30, the matrix cores for 0.30 and
// 0.29, VALU issue for 0.37 and 0.33; two waves per SIMD and a barrier per phase
// overlap these only in part (waves wait 0.46 and 0.37 of their cycles).  As one
// kernel per layer and gradient, the largest map (61.5 KB per sample) crossed memory
// six times, its gradient included, and each input pixel was gathered once per tap.
// Measured, 32,768 samples: 2.7 -> 0.60 ms for the third layer, 9.5 -> 1.65 ms for
// the second and first.
//
// A weight gradient is dY^T times the windows of the input, summed over the
// output pixels: both operands lie in LDS pixel by pixel, so their fragments
// (8 consecutive pixels of one channel per lane) come from the transposing LDS
// read ds_read_b64_tr_b16.  The FP32 sums of a workgroup's samples stay in
// registers and leave once, into one slab per workgroup; the slabs are added in
// order.  No atomics: the result does not depend on timing.  An input gradient
// is the adjoint, with the weights in registers (A operand) and dY's pixels as
// the B operand, its sum over ascending steps of (tap, output channel).
#include "gal_internal.h"
#include "gal_policy.h"

#include <algorithm>

namespace gal {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t quad __attribute__((ext_vector_type(4)));   // 16 bytes: 8 BF16 values or 4 depths

constexpr int kThreads = 512;   // 8 waves
constexpr int kRes = kPolicyRes;
constexpr int kS1 = 31, kS2 = 14, kS3 = 12;  // map edges
constexpr int kC1 = 32, kC2 = 64, kC3 = 32;  // channels
constexpr int kPix = 144;                    // bytes per 64-channel pixel in LDS (16 of padding: no bank conflicts)

__device__ __forceinline__ bf16x8 frag(const quad &q) { return __builtin_bit_cast(bf16x8, q); }

__device__ __forceinline__ floatx4 mfma(const bf16x8 &a, const bf16x8 &b, const floatx4 &c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// v, as a value the compiler cannot see through: addresses derived from it are
// computed where they are used, not hoisted out of the sample loop into
// registers that the sums and weights need.
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}

__device__ __forceinline__ bf16x8 ones()
{
    return __builtin_bit_cast(bf16x8, quad{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
}

// Transposing reads of two 4 x 16 blocks: within 16 lanes, lane i gives the
// address of 4 values, columns 4 (i % 4) .. of row i / 4, and receives column i
// of the 4 rows; lo and hi hold rows 0..3 and 4..7 of the lane group's 8.
__device__ __forceinline__ bf16x8 tr_frag(const unsigned char *lo, const unsigned char *hi)
{
    typedef __attribute__((address_space(3))) shortx4 lds4;
    const shortx4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(lo));
    const shortx4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(hi));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// bf16(acc) of 8 consecutive channels where the activation h is positive, else 0
__device__ __forceinline__ quad masked8(const floatx4 &a0, const floatx4 &a1, const quad &h)
{
    const shortx8 hv = __builtin_bit_cast(shortx8, h);
    bf16x8 o;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = (__bf16)(hv[k] > 0 ? (k < 4 ? a0[k & 3] : a1[k & 3]) : 0.f);
    return __builtin_bit_cast(quad, o);
}

// the depth scaling of the forward pass (k_policy_enc.hip)
__device__ __forceinline__ __bf16 depth_bf16(uint32_t D)
{
    const uint32_t d = D < 16777215u ? D : 16777215u;
    const int x = (int)__float_as_uint((float)d) + (1 - (24 << 23));
    return (__bf16)__int_as_float(x > 0 ? x : 0);
}

// ------------------------------------------------------------- third layer
// LDS of one sample: d3 with a border of zeros (rows and columns -2 ..), 4 slots
// of 8 channels per pixel, XORed with column bits; h2 pixel by pixel.
constexpr int kD3Rows = 16, kD3Cols = 18;
struct Lds3 {
    quad d3[kD3Rows * kD3Cols * 4];
    unsigned char h2[kS2 * kS2 * kPix];
};
__device__ __forceinline__ int d3_slot(int oy, int ox, int s)
{
    return ((oy + 2) * kD3Cols + ox + 2) * 4 + (s ^ (((ox + 2) >> 2) & 3));
}

__device__ __forceinline__ void load3(const uint16_t *d3, const uint16_t *h2, int s, quad (&qd)[2], quad (&qh)[4])
{
    const int t = threadIdx.x;
    const quad *a = reinterpret_cast<const quad *>(d3) + (size_t)s * (kS3 * kS3 * 4);
    const quad *b = reinterpret_cast<const quad *>(h2) + (size_t)s * (kS2 * kS2 * 8);
#pragma unroll
    for (int i = 0; i < 2; ++i) qd[i] = a[min(i * kThreads + t, kS3 * kS3 * 4 - 1)];
#pragma unroll
    for (int i = 0; i < 4; ++i) qh[i] = b[min(i * kThreads + t, kS2 * kS2 * 8 - 1)];
}
__device__ __forceinline__ void store3(Lds3 &L, const quad (&qd)[2], const quad (&qh)[4])
{
    const int t = threadIdx.x;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int k = i * kThreads + t, p = k >> 2, oy = p / kS3;
        if (k < kS3 * kS3 * 4) L.d3[d3_slot(oy, p - oy * kS3, k & 3)] = qd[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = i * kThreads + t;
        if (k < kS2 * kS2 * 8) *reinterpret_cast<quad *>(&L.h2[(k >> 3) * kPix + (k & 7) * 16]) = qh[i];
    }
}

// Per sample: dW3 [32][9 taps x 64] += d3^T h2 windows (5 steps of 32 pixels,
// the last 16 on the zero border; wave w sums the 16 columns w, w + 8, ... of
// the 36), db3 += d3, and d2 = [h2 > 0] times the adjoint of d3 (each wave 32
// channels of 3 or 4 rows).  Two buffers: the next sample arrives through
// registers meanwhile, one barrier per sample.
__global__ __launch_bounds__(kThreads, 2) void k_back3(const uint16_t *__restrict__ d3, const uint16_t *__restrict__ h2,
                                                       const uint16_t *__restrict__ wt3, int n,
                                                       uint16_t *__restrict__ d2, float *__restrict__ part)
{
    __shared__ __attribute__((aligned(16))) Lds3 L[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int cg = wave >> 2, mg = wave & 3;     // input gradient: channel half, row group
    const int cb = wave & 3, tap0 = wave >> 2;   // weight gradient: 16 channels, taps tap0, tap0 + 2, ...
    int s = blockIdx.x;
    quad qd0[2], qh0[4];
    load3(d3, h2, s, qd0, qh0);
    bf16x8 w[2][9];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ks = 0; ks < 9; ++ks)
            w[j][ks] = frag(*reinterpret_cast<const quad *>(
                wt3 + (size_t)(32 * cg + 8 * (r16 >> 2) + 4 * j + (r16 & 3)) * (9 * kC3) + 32 * ks + 8 * g));
    for (int i = tid; i < kD3Rows * kD3Cols * 4; i += kThreads) L[0].d3[i] = L[1].d3[i] = quad{0u, 0u, 0u, 0u};
    __syncthreads();
    store3(L[0], qd0, qh0);
    __syncthreads();
    floatx4 acc[5][2], accb[2];
#pragma unroll
    for (int k = 0; k < 5; ++k) acc[k][0] = acc[k][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    accb[0] = accb[1] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int row0 = mg < 2 ? 4 * mg : 8 + 3 * (mg - 2), nrows = mg < 2 ? 4 : 3;
    for (int buf = 0;; buf ^= 1) {
        // (the last sample loads itself again, unused: a conditional load would keep
        // its registers through the whole loop)
        const bool more = s + (int)gridDim.x < n;
        const int next = more ? s + (int)gridDim.x : s;
        quad qd[2], qh[4];
        load3(d3, h2, next, qd, qh);
        Lds3 &B = L[buf];
        const int ln = opaque(lane);
        const int r = ln & 15, gg = ln >> 4;
        // ---- weight gradient
        {
            const unsigned char *db = reinterpret_cast<const unsigned char *>(B.d3);
            const int c1 = (r & 3) >> 1, half = (r & 1) * 8;
#pragma unroll
            for (int t = 0; t < 5; ++t) {
                const unsigned char *pa[2][2], *pb[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int m = 32 * t + 8 * gg + 4 * h + (r >> 2), oy = m / kS3, ox = m - oy * kS3;
                    pa[0][h] = db + d3_slot(oy, ox, c1) * 16 + half;
                    pa[1][h] = db + d3_slot(oy, ox, 2 + c1) * 16 + half;
                    pb[h] = B.h2 + (min(oy, kS3 - 1) * kS2 + ox) * kPix + cb * 32 + c1 * 16 + half;
                }
                bf16x8 a[2];
                a[0] = tr_frag(pa[0][0], pa[0][1]);
                a[1] = tr_frag(pa[1][0], pa[1][1]);
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    const int tap = tap0 + 2 * k;
                    if (tap < 9) {
                        const int off = ((tap / 3) * kS2 + tap % 3) * kPix;
                        const bf16x8 b = tr_frag(pb[0] + off, pb[1] + off);
                        acc[k][0] = mfma(a[0], b, acc[k][0]);
                        acc[k][1] = mfma(a[1], b, acc[k][1]);
                    }
                }
                if (wave == 7) {
                    accb[0] = mfma(a[0], ones(), accb[0]);
                    accb[1] = mfma(a[1], ones(), accb[1]);
                }
            }
        }
        // ---- input gradient: rows qy, pixel qx = lane % 16 (14 used)
        const quad *px[3];
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) px[kx] = &B.d3[d3_slot(row0, r - kx, gg)];
        for (int i = 0; i < nrows; ++i) {
            floatx4 x[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int ks = 0; ks < 9; ++ks) {
                const int ky = ks / 3, kx = ks - 3 * ky;
                const bf16x8 y = frag(px[kx][(i - ky) * kD3Cols * 4]);
                x[0] = mfma(w[0][ks], y, x[0]);
                x[1] = mfma(w[1][ks], y, x[1]);
            }
            if (r < kS2) {
                const int p = (row0 + i) * kS2 + r;
                const quad hv = *reinterpret_cast<const quad *>(&B.h2[p * kPix + (4 * cg + gg) * 16]);
                *reinterpret_cast<quad *>(d2 + ((size_t)s * kS2 * kS2 + p) * kC2 + 32 * cg + 8 * gg) =
                    masked8(x[0], x[1], hv);
            }
        }
        if (!more) break;
        store3(L[buf ^ 1], qd, qh);
        __syncthreads();
        s = next;
    }
    // slab: W [32][576], b [32]
    float *out = part + (size_t)blockIdx.x * (kC3 * 9 * kC2 + kC3);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        const int tap = tap0 + 2 * k;
        if (tap >= 9) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                out[(size_t)(16 * j + 4 * g + e) * (9 * kC2) + tap * kC2 + cb * 16 + r16] = acc[k][j][e];
    }
    if (wave == 7 && r16 == 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) out[kC3 * 9 * kC2 + 16 * j + 4 * g + e] = accb[j][e];
    }
}

// ------------------------------------------------- second and first layers
// LDS of one sample: the image as BF16 (row pitch 160: the two image rows of a
// transposing read fall in different banks); h1, later d1 in place, as rows of
// 32 pixel columns, even columns first (column 31 zero), 4 slots of 8 channels
// XORed with column bits; d2 with a border of zeros (rows and columns -1 ..).
constexpr int kImgPitch = 160;
constexpr int kD2Edge = 17;
struct Lds21 {
    uint16_t img[kRes * kImgPitch];
    quad h1[kS1 * 32 * 4];
    unsigned char d2[kD2Edge * kD2Edge * kPix];
};
__device__ __forceinline__ int h1_slot(int xs, int g) { return xs * 4 + (g ^ ((xs >> 2) & 3)); }

constexpr int kH1Quads = kS1 * kS1 * 4, kD2Quads = kS2 * kS2 * 8;
constexpr int kImgLoads = kRes * kRes / 8 / kThreads;   // 16-byte loads per thread of half an image
__device__ __forceinline__ void load_h1(const uint16_t *h1, int s, quad (&q)[8])
{
    const quad *a = reinterpret_cast<const quad *>(h1) + (size_t)s * kH1Quads;
    const int t = opaque(threadIdx.x);
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = a[min(i * kThreads + t, kH1Quads - 1)];
}
__device__ __forceinline__ void store_h1(Lds21 &L, const quad (&q)[8])
{
    const int t = opaque(threadIdx.x);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = i * kThreads + t, p = k >> 2, y = p / kS1, x = p - y * kS1;
        if (k < kH1Quads) L.h1[y * 128 + h1_slot((x & 1) * 16 + (x >> 1), k & 3)] = q[i];
    }
}
__device__ __forceinline__ void load_d2(const uint16_t *d2, int s, quad (&q)[4])
{
    const quad *a = reinterpret_cast<const quad *>(d2) + (size_t)s * kD2Quads;
    const int t = opaque(threadIdx.x);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = a[min(i * kThreads + t, kD2Quads - 1)];
}
__device__ __forceinline__ void store_d2(Lds21 &L, const quad (&q)[4])
{
    const int t = opaque(threadIdx.x);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = i * kThreads + t, p = k >> 3, y = p / kS2, x = p - y * kS2;
        if (k < kD2Quads)
            *reinterpret_cast<quad *>(&L.d2[((y + 1) * kD2Edge + x + 1) * kPix + (k & 7) * 16]) = q[i];
    }
}
__device__ __forceinline__ void load_image(const uint32_t *depth, int s, int h, quad (&q)[kImgLoads])
{
    const quad *src = reinterpret_cast<const quad *>(depth + (size_t)s * kRes * kRes + h * (kRes * kRes / 2));
    const int t = opaque(threadIdx.x);
#pragma unroll
    for (int i = 0; i < kImgLoads; ++i) q[i] = src[i * kThreads + t];
}
__device__ __forceinline__ void store_image(Lds21 &L, int h, const quad (&q)[kImgLoads])
{
    const int t = opaque(threadIdx.x);
    uint16_t *dst = &L.img[(h * (kRes / 2) + (t >> 5)) * kImgPitch + (t & 31) * 4];
#pragma unroll
    for (int i = 0; i < kImgLoads; ++i) {
        bf16x4 o;
        o[0] = depth_bf16(q[i].x);
        o[1] = depth_bf16(q[i].y);
        o[2] = depth_bf16(q[i].z);
        o[3] = depth_bf16(q[i].w);
        *reinterpret_cast<bf16x4 *>(dst + i * (kThreads / 32) * kImgPitch) = o;
    }
}

constexpr int kW1 = kC1 * 64, kW2 = kC2 * 16 * kC1;
constexpr int kSlab21 = kW1 + kC1 + kW2 + kC2;   // the parameter layout: conv1 W, b, conv2 W, b

// Per sample, in three passes with a barrier between them:
//  1. dW2 [64][16 taps x 32] += d2^T h1 windows: 7 steps of two output rows (16
//     columns each, the last two on the zero border); wave w sums taps 2 w and
//     2 w + 1 (64 x 64 values, 64 registers).
//  2. d1 = [h1 > 0] times the adjoint of d2, over h1 in place.  The stride-2
//     layer's input pixels fall into four parity classes, each reached by 4 of
//     the 16 taps: wave w draws half the rows of class w % 4, whose weights (32 x
//     256) fill 64 registers.
//  3. dW1 [32][64] += d1^T image windows, one step per output row: 4 groups of
//     rows x 2 halves of the columns.
// The image arrives during 1, the next sample's d2 during 2 and its h1 during 3.
__global__ __launch_bounds__(kThreads, 2) void k_back21(const uint32_t *__restrict__ depth,
                                                        const uint16_t *__restrict__ h1,
                                                        const uint16_t *__restrict__ d2,
                                                        const uint16_t *__restrict__ wt2, int n,
                                                        float *__restrict__ part)
{
    __shared__ __attribute__((aligned(16))) Lds21 L;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    const int py = (wave >> 1) & 1, px = wave & 1, hw = wave >> 2;   // pass 2: class and half of its rows
    const int rg = wave >> 1, kg = wave & 1;                         // pass 3: row group, column half
    int s = blockIdx.x;
    quad qh0[8], qd0[4];
    load_h1(h1, s, qh0);
    load_d2(d2, s, qd0);
    for (int i = tid; i < kD2Edge * kD2Edge * kPix / 16; i += kThreads)
        reinterpret_cast<quad *>(L.d2)[i] = quad{0u, 0u, 0u, 0u};
    for (int i = tid; i < kS1 * 4; i += kThreads) L.h1[(i >> 2) * 128 + h1_slot(31, i & 3)] = quad{0u, 0u, 0u, 0u};
    for (int i = tid; i < kRes * (kImgPitch - kRes) / 8; i += kThreads)
        *reinterpret_cast<quad *>(&L.img[(i >> 2) * kImgPitch + kRes + (i & 3) * 8]) = quad{0u, 0u, 0u, 0u};
    __syncthreads();
    store_h1(L, qh0);
    store_d2(L, qd0);
    floatx4 acc2[4][4], accb2, acc1[2][2], accb1[2];   // [16 o][taps, 16 c], [16 c][16 k]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc2[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        acc1[i][0] = acc1[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
        accb1[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    accb2 = floatx4{0.f, 0.f, 0.f, 0.f};
    unsigned char *h1b = reinterpret_cast<unsigned char *>(L.h1);
    for (;;) {
        __syncthreads();
        const int ln = opaque(lane);
        const int r = ln & 15, gg = ln >> 4;
        const int c1 = (r & 3) >> 1, half = (r & 1) * 8;
        quad qi[kImgLoads];
        load_image(depth, s, 0, qi);
        bf16x8 w[2][8];   // pass 2's weights: [16 channels][step]
        // ---- 1: step t covers output rows 2 t + gg / 2, columns 8 (gg % 2) + 0..7
        {
            const unsigned char *pa[2], *pb[2][2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ox = 8 * (gg & 1) + 4 * h + (r >> 2), oy = gg >> 1;
                pa[h] = L.d2 + ((oy + 1) * kD2Edge + ox + 1) * kPix + c1 * 16 + half;
                // the border's columns read the last window (times zero)
                const int xs = min(ox, kS2 - 1) + (wave & 1);
#pragma unroll
                for (int c = 0; c < 2; ++c)
                    pb[h][c] = h1b + ((2 * oy + (wave >> 1)) * 128 + h1_slot(xs, 2 * c + c1)) * 16 + half;
            }
            auto step = [&]() {
                bf16x8 a[4], b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) a[i] = tr_frag(pa[0] + 32 * i, pa[1] + 32 * i);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // tap 2 w + j / 2 (odd columns 16 further), 16 channels j % 2
                    const int off = (j >> 1) * 1024;
                    b[j] = tr_frag(pb[0][j & 1] + off, pb[1][j & 1] + off);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc2[i][j] = mfma(a[i], b[j], acc2[i][j]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (wave == i) accb2 = mfma(a[i], ones(), accb2);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    pa[h] += 2 * kD2Edge * kPix;
                    pb[h][0] += 4 * 2048;
                    pb[h][1] += 4 * 2048;
                }
            };
#pragma unroll 1
            for (int t = 0; t < 3; ++t) step();
            store_image(L, 0, qi);
            load_image(depth, s, 1, qi);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const uint16_t *row = wt2 + ((size_t)(8 * (r >> 2) + 4 * j + (r & 3)) * 16 + py * 4 + px) * kC2 + 8 * gg;
#pragma unroll
                for (int ks = 0; ks < 8; ++ks)   // tap (jy, jx) of the class, half of the output channels
                    w[j][ks] = frag(*reinterpret_cast<const quad *>(
                        row + ((ks >> 2) * 8 + ((ks >> 1) & 1) * 2) * kC2 + 32 * (ks & 1)));
            }
#pragma unroll 1
            for (int t = 3; t < 7; ++t) step();
        }
        store_image(L, 1, qi);
        // (the last sample loads itself again, unused: a conditional load would keep
        // its registers through the whole loop)
        const bool more = s + (int)gridDim.x < n;
        const int next = more ? s + (int)gridDim.x : s;
        __syncthreads();
        quad qd[4];
        load_d2(d2, next, qd);
        // ---- 2: rows qy of the class, pixel qx = lane % 16
        {
            const unsigned char *pd[2];
#pragma unroll
            for (int jx = 0; jx < 2; ++jx)
                pd[jx] = L.d2 + ((8 * hw + 1) * kD2Edge + (r - jx) + 1) * kPix + gg * 16;
            const int nr = 8 - (hw & py);   // class rows 16 or 15 in halves
            const int xs = px * 16 + r;
            quad *ph = &L.h1[(16 * hw + py) * 128 + h1_slot(xs, gg)];
#pragma unroll 1
            for (int i = 0; i < nr; i += 2) {
                floatx4 x[2][2];
#pragma unroll
                for (int k = 0; k < 2; ++k) x[k][0] = x[k][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const int jy = ks >> 2, jx = (ks >> 1) & 1;
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const bf16x8 y = frag(*reinterpret_cast<const quad *>(
                            pd[jx] + (i + k - jy) * kD2Edge * kPix + 64 * (ks & 1)));
                        x[k][0] = mfma(w[0][ks], y, x[k][0]);
                        x[k][1] = mfma(w[1][ks], y, x[k][1]);
                    }
                }
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    if (i + k < nr) {
                        quad *dst = ph + (i + k) * 256;
                        *dst = masked8(x[k][0], x[k][1], *dst);
                    }
            }
        }
        __syncthreads();
        quad qh[8];
        store_d2(L, qd);
        load_h1(h1, next, qh);
        // ---- 3: output rows rg, rg + 4, ...; pixel columns in the map's own order
        // (even ones first), on both sides
        {
            const unsigned char *pa[2][2], *pb[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int xs = 8 * gg + 4 * h + (r >> 2), x = xs < 16 ? 2 * xs : 2 * (xs - 16) + 1;
#pragma unroll
                for (int c = 0; c < 2; ++c) pa[h][c] = h1b + (rg * 128 + h1_slot(xs, 2 * c + c1)) * 16 + half;
                pb[h] = reinterpret_cast<const unsigned char *>(
                    &L.img[(4 * rg + 4 * kg + c1) * kImgPitch + 4 * x + 4 * (r & 1)]);
            }
#pragma unroll 1
            for (int oy = rg; oy < kS1; oy += 4) {
                bf16x8 a[2], b[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) a[c] = tr_frag(pa[0][c], pa[1][c]);
#pragma unroll
                for (int j = 0; j < 2; ++j) b[j] = tr_frag(pb[0] + j * 4 * kImgPitch, pb[1] + j * 4 * kImgPitch);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc1[c][j] = mfma(a[c], b[j], acc1[c][j]);
                    if (kg == 0) accb1[c] = mfma(a[c], ones(), accb1[c]);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    pa[h][0] += 4 * 2048;
                    pa[h][1] += 4 * 2048;
                    pb[h] += 16 * kImgPitch * 2;
                }
            }
        }
        __syncthreads();
        if (!more) break;
        store_h1(L, qh);
        s = next;
    }
    // ---- the slab: dW1 and db1 as the row groups' sums in order, dW2, db2
    float *out = part + (size_t)blockIdx.x * kSlab21;
    float *red = reinterpret_cast<float *>(L.h1);   // [4 groups][32][64], then [4][32]
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int o = 16 * c + 4 * g + e;
#pragma unroll
            for (int j = 0; j < 2; ++j) red[(rg * kC1 + o) * 64 + 16 * (2 * kg + j) + r16] = acc1[c][j][e];
            if (kg == 0 && r16 == 0) red[4 * kW1 + rg * kC1 + o] = accb1[c][e];
        }
    __syncthreads();
    for (int i = tid; i < kW1 + kC1; i += kThreads) {
        const float *v = i < kW1 ? red + i : red + 4 * kW1 + (i - kW1);
        const int st = i < kW1 ? kW1 : kC1;
        out[i] = ((v[0] + v[st]) + v[2 * st]) + v[3 * st];
    }
    out += kW1 + kC1;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                out[(size_t)(16 * i + 4 * g + e) * (16 * kC1) + (2 * wave + (j >> 1)) * kC1 + 16 * (j & 1) + r16] =
                    acc2[i][j][e];
    if (wave < 4 && r16 == 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[kW2 + 16 * wave + 4 * g + e] = accb2[e];
    }
}

// The adjoint weights of layers 2 and 3: wt[c][tap][o] = W[o][tap][c].
__global__ void k_adjoint_weights(const uint16_t *__restrict__ w2, const uint16_t *__restrict__ w3,
                                  uint16_t *__restrict__ wt2, uint16_t *__restrict__ wt3)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool second = i < kW2;
    if (!second) i -= kW2;
    const int taps = second ? 16 : 9, O = second ? kC2 : kC3, C = second ? kC1 : kC2;
    if (i >= O * taps * C) return;
    const int o = i / (taps * C), rem = i - o * taps * C, tap = rem / C, c = rem - tap * C;
    (second ? wt2 : wt3)[(c * taps + tap) * O + o] = (second ? w2 : w3)[i];
}

}  // namespace

size_t encoder_backward_floats()
{
    return (size_t)kPolicyCUs * std::max(kSlab21, kC3 * 9 * kC2 + kC3);
}

size_t encoder_backward_weights() { return (size_t)kW2 + kC3 * 9 * kC2; }

hipError_t encoder_backward(const uint32_t *depth, const uint16_t *h1, const uint16_t *h2, const uint16_t *d3,
                            uint16_t *d2, const uint16_t *w2, const uint16_t *w3, uint16_t *wt, int n, float *part,
                            size_t part_floats, float *g12, float *g3, hipStream_t s)
{
    if (n <= 0 || part_floats < encoder_backward_floats()) return hipErrorInvalidValue;
    const int grid = std::min(n, kPolicyCUs);   // one workgroup per CU
    hipLaunchKernelGGL(k_adjoint_weights, dim3((kW2 + kC3 * 9 * kC2 + 255) / 256), dim3(256), 0, s, w2, w3, wt, wt + kW2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_back3, dim3(grid), dim3(kThreads), 0, s, d3, h2, wt + kW2, n, d2, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = sum_parts(part, grid, kC3 * 9 * kC2 + kC3, g3, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_back21, dim3(grid), dim3(kThreads), 0, s, depth, h1, d2, wt, n, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return sum_parts(part, grid, kSlab21, g12, s);
}

}  // namespace gal
