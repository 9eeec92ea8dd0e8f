// BF16 GEMM on the matrix cores with FP32 accumulation, for operands whose rows
// are 16-byte aligned (every layer of the surrogate's training and of the
// policy's fully connected layer; mlp_gemm keeps a general kernel for the rest).
//
// C[M][N] = sum_k A(m, k) B(n, k).  Either operand lies k-contiguous (rows of k)
// or k-strided (rows of m or n, one per k).  K advances 64 at a time through a
// ring of LDS stages filled straight from memory (global_load_lds, no
// registers), one barrier per stage; a k-strided operand's fragments come from
// the transposing LDS read.  What bounds it: what reaches LDS on large products,
// 10-13 TB/s from L2 over the chip (C 32768 x 512, K 4608: 2.4 GB in 199 us, the
// matrix cores busy for 0.31 of the time, the LDS for 0.15), of which the products
// with the largest operands take 5.2 TB/s from memory; the latency of the stages in
// flight on small ones; measured at the tile rule below.
//
// Sums run over ascending 32-wide steps of k in FP32, so results do not depend
// on the tile shape.
#include "gal_internal.h"
#include "gal_mlp.h"

#include <algorithm>

namespace gal {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t quad __attribute__((ext_vector_type(4)));

constexpr int kStageK = 64;

struct GemmArgs {
    const uint16_t *a, *b;
    int M, N, K, lda, ldb, ldc;
    int tiles_m, tiles_n, splits, kchunk;   // kchunk: k per split, a multiple of 32
    const float *bias;
    const uint16_t *mask;
    int ldm;
    float *cf;
    uint16_t *cb;
};

// 64 lanes x 16 bytes from memory into LDS at lds .. lds + 1023, without
// registers.  The compiler does not see the transfer: the caller waits for it
// (vmcnt) and orders it with barriers.
__device__ __forceinline__ void dma16(const uint16_t *src, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(src) : "memory");
}

template <int kN>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kN) : "memory");
}

// every wave's LDS reads of the stage before are done, then all meet
__device__ __forceinline__ void stage_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__device__ __forceinline__ uint32_t lds_addr(const void *p)
{
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p;
}

// what a k-strided operand's rows past the last k are read from
__device__ const quad kZeros[1] = {};

// One operand's tile in LDS: R rows (m or n) x 64 k of BF16.
//  k-contiguous: R rows of 128 bytes, 8 slots of 8 k, the slot XORed with a key
//    of the row: its low 3 bits (A), or for B, whose fragments take rows 0..3,
//    8..11, ..., bits 0, 1 and 3: lanes of one read fall in different banks.
//  k-strided: 64 rows of k, R / 8 slots of 8 columns, XORed with 4 (k % 4).
template <int R, bool kStrided, bool kIsB>
struct Tile {
    static constexpr int kBytes = R * kStageK * 2;
    static constexpr int kDma = kBytes / 1024 / 4;   // transfers per wave (4 waves)
    // byte offset (elements) of this lane's source in each transfer, for a tile
    // whose first row (m or n) is r0; rows past the last repeat it
    int off[kDma];
    int krow[kDma];   // k-strided: the source's k within the stage
    __device__ __forceinline__ void init(int r0, int rows, int ld, int wave, int lane)
    {
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const int c = wave * kDma + i;   // 1 KB piece of the tile
            if (kStrided) {
                constexpr int kSlots = R / 8;
                const int k = c * (64 / kSlots) + lane / kSlots;
                const int slot = (lane % kSlots) ^ (4 * (k & 3) & (kSlots - 1));
                krow[i] = k;
                off[i] = min(r0 + slot * 8, rows - 8);
            } else {
                const int r = c * 8 + (lane >> 3);
                const int key = kIsB ? ((r & 3) | ((r >> 3 & 1) << 2)) : (r & 7);
                krow[i] = ((lane & 7) ^ key) * 8;
                off[i] = min(r0 + r, rows - 1);
            }
        }
    }
    // request stage k0 .. k0 + 63 of p; beyond klast: zeros (k-strided, where K may
    // end anywhere), or valid values that no step takes (k-contiguous)
    __device__ __forceinline__ void fetch(const uint16_t *p, int ld, int k0, int klast, uint32_t lds, int wave) const
    {
        const bool tail = k0 + kStageK - 1 > klast;
#pragma unroll
        for (int i = 0; i < kDma; ++i) {
            const uint16_t *src;
            if (kStrided) {
                src = p + (size_t)(k0 + krow[i]) * ld + off[i];
                if (tail && k0 + krow[i] > klast) src = reinterpret_cast<const uint16_t *>(kZeros);
            } else {
                src = p + (size_t)off[i] * ld + min(k0 + krow[i], klast - 7);
            }
            dma16(src, lds + (wave * kDma + i) * 1024);
        }
    }
};

__device__ __forceinline__ bf16x8 tr_frag(const unsigned char *lo, const unsigned char *hi)
{
    typedef __attribute__((address_space(3))) shortx4 lds4;
    const shortx4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(lo));
    const shortx4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4 *)(hi));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The fragment (16 rows of m or n x 32 k) of block blk, step ks of a stage: lane
// l holds k 8 (l / 16) .. + 7 of its row.  A: row l % 16 of 16 consecutive ones.
// B: blocks 2 i and 2 i + 1 share 32 rows so that MFMA row r of block 2 i + e is
// row 32 i + 8 (r / 4) + 4 e + r % 4: a lane's accumulators of the two blocks are
// then 8 consecutive n of one m.
template <int R, bool kStrided, bool kIsB>
__device__ __forceinline__ bf16x8 fragment(const unsigned char *t, int blk, int ks, int lane)
{
    const int r = lane & 15, g = lane >> 4;
    if (!kStrided) {
        const int row = kIsB ? 32 * (blk >> 1) + 8 * (r >> 2) + 4 * (blk & 1) + (r & 3) : 16 * blk + r;
        const int key = kIsB ? ((r & 3) | ((r >> 2 & 1) << 2)) : (r & 7);
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const quad *>(t + row * 128 + (((4 * ks + g) ^ key) * 16)));
    }
    // k rows 32 ks + 8 g + r / 4 and 4 on; columns in pieces of 4
    const int c = r & 3, k = 32 * ks + 8 * g + (r >> 2);
    const int slot = kIsB ? 4 * (blk >> 1) + c : 2 * blk + (c >> 1), half = kIsB ? (blk & 1) : (c & 1);
    const unsigned char *p = t + k * (R * 2) + ((slot ^ (4 * (k & 3) & (R / 8 - 1))) * 16) + half * 8;
    return tr_frag(p, p + 4 * R * 2);
}

// The workgroup's tile id: dealt to the XCDs in contiguous runs, so that
// neighbouring tiles, which share rows, meet in one L2.
__device__ __forceinline__ int tile_id()
{
    const int total = gridDim.x, xcd = blockIdx.x & 7, run = total >> 3, extra = total & 7;
    return xcd * run + min(xcd, extra) + (blockIdx.x >> 3);
}

// acc = the products of one TM x TN tile over k kbeg .. kend - 1 (4 waves, 2 x 2
// of them, 16-wide blocks); with kSums also A's column sums, in every row of
// accs (by a B operand of ones).
template <int TM, int TN, int kStages, bool kSA, bool kSB, bool kSums>
__device__ __forceinline__ void tile_products(const uint16_t *a, int lda, int M, int m0, const uint16_t *b, int ldb,
                                              int N, int n0, int kbeg, int kend, unsigned char *lds, int lane, int wave,
                                              bool sums, floatx4 (&acc)[TM / 32][TN / 32], floatx4 (&accs)[TM / 32])
{
    using TA = Tile<TM, kSA, false>;
    using TB = Tile<TN, kSB, true>;
    constexpr int kBM = TM / 32, kBN = TN / 32;
    constexpr int kStageBytes = TA::kBytes + TB::kBytes;
    constexpr int kLoads = TA::kDma + TB::kDma;   // transfers per wave and stage
    constexpr int kAhead = kStages - 1;
    const int wm = wave >> 1, wn = wave & 1;
    const int nst = (kend - kbeg + kStageK - 1) / kStageK;
    TA ta;
    TB tb;
    ta.init(m0, M, lda, wave, lane);
    tb.init(n0, N, ldb, wave, lane);
    const uint32_t base = lds_addr(lds);
    auto fetch = [&](int s) {
        const uint32_t buf = base + (uint32_t)(s % kStages) * kStageBytes;
        ta.fetch(a, lda, kbeg + s * kStageK, kend - 1, buf, wave);
        tb.fetch(b, ldb, kbeg + s * kStageK, kend - 1, buf + TA::kBytes, wave);
    };
#pragma unroll
    for (int i = 0; i < kBM; ++i) {
#pragma unroll
        for (int j = 0; j < kBN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
        accs[i] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    const bf16x8 one = __builtin_bit_cast(bf16x8, quad{0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u});
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
        if (s < nst) fetch(s);
    int buf = 0;
    for (int s = 0; s < nst; ++s) {
        if (s + kAhead <= nst) wait_vm<(kAhead - 1) * kLoads>();
        else wait_vm<0>();
        stage_barrier();
        // (the buffer of the stage before this one is free now)
        if (s + kAhead < nst) fetch(s + kAhead);
        unsigned char *sa = lds + buf * kStageBytes, *sb = sa + TA::kBytes;
        const int left = kend - (kbeg + s * kStageK);   // k of this stage
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            if (ks == 1 && left <= 32) break;
            bf16x8 fa[kBM], fb[kBN];
#pragma unroll
            for (int i = 0; i < kBM; ++i) fa[i] = fragment<TM, kSA, false>(sa, wm * kBM + i, ks, lane);
#pragma unroll
            for (int j = 0; j < kBN; ++j) fb[j] = fragment<TN, kSB, true>(sb, wn * kBN + j, ks, lane);
#pragma unroll
            for (int i = 0; i < kBM; ++i) {
#pragma unroll
                for (int j = 0; j < kBN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
                if (kSums && sums) accs[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(one, fa[i], accs[i], 0, 0, 0);
            }
        }
        buf = buf + 1 == kStages ? 0 : buf + 1;
    }
}

template <int TM, int TN, int kStages>
constexpr int ring_bytes() { return kStages * (TM + TN) * kStageK * 2; }

// One TM x TN tile of one split of K per workgroup, n fastest.
template <int TM, int TN, int kStages, bool kSA, bool kSB, int EPI>
__global__ __launch_bounds__(256, 2) void k_gemm_tiles(GemmArgs g)
{
    constexpr int kBM = TM / 32, kBN = TN / 32;   // 16-wide blocks per wave
    __shared__ __attribute__((aligned(1024))) unsigned char lds[ring_bytes<TM, TN, kStages>()];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    int id = tile_id();
    const int tn = id % g.tiles_n;
    id /= g.tiles_n;
    const int tm = id % g.tiles_m, z = id / g.tiles_m;
    const int m0 = tm * TM, n0 = tn * TN;
    const int kbeg = z * g.kchunk, kend = min(g.K, kbeg + g.kchunk);
    floatx4 acc[kBM][kBN], none[kBM];
    tile_products<TM, TN, kStages, kSA, kSB, false>(g.a, g.lda, g.M, m0, g.b, g.ldb, g.N, n0, kbeg, kend, lds, lane,
                                                    wave, false, acc, none);
    // lane: row m = 16 (block) + lane % 16, 8 consecutive n per pair of blocks
    float *cf = g.cf;
    if (EPI == kEpiF32 && g.splits > 1) cf += (size_t)z * g.M * g.ldc;
#pragma unroll
    for (int i = 0; i < kBM; ++i) {
        const int m = m0 + 16 * (wm * kBM + i) + (lane & 15);
        if (m >= g.M) continue;
#pragma unroll
        for (int j = 0; j < kBN; j += 2) {
            const int n = n0 + 16 * (wn * kBN + j) + 8 * (lane >> 4);
            if (n >= g.N) continue;
            floatx4 v0 = acc[i][j], v1 = acc[i][j + 1];
            if (EPI == kEpiF32) {
                if (g.bias) {
                    v0 += *reinterpret_cast<const floatx4 *>(g.bias + n);
                    v1 += *reinterpret_cast<const floatx4 *>(g.bias + n + 4);
                }
                floatx4 *dst = reinterpret_cast<floatx4 *>(cf + (size_t)m * g.ldc + n);
                dst[0] = v0;
                dst[1] = v1;
            } else {
                bf16x8 o;
                if (EPI == kEpiBiasReluBf16) {
                    v0 += *reinterpret_cast<const floatx4 *>(g.bias + n);
                    v1 += *reinterpret_cast<const floatx4 *>(g.bias + n + 4);
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (__bf16)fmaxf(e < 4 ? v0[e & 3] : v1[e & 3], 0.f);
                } else {
                    const shortx8 h = *reinterpret_cast<const shortx8 *>(g.mask + (size_t)m * g.ldm + n);
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (__bf16)(h[e] > 0 ? (e < 4 ? v0[e & 3] : v1[e & 3]) : 0.f);
                }
                *reinterpret_cast<bf16x8 *>(g.cb + (size_t)m * g.ldc + n) = o;
            }
        }
    }
}

// Weight gradients of several layers in one launch (256 rows of dY^T each):
// splits of the rows x jobs x tiles, every split's results in its own slab.  One
// launch instead of a GEMM, its sum and a bias sum per layer.
constexpr int kMaxJobs = 4;
struct DwGroup {
    DwJob job[kMaxJobs];
    int first[kMaxJobs + 1];   // tiles before job l
    int rows, chunk;
    int64_t slab;
    float *part;
};

template <int T, int kStages>
__global__ __launch_bounds__(256, 2) void k_dw_group(DwGroup g)
{
    constexpr int kB = T / 32, kM = kMlpHidden;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[ring_bytes<T, T, kStages>()];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    int id = tile_id();
    const int total = g.first[kMaxJobs], z = id / total;
    id -= z * total;
    int l = 0;
    while (id >= g.first[l + 1]) ++l;
    id -= g.first[l];
    const DwJob &job = g.job[l];
    const int tm = id % (kM / T), tn = id / (kM / T);
    const int m0 = tm * T, n0 = tn * T;
    const int kbeg = z * g.chunk, kend = min(g.rows, kbeg + g.chunk);
    floatx4 acc[kB][kB], accs[kB];
    const bool sums = tn == 0 && wn == 0;
    tile_products<T, T, kStages, true, true, true>(job.dy, kM, kM, m0, job.x, job.N, job.N, n0, kbeg, kend, lds, lane,
                                                   wave, sums, acc, accs);
    float *out = g.part + (size_t)z * g.slab;
#pragma unroll
    for (int i = 0; i < kB; ++i) {
        const int m = m0 + 16 * (wm * kB + i) + (lane & 15);
#pragma unroll
        for (int j = 0; j < kB; j += 2) {
            const int n = n0 + 16 * (wn * kB + j) + 8 * (lane >> 4);
            if (n >= job.N) continue;
            floatx4 *dst = reinterpret_cast<floatx4 *>(out + job.w + (size_t)m * job.N + n);
            dst[0] = acc[i][j];
            dst[1] = acc[i][j + 1];
        }
        if (sums && lane < 16) out[job.b + m] = accs[i][0];
    }
}

bool aligned16(const void *p) { return (uintptr_t)p % 16 == 0; }

template <int TM, int TN, int kStages, bool kSA, bool kSB, int EPI>
hipError_t launch_tiles(GemmArgs &g, hipStream_t s)
{
    g.tiles_m = (g.M + TM - 1) / TM;
    g.tiles_n = (g.N + TN - 1) / TN;
    const int64_t grid = (int64_t)g.tiles_m * g.tiles_n * g.splits;
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_gemm_tiles<TM, TN, kStages, kSA, kSB, EPI>), dim3((unsigned)grid), dim3(256), 0, s, g);
    return hipGetLastError();
}

template <bool kSA, bool kSB, int EPI>
hipError_t launch(GemmArgs &g, hipStream_t s)
{
    // The larger the tile, the fewer LDS reads per product, as long as the tiles
    // keep two workgroups on every CU: 128 x 128 from 384 tiles, 128 x 64 from 512
    // of those, else 64 x 64 (more stages in the ring for the smaller tiles, whose
    // stages are shorter).  Measured in us as 128 x 128 / 128 x 64 / 64 x 64:
    //   C 32768 x 512,  k-contiguous, K 4608 (1024 tiles): 173 / 217 / 282
    //   C 32768 x 4608, B k-strided,  K 512  (9216 tiles): 288 / 348 / 440
    //   C 512 x 4608, both k-strided, K 32768 in 3 (432 tiles): 173 / 308 / 402
    //   C 8192 x 512,   k-contiguous, K 4608 (256 tiles): 49 / 42 / 56
    //   C 16384 x 256,  k-contiguous, K 2112 (256 tiles): 28 / 23 / 29
    //   C 4096 x 256,   k-contiguous, K 2112 (64 tiles):  23 / 17 / 13
    // (the kernel before, one 64 x 64 tile at a time: 430, 765, 1520, -, -, 34)
    const int mb = (g.M + 127) / 128;
    const int64_t t128 = (int64_t)mb * ((g.N + 127) / 128) * g.splits;
    const int64_t t64 = (int64_t)mb * ((g.N + 63) / 64) * g.splits;
    if (t128 >= 384) return launch_tiles<128, 128, 2, kSA, kSB, EPI>(g, s);
    if (t64 >= 512) return launch_tiles<128, 64, 3, kSA, kSB, EPI>(g, s);
    return launch_tiles<64, 64, 4, kSA, kSB, EPI>(g, s);
}

}  // namespace

bool gemm_tiles_fit(bool strided_a, bool strided_b, const uint16_t *A, const uint16_t *B, int M, int N, int K, int lda,
                    int ldb, const void *bias, const void *mask, int ldm, const void *C, int ldc)
{
    if (M < 1 || N < 8 || N % 8 || K < 32 || lda % 8 || ldb % 8 || ldc % 8 || !aligned16(A) || !aligned16(B) ||
        !aligned16(C))
        return false;
    if ((bias && !aligned16(bias)) || (mask && (!aligned16(mask) || ldm % 8))) return false;
    if (strided_a && (M < 8 || M % 8)) return false;
    return (strided_a && strided_b) || K % 32 == 0;   // k-contiguous rows are read in whole steps
}

hipError_t gemm_dw_group(const DwJob *jobs, int n, int rows, float *part, int64_t slab_floats, size_t part_floats,
                         int *splits, hipStream_t s)
{
    if (n < 1 || n > kMaxJobs || rows < 1) return hipErrorInvalidValue;
    // 64 x 64 tiles in up to three splits (two workgroups per CU), from 2048 rows on
    // 128 x 128 in up to eleven (of at least 256 rows each), where the larger tile's
    // fewer LDS reads outweigh the sum of more slabs; near the line they differ
    // little.  The whole gradient with 64 and 128, us: 512 rows 36.5 and 38.1, 1024
    // 41.3 and 40.2, 2048 47.3 and 44.0, 4096 59.8 and 49.4, 16384 154 and 101.
    const int T = rows >= 2048 ? 128 : 64;
    DwGroup g = {};
    int tiles = 0;
    for (int l = 0; l < n; ++l) {
        if (!aligned16(jobs[l].dy) || !aligned16(jobs[l].x) || jobs[l].N % 8) return hipErrorInvalidValue;
        g.job[l] = jobs[l];
        g.first[l] = tiles;
        tiles += (kMlpHidden / T) * ((jobs[l].N + T - 1) / T);
    }
    for (int l = n; l <= kMaxJobs; ++l) g.first[l] = tiles;
    int sp = std::min((T == 64 ? 540 : 512) / tiles, rows / 256);
    sp = (int)std::min<int64_t>(sp, (int64_t)(part_floats / (size_t)slab_floats));
    sp = std::max(sp, 1);
    if (part_floats < (size_t)slab_floats) return hipErrorInvalidValue;
    g.rows = rows;
    g.chunk = ((rows + sp - 1) / sp + 31) / 32 * 32;
    g.slab = slab_floats;
    g.part = part;
    *splits = sp;
    if (T == 64)
        hipLaunchKernelGGL((k_dw_group<64, 4>), dim3(tiles * sp), dim3(256), 0, s, g);
    else
        hipLaunchKernelGGL((k_dw_group<128, 2>), dim3(tiles * sp), dim3(256), 0, s, g);
    return hipGetLastError();
}

hipError_t gemm_tiles(int variant, const uint16_t *A, const uint16_t *B, int M, int N, int K, int lda, int ldb,
                      const float *bias, const uint16_t *mask, int ldm, float *Cf, uint16_t *Cb, int ldc, int splits,
                      hipStream_t s)
{
    GemmArgs g = {};
    g.a = A;
    g.b = B;
    g.M = M;
    g.N = N;
    g.K = K;
    g.lda = lda;
    g.ldb = ldb;
    g.ldc = ldc;
    g.splits = splits;
    g.kchunk = ((K + splits - 1) / splits + 31) / 32 * 32;
    g.bias = bias;
    g.mask = mask;
    g.ldm = ldm;
    g.cf = Cf;
    g.cb = Cb;
    switch (variant) {
    case kGemmFwd: return launch<false, false, kEpiBiasReluBf16>(g, s);
    case kGemmDx: return launch<false, true, kEpiMaskBf16>(g, s);
    case kGemmDw:
    case kGemmTnF32: return launch<true, true, kEpiF32>(g, s);
    case kGemmNtF32: return launch<false, false, kEpiF32>(g, s);
    case kGemmNnF32: return launch<false, true, kEpiF32>(g, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gal
