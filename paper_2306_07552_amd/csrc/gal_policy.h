// Internal definitions of the policy network that consumes the depth stack
// (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gal {

constexpr int kPolicyRes = 128;      // depth image edge the encoder takes
constexpr int kPolicyFeat = 512;     // encoder features
constexpr int kPolicyProprio = 7;    // joint angles fed to the heads beside the features
constexpr int kPolicyMaxAct = 32;    // action dimensions
constexpr int kPolicyCUs = 256;      // compute units of the chip: workgroups of the persistent kernels

// The three convolutions of the encoder on n depth images: BF16 weights in the
// parameter layout (rows of (ky, kx, channel)), FP32 biases; NHWC BF16 maps of
// each layer out.
struct EncoderWeights {
    const uint16_t *w1, *w2, *w3;
    const float *b1, *b2, *b3;
};
hipError_t encoder_forward(const uint32_t *depth, const EncoderWeights &w, int n, uint16_t *h1, uint16_t *h2,
                           uint16_t *h3, hipStream_t s);

// The fully connected layer Y = bf16(relu(X W^T + b)) (X [rows][K], W [N][K]):
// one pass, or split over K into ws when the tiles alone leave the chip idle;
// the heads then add the splits in order (`parts`: splits slabs of `stride`
// values, splits 1 = Y is already in out).  The workspace needed: at most
// fc_splits(rows, N, K) * rows * N floats.
struct FcParts {
    const float *part;
    int splits;
    int64_t stride;
    const float *bias;
};
int fc_splits(int rows, int N, int K);
hipError_t fc_forward(const uint16_t *x, const uint16_t *W, const float *bias, int rows, int N, int K, float *ws,
                      size_t ws_floats, uint16_t *out, FcParts *parts, hipStream_t s);
// The heads on the features h (written from fc first where it holds splits).
hipError_t policy_heads(const FcParts &fc, uint16_t *h, const float *state, const float *aw, const float *ab,
                        const float *vw, const float *vb, const float *log_std, int A, int n_envs, const float *noise,
                        float *actions, float *value, float *logp, hipStream_t s);

// Backward of the three convolutions from d3 (the gradient of the third's
// pre-activation, BF16 [n][12][12][32]): the FP32 gradients of conv1 W, b,
// conv2 W, b into g12 and of conv3 W, b into g3 (parameter layout).  d2 (BF16
// [n][14][14][64]) receives the second layer's gradient; wt
// (encoder_backward_weights() BF16 values) and part (encoder_backward_floats())
// are scratch.
size_t encoder_backward_floats();
size_t encoder_backward_weights();
hipError_t encoder_backward(const uint32_t *depth, const uint16_t *h1, const uint16_t *h2, const uint16_t *d3,
                            uint16_t *d2, const uint16_t *w2, const uint16_t *w3, uint16_t *wt, int n, float *part,
                            size_t part_floats, float *g12, float *g3, hipStream_t s);
// out[i] = sum over splits of part[z][i] (FP32, n values each) in a fixed order.
hipError_t sum_parts(const float *part, int splits, int64_t n, float *out, hipStream_t s);
// The loss per sample: a row of 2 A + 4 values each (gradients of the heads'
// outputs, loss terms) and the features' gradient d4 (BF16).
hipError_t ppo_heads(const FcParts &fc, uint16_t *h, const float *state, const float *aw, const float *ab,
                     const float *vw, const float *vb, const float *log_std, int A, int S, const float *actions,
                     const float *old_logp, const float *adv, const float *ret, float clip, float vcoef, float *rows,
                     uint16_t *d4, hipStream_t s);
// The heads' parameter gradients, the fully connected layer's bias gradient and
// the loss statistics, summed over the samples through part in a fixed order.
struct HeadGrads {
    float *aw, *ab, *vw, *vb, *ls, *fcb;
};
hipError_t ppo_head_grads(const uint16_t *h, const float *state, const float *rows, const uint16_t *d4,
                          const float *log_std, int A, int S, float ecoef, const HeadGrads &g, float *stats, float *part,
                          size_t part_floats, hipStream_t s);
hipError_t gae(const float *rew, const float *val, const uint8_t *done, const float *last, int T, int N, float gamma,
               float lam, float *adv, float *ret, hipStream_t s);

}  // namespace gal
