// Host runtime of the collision-surrogate MLP (declared in include/gal.h):
// parameters, training step (forward, logistic loss, backward, Adam) and
// inference, all on the device with the MFMA kernels of k_gemm.hip, k_mlp.hip,
// k_mlp_train.hip and k_sur_infer.hip.
#include "gal.h"
#include "gal_mlp.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <random>
#include <string>
#include <vector>

namespace gal {
int api_fail(int code, const char *fmt, ...);
}

namespace {

#define MLP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return gal::api_fail(GAL_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr int kDims[6] = {gal::kMlpIn, gal::kMlpHidden, gal::kMlpHidden, gal::kMlpHidden,
                          gal::kMlpHidden, 1};

}  // namespace

struct gal_mlp {
    std::vector<void *> allocs;
    int32_t max_rows = 0;
    int64_t off_w[5], off_b[5], n_params = 0;
    float *w = nullptr, *m = nullptr, *v = nullptr, *g = nullptr;
    uint16_t *wb = nullptr;
    uint16_t *wi = nullptr;     // inference copy of the matrix layers (fragment order)
    uint16_t *wf = nullptr, *wt = nullptr;   // training copies of layers 2..4 (forward, transposed)
    uint16_t *h[4] = {nullptr, nullptr, nullptr, nullptr};    // h[1..3]
    uint16_t *dp[4] = {nullptr, nullptr, nullptr, nullptr};   // pre-activation gradients of layers 1..4
    float *z = nullptr, *loss = nullptr;
    float *head_part = nullptr; // the logit's gradients and the loss, per workgroup
    float *part = nullptr;      // inference: the first layer's partial sums
    float *dw_part = nullptr;   // split-K partial sums of the weight gradients
    size_t dw_part_floats = 0;
    int64_t t = 0;
    ~gal_mlp()
    {
        for (void *p : allocs) (void)hipFree(p);
    }
    template <class T>
    int alloc(T **out, size_t count)
    {
        void *p = nullptr;
        const size_t bytes = std::max<size_t>(count * sizeof(T), 16);
        if (hipMalloc(&p, bytes) != hipSuccess)
            return gal::api_fail(GAL_ENOMEM, "hipMalloc(%zu bytes) failed", bytes);
        allocs.push_back(p);
        *out = static_cast<T *>(p);
        return GAL_OK;
    }
};

extern "C" {

int gal_mlp_num_params(int64_t *n)
{
    if (!n) return gal::api_fail(GAL_EINVAL, "null argument");
    int64_t c = 0;
    for (int l = 0; l < 5; ++l) c += (int64_t)kDims[l + 1] * kDims[l] + kDims[l + 1];
    *n = c;
    return GAL_OK;
}

int gal_mlp_create(int32_t max_rows, uint64_t seed, gal_mlp **out)
{
    if (!out || max_rows < 1 || max_rows > (1 << 22)) return gal::api_fail(GAL_EINVAL, "bad arguments");
    *out = nullptr;
    gal_mlp *m = new gal_mlp();
    m->max_rows = max_rows;
    int64_t off = 0;
    for (int l = 0; l < 5; ++l) {
        m->off_w[l] = off;
        off += (int64_t)kDims[l + 1] * kDims[l];
        m->off_b[l] = off;
        off += kDims[l + 1];
    }
    m->n_params = off;
    int rc;
    if ((rc = m->alloc(&m->w, off)) || (rc = m->alloc(&m->m, off)) || (rc = m->alloc(&m->v, off)) ||
        (rc = m->alloc(&m->g, off)) || (rc = m->alloc(&m->wb, off)) ||
        (rc = m->alloc(&m->wi, gal::sur_infer_layout_elems())) ||
        (rc = m->alloc(&m->wf, gal::mlp_mid_weights())) || (rc = m->alloc(&m->wt, gal::mlp_mid_weights())) ||
        (rc = m->alloc(&m->z, max_rows)) || (rc = m->alloc(&m->head_part, gal::mlp_mid_part_floats())) ||
        (rc = m->alloc(&m->part, gal::sur_infer_part_floats_max(max_rows))) ||
        (rc = m->alloc(&m->dw_part, (m->dw_part_floats = (size_t)gal::kMaxDwSplits * kDims[1] * kDims[0]))) ||
        (rc = m->alloc(&m->loss, 1))) {
        delete m;
        return rc;
    }
    for (int l = 0; l < 4; ++l)
        if ((l > 0 && (rc = m->alloc(&m->h[l], (size_t)max_rows * gal::kMlpHidden))) ||
            (rc = m->alloc(&m->dp[l], (size_t)max_rows * gal::kMlpHidden))) {
            delete m;
            return rc;
        }
    // He-uniform initialisation of the weights, zero biases
    std::vector<float> host(off, 0.0f);
    std::mt19937_64 rng(seed);
    for (int l = 0; l < 5; ++l) {
        const float lim = std::sqrt(6.0f / (float)kDims[l]);
        std::uniform_real_distribution<float> U(-lim, lim);
        for (int64_t i = 0; i < (int64_t)kDims[l + 1] * kDims[l]; ++i) host[m->off_w[l] + i] = U(rng);
    }
    int rc2 = gal_mlp_set_weights(m, host.data(), (size_t)off);
    if (rc2) {
        delete m;
        return rc2;
    }
    *out = m;
    return GAL_OK;
}

int gal_mlp_set_weights(gal_mlp *m, const float *host, size_t count)
{
    if (!m || !host) return gal::api_fail(GAL_EINVAL, "null argument");
    if ((int64_t)count != m->n_params) return gal::api_fail(GAL_EINVAL, "need %lld parameters", (long long)m->n_params);
    MLP_TRY(hipMemcpy(m->w, host, sizeof(float) * count, hipMemcpyHostToDevice));
    MLP_TRY(hipMemset(m->m, 0, sizeof(float) * count));
    MLP_TRY(hipMemset(m->v, 0, sizeof(float) * count));
    MLP_TRY(gal::mlp_to_bf16(m->w, (int64_t)count, m->wb, nullptr));
    MLP_TRY(gal::mlp_refresh_copies(m, nullptr));
    MLP_TRY(hipDeviceSynchronize());
    m->t = 0;
    return GAL_OK;
}

int gal_mlp_get_weights(gal_mlp *m, float *host, size_t count)
{
    if (!m || !host) return gal::api_fail(GAL_EINVAL, "null argument");
    if ((int64_t)count != m->n_params) return gal::api_fail(GAL_EINVAL, "need %lld parameters", (long long)m->n_params);
    MLP_TRY(hipDeviceSynchronize());
    MLP_TRY(hipMemcpy(host, m->w, sizeof(float) * count, hipMemcpyDeviceToHost));
    return GAL_OK;
}

}  // extern "C"

namespace gal {

int mlp_max_rows(const gal_mlp *m) { return m->max_rows; }

// the inference and training copies of the matrix layers, after the BF16 weights changed
hipError_t mlp_refresh_copies(gal_mlp *m, hipStream_t s)
{
    hipError_t e = mlp_mid_layout(m->wb + m->off_w[1], m->wb + m->off_w[2], m->wb + m->off_w[3], m->wf, m->wt, s);
    if (e != hipSuccess) return e;
    return sur_infer_layout(m->wb + m->off_w[0], m->wb + m->off_w[1], m->wb + m->off_w[2],
                            m->wb + m->off_w[3], m->wi, s);
}

// inference: the inputs x, or (x null) the features of the batch envs
// described by `src` computed on the fly; logits into z (may be null),
// routing flags and counts with route
int mlp_infer_rows(gal_mlp *m, const uint16_t *x, const SurInferArgs *src, int rows, float *z,
                   const RouteArgs *route, hipStream_t s, float *part)
{
    SurInferArgs a = src ? *src : SurInferArgs{};
    a.t.w0 = m->wi;
    a.t.b0 = m->w + m->off_b[0];
    for (int l = 0; l < 4; ++l) {
        a.t.w[l] = l < 3 ? m->wi + (size_t)kMlpIn * kMlpHidden + (size_t)l * kMlpHidden * kMlpHidden
                         : m->wb + m->off_w[4];
        a.t.b[l] = m->w + m->off_b[l + 1];
    }
    a.x = x;
    a.rows = rows;
    a.part = part ? part : m->part;
    a.z = z;
    a.route = route ? 1 : 0;
    if (route) a.ra = *route;
    MLP_TRY(sur_infer(a, s));
    return GAL_OK;
}

// The loss and its gradient over rows inputs into m->loss and m->g, and into
// loss_out and grads (may be null): the first layer, everything up to the
// pre-activation gradients, all weight gradients, their sums.
int mlp_gradients_rows(gal_mlp *m, const uint16_t *x, const float *y, int rows, float pos_w, float *grads,
                       float *loss_out, hipStream_t s)
{
    MLP_TRY(mlp_gemm(kGemmFwd, x, m->wb + m->off_w[0], rows, kMlpHidden, kMlpIn, kMlpIn, kMlpIn, m->w + m->off_b[0],
                     nullptr, 0, nullptr, m->h[1], kMlpHidden, s));
    MlpMidArgs a = {};
    a.h1 = m->h[1];
    a.h2 = m->h[2];
    a.h3 = m->h[3];
    for (int l = 0; l < 4; ++l) a.dp[l] = m->dp[l];
    a.wf = m->wf;
    a.wt = m->wt;
    for (int l = 0; l < 3; ++l) a.b[l] = m->w + m->off_b[l + 1];
    a.w5 = m->wb + m->off_w[4];
    a.b5 = m->w + m->off_b[4];
    a.y = y;
    a.rows = rows;
    a.pos_w = pos_w;
    a.part = m->head_part;
    int slabs = 0, splits = 0;
    MLP_TRY(mlp_mid(a, &slabs, s));
    // the weight gradients.  The first layer's, where the inputs are not 16-byte
    // aligned, comes from the general GEMM straight into m->g; its bias gradient then
    // rides on a product with the next layer's input, which lands in the slabs'
    // unused place of the first layer's weights
    const bool aligned = (uintptr_t)x % 16 == 0;
    DwJob jobs[4];
    for (int l = 0; l < 4; ++l)
        jobs[l] = DwJob{m->dp[l], l == 0 ? x : m->h[l], kDims[l], m->off_w[l], m->off_b[l]};
    if (!aligned) {
        jobs[0].x = m->h[1];
        jobs[0].N = kMlpHidden;
        MLP_TRY(mlp_gemm(kGemmDw, m->dp[0], x, kMlpHidden, kMlpIn, rows, kMlpHidden, kMlpIn, nullptr, nullptr, 0,
                         m->g + m->off_w[0], nullptr, kMlpIn, s, m->dw_part, m->dw_part_floats));
        if (grads)
            MLP_TRY(hipMemcpyAsync(grads, m->g, sizeof(float) * m->off_b[0], hipMemcpyDeviceToDevice, s));
    }
    MLP_TRY(gemm_dw_group(jobs, 4, rows, m->dw_part, m->off_w[4], m->dw_part_floats, &splits, s));
    MLP_TRY(mlp_grad_sum(m->dw_part, splits, aligned ? 0 : m->off_b[0], m->off_w[4], m->head_part, slabs, m->g, grads,
                         m->loss, loss_out, s));
    return GAL_OK;
}

}  // namespace gal

extern "C" {

int gal_mlp_forward(gal_mlp *m, const uint16_t *x_dev, int32_t rows, float *logits_dev, void *stream)
{
    if (!m || !x_dev || rows < 0 || rows > m->max_rows) return gal::api_fail(GAL_EINVAL, "bad arguments");
    if ((uintptr_t)x_dev % 16) return gal::api_fail(GAL_EINVAL, "x_dev must be 16-byte aligned");
    hipStream_t s = (hipStream_t)stream;
    return gal::mlp_infer_rows(m, x_dev, nullptr, rows, logits_dev ? logits_dev : m->z, nullptr, s);
}

int gal_mlp_gradients(gal_mlp *m, const uint16_t *x_dev, const float *labels_dev, int32_t rows,
                      float pos_weight, float *grads_dev, float *loss_dev, void *stream)
{
    if (!m || !x_dev || !labels_dev || rows < 1 || rows > m->max_rows)
        return gal::api_fail(GAL_EINVAL, "bad arguments");
    hipStream_t s = (hipStream_t)stream;
    return gal::mlp_gradients_rows(m, x_dev, labels_dev, rows, pos_weight, grads_dev, loss_dev, s);
}

int gal_mlp_train_step(gal_mlp *m, const uint16_t *x_dev, const float *labels_dev, int32_t rows,
                       float pos_weight, float lr, float *loss_dev, void *stream)
{
    if (!m || !x_dev || !labels_dev || rows < 1 || rows > m->max_rows || !(lr > 0.0f))
        return gal::api_fail(GAL_EINVAL, "bad arguments");
    hipStream_t s = (hipStream_t)stream;
    int rc = gal::mlp_gradients_rows(m, x_dev, labels_dev, rows, pos_weight, nullptr, loss_dev, s);
    if (rc) return rc;
    m->t += 1;
    MLP_TRY(gal::mlp_adam(m->w, m->m, m->v, m->g, m->n_params, lr, 0.9f, 0.999f, 1e-8f, m->t, m->wb, s));
    MLP_TRY(gal::mlp_refresh_copies(m, s));
    return GAL_OK;
}

int gal_mlp_gemm_test(int32_t variant, const uint16_t *a_dev, const uint16_t *b_dev, int32_t M,
                      int32_t N, int32_t K, int32_t lda, int32_t ldb, float *c_dev, int32_t ldc,
                      void *stream)
{
    if (variant < gal::kGemmNtF32 || variant > gal::kGemmTnF32 || !a_dev || !b_dev || !c_dev)
        return gal::api_fail(GAL_EINVAL, "bad arguments");
    MLP_TRY(gal::mlp_gemm(variant, a_dev, b_dev, M, N, K, lda, ldb, nullptr, nullptr, 0, c_dev,
                          nullptr, ldc, (hipStream_t)stream));
    return GAL_OK;
}

void gal_mlp_destroy(gal_mlp *m) { delete m; }

}  // extern "C"
