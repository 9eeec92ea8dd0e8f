"""Infinities in the last row of a sum over rows whose count is no multiple of the
kernels' steps: the rows that fill the last step up must not meet them (0 times an
infinity is NaN, where the sum is infinite)."""
import numpy as np
import pytest

from test_gpu_surrogate import bf16_bits, bits_to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(64, 64, 33), (72, 136, 70), (136, 264, 127), (2104, 3080, 97), (8200, 520, 95),
                                   (66, 64, 70)])
@pytest.mark.parametrize("side", ["a", "b"])
def test_gemm_with_an_infinite_last_row(M, N, K, side):
    """C = A^T B where the last row of one operand holds infinities: exact where the
    other operand's last row is not 0, at the edges of each tile shape and in the
    general kernel (66 columns)."""
    import torch
    print("case: infinite last row", M, N, K, side, flush=True)
    from paper_2306_07552_amd import gal
    rng = np.random.default_rng([M, N, K])
    a, b = rng.normal(size=(K, M)), rng.normal(size=(K, N))
    a[-1], b[-1] = np.where(a[-1] < 0, -1.0, 1.0), np.where(b[-1] < 0, -1.0, 1.0)
    inf = a if side == "a" else b
    inf[-1, ::3] = np.inf
    ab, bb = bf16_bits(a), bf16_bits(b)
    A, B = bits_to_f64(ab), bits_to_f64(bb)
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    gal.gemm_test(5, torch.from_numpy(ab.view(np.int16)).cuda(), torch.from_numpy(bb.view(np.int16)).cuda(), M, N, K,
                  M, N, c, N)
    got = c.cpu().numpy().astype(np.float64)
    want = A[:-1].T @ B[:-1] + np.outer(A[-1], B[-1])
    far = np.isinf(want)
    assert far.any() and not np.isnan(want).any()
    assert np.array_equal(got[far], want[far])
    bound = (np.abs(A[:-1]).T @ np.abs(B[:-1]) + np.abs(np.outer(A[-1], B[-1]))) * (K + 2) * 2.0 ** -24 + 1e-30
    assert np.all(np.abs(got[~far] - want[~far]) <= bound[~far])


@pytest.mark.parametrize("rows", [1, 17, 40, 4097])
def test_gradients_with_an_infinite_last_row(rows):
    """A network that passes one input on, whose second layer overflows for the last
    row: the weight gradients of the logit and of the layers above the overflow are
    infinite, and nothing that the other rows alone determine is touched.  (The loss is
    NaN, by its term z y of an infinite z and a label 0.)"""
    import torch
    print("case: gradients with an infinite last row", rows, flush=True)
    from paper_2306_07552_amd import gal
    m = gal.Mlp(max_rows=rows, seed=1)
    lay = gal.Mlp.layout()
    w = np.zeros(m.num_params, np.float32)
    for l, v in enumerate((1.0, 2.0 ** 100, 1.0, 1.0, 1.0)):
        w[lay[2 * l][0]] = v
    m.set_weights(w)
    x = np.zeros((rows, 2112), np.float32)
    x[:, 0] = 2.0 ** -100
    x[-1, 0] = 2.0 ** 60
    g, loss = torch.empty(m.num_params, device="cuda"), torch.empty(1, device="cuda")
    m.gradients(torch.from_numpy(bf16_bits(x).view(np.int16)).cuda(), torch.zeros(rows, device="cuda"), 3.0, grads=g,
                loss=loss)
    got = g.cpu().numpy()
    assert np.isnan(loss.item())
    p = {}
    for i, (off, shape) in enumerate(lay):
        p[i] = got[off:off + int(np.prod(shape))].reshape(shape)
    head, head_b = p[8].ravel(), p[9].ravel()
    assert head[0] == np.inf and np.all(head[1:] == 0)
    # 1 / rows times the sigmoids: of 1, and of infinity in the last row
    q = ((rows - 1) / (1 + np.exp(-1.0)) + 1) / rows
    assert abs(head_b[0] - q) <= 1e-5 * q
    for l in (2, 3):   # unit 0 of the layers fed by the infinite unit: its own gradient, and zeros beside it
        assert p[2 * l][0, 0] == np.inf and np.all(p[2 * l][0, 1:] == 0), l
        assert abs(p[2 * l + 1][0] - q) <= 1e-2 * q
