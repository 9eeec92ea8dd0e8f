"""The tiled GEMM at its edges (through gal_mlp_gemm_test) against numpy on the
same BF16 values: one row, remainders of each tile size, K at a step's, a
stage's and the ring's ends, both strided and contiguous operands, leading
dimensions wider than the tile, the sizes where each tile shape is chosen, and
rows that are not 16-byte aligned (the general kernel).  The bound is the FP32
accumulation's: K + 2 roundings of 2^-24 of the terms' absolute sum."""
import numpy as np
import pytest

from test_gpu_surrogate import bf16_bits, bits_to_f64, oracle_net

pytestmark = pytest.mark.gpu

CASES = [(3, 1, 8, 32, 0), (3, 63, 64, 96, 0), (3, 65, 72, 2112, 8), (3, 129, 136, 64, 0), (3, 300, 256, 544, 16),
         (3, 2100, 3080, 96, 0), (3, 8200, 520, 160, 0), (3, 70, 64, 96, 4),
         (4, 1, 8, 32, 0), (4, 130, 72, 288, 8), (4, 2100, 3080, 64, 0), (4, 8200, 520, 96, 0),
         (5, 8, 8, 32, 0), (5, 64, 136, 33, 0), (5, 72, 64, 63, 8), (5, 136, 264, 65, 0), (5, 256, 2112, 1000, 0),
         (5, 2104, 3080, 97, 0), (5, 8200, 520, 70, 0), (5, 66, 64, 100, 0)]


@pytest.mark.parametrize("variant,M,N,K,pad", CASES)
def test_gemm_tiles_match_numpy(variant, M, N, K, pad):
    import torch
    print(f"case: gemm tiles variant {variant} {M}x{N}x{K} pad {pad}", flush=True)
    from paper_2306_07552_amd import gal
    rng = np.random.default_rng([variant, M, N, K])

    def operand(rows, cols):
        bits = bf16_bits(rng.normal(size=(rows, cols + pad)))
        return torch.from_numpy(bits.view(np.int16)).cuda(), bits_to_f64(bits)[:, :cols], cols + pad

    ta, A, lda = operand(K, M) if variant == 5 else operand(M, K)
    tb, B, ldb = operand(N, K) if variant == 3 else operand(K, N)
    A = A.T if variant == 5 else A
    B = B.T if variant == 3 else B
    c = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    gal.gemm_test(variant, ta, tb, M, N, K, lda, ldb, c, N)
    got = c.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - A @ B) <= (np.abs(A) @ np.abs(B)) * (K + 2) * 2.0 ** -24 + 1e-30)


@pytest.mark.parametrize("rows,shift", [(1, 0), (15, 0), (17, 0), (300, 0), (300, 1), (2048, 0), (4100, 0)])
def test_mlp_gradient_row_counts(rows, shift):
    """The surrogate's loss and gradient at one row, the remainders of its row
    tiles, the sizes where its weight gradients change tiles and its middle part
    the rows per workgroup, and (shift 1) inputs whose rows are not 16-byte
    aligned, against the FP64 oracle, which rounds to BF16 at the same points: 1e-3
    relative L2 per tensor (an occasional rounding that FP32 sums flip, 2^-8 of one
    value), 4e-3 below 16 rows, where one flip weighs more."""
    import torch
    print("case: mlp gradients", rows, shift, flush=True)
    from paper_2306_07552_amd import gal
    rng = np.random.default_rng([rows, shift])
    m = gal.Mlp(max_rows=rows, seed=3)
    x = bf16_bits((rng.uniform(size=(rows, 2112)) < 0.3) * rng.choice([1.0, 0.5], size=(rows, 2112)))
    y = (rng.uniform(size=rows) < 0.5).astype(np.float32)
    flat = torch.zeros(rows * 2112 + 8, dtype=torch.int16, device="cuda")
    flat[shift:shift + rows * 2112] = torch.from_numpy(x.view(np.int16).ravel()).cuda()
    tx = flat[shift:shift + rows * 2112].view(rows, 2112)
    g, loss = torch.empty(m.num_params, device="cuda"), torch.empty(1, device="cuda")
    m.gradients(tx, torch.from_numpy(y).cuda(), 3.0, grads=g, loss=loss)
    got = g.cpu().numpy().astype(np.float64)
    ref_loss, dW, db = oracle_net(m.get_weights()).backward(bits_to_f64(x), y, 3.0)
    tol = 1e-3 if rows >= 16 else 4e-3
    assert abs(loss.item() - ref_loss) <= tol * (1 + abs(ref_loss))
    refs = [t for l in range(5) for t in (dW[l], db[l])]
    for (off, shape), ref in zip(gal.Mlp.layout(), refs):
        d = np.linalg.norm(got[off:off + ref.size] - ref.ravel())
        assert d <= tol * max(np.linalg.norm(ref), 1e-30), (off, shape, d)
