"""GPU parity of the policy at the batch sizes where its kernels' splits change:
one sample, fewer samples than workgroups, one more than a whole round of
them, a ragged last round.  Every encoder layer, the heads and the actions of
sampled envs against the FP64 oracle, on images that hold every kind of depth
value (zero, one, no hit, beyond 24 bits)."""
import numpy as np
import pytest

from test_gpu_policy import check_policy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 255, 257, 600])
def test_policy_batch_sizes(n):
    import torch
    print("case: policy sizes", n, flush=True)
    from paper_2306_07552_amd import gal
    rng = np.random.default_rng(n)
    depth = rng.integers(0, 1 << 24, size=(n, 128, 128), dtype=np.uint32)
    depth[:, :40] = 0xFFFFFF
    depth[:, 100:104, ::3] = 0
    depth[:, 104:108, ::3] = 1
    depth[:, 60, :] = 0x1000003          # beyond 24 bits: clamped
    state = rng.normal(size=(n, 10)).astype(np.float32)
    noise = rng.normal(size=(n, 9)).astype(np.float32)
    pol = gal.Policy(n, act_dim=9, seed=4)
    theta = pol.get_weights()
    d = torch.from_numpy(depth.view(np.int32)).cuda()
    act = torch.empty((n, 9), device="cuda")
    val, lp = torch.empty(n, device="cuda"), torch.empty(n, device="cuda")
    pol.act(d, torch.from_numpy(state).cuda(), act, noise=torch.from_numpy(noise).cuda(), value=val, logp=lp)
    torch.cuda.synchronize()
    envs = np.unique(np.array([0, n // 3, n // 2, min(255, n - 1), min(256, n - 1), n - 1]))
    check_policy(pol, theta, np.minimum(depth[envs], 0xFFFFFF), state[envs], noise[envs].astype(np.float64),
                 act.cpu().numpy()[envs], val.cpu().numpy()[envs], lp.cpu().numpy()[envs], envs)
