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


@pytest.mark.parametrize("S", [16, 256, 512, 1024])
def test_ppo_gradient_is_the_mean_of_its_samples(S):
    """The gradient over S samples drawn from 16 different ones is the mean of
    the 16 one-sample gradients, weighted by their counts: one sample per
    workgroup, fewer, and loops of two and four.  1 / S is a power of two, so
    every BF16 value is an exact multiple of the one-sample call's and only the
    FP32 sums differ: over up to 2^20 terms of random sign their rounding grows as
    2^10 2^-24 of the terms' root sum of squares, and 1e-3 relative L2 leaves 16
    times that for cancellation."""
    import torch
    from oracle import oracle_policy as OP
    from test_gpu_ppo import ppo_case
    print("case: ppo gradients as a mean", S, flush=True)
    from paper_2306_07552_amd import gal
    small, _, _, _, (out, act, old, adv, ret) = ppo_case(torch, 16, 36)
    pol = gal.Policy(S, act_dim=9)
    pol.set_weights(small.get_weights())
    depth = out["depth"].reshape(16, -1)
    old, adv, ret = (torch.from_numpy(x).cuda() for x in (old, adv, ret))
    g = torch.empty(pol.num_params, device="cuda")
    one = np.zeros((16, pol.num_params))
    for k in range(16):
        pol.ppo_gradients(depth[k].contiguous(), out["state"][k:k + 1].contiguous(), act[k:k + 1].contiguous(),
                          old[k:k + 1], adv[k:k + 1], ret[k:k + 1], grads=g)
        one[k] = g.cpu().numpy()
    idx = np.random.default_rng(S).integers(0, 16, size=S)
    i = torch.from_numpy(idx).cuda()
    pol.ppo_gradients(depth[i].contiguous(), out["state"][i].contiguous(), act[i].contiguous(), old[i].contiguous(),
                      adv[i].contiguous(), ret[i].contiguous(), grads=g)
    got, ref = g.cpu().numpy().astype(np.float64), one[idx].mean(axis=0)
    off = 0
    for name, shp in OP.layout(9):
        n = int(np.prod(shp))
        a, b = got[off:off + n], ref[off:off + n]
        assert np.linalg.norm(a - b) <= 1e-3 * max(np.linalg.norm(b), 1e-30), name
        off += n


@pytest.mark.parametrize("A,S", [(1, 1), (1, 40), (11, 33), (12, 257), (32, 40), (9, 4097)])
def test_ppo_head_gradients(A, S):
    """The heads' gradients, the fc bias's and the statistics at the smallest and
    largest action counts, at the group size of the summing kernel and one more,
    and with one and four samples per wave, in FP64 from the device's own features
    and feature gradients.  FP32 sums of 519 terms leave the means within 2^-14 of
    their terms, hence log-densities of up to 32 actions within about 1e-3 and the
    ratios with them: 3e-3 relative L2; ratios stay off the clip range's ends."""
    import torch
    print("case: ppo head gradients", A, S, flush=True)
    from oracle import oracle_policy as OP
    from paper_2306_07552_amd import gal
    rng = np.random.default_rng([A, S])
    pol = gal.Policy(S, act_dim=A, seed=7)
    theta = pol.get_weights()
    P = OP.unpack(theta, A)
    depth = torch.from_numpy(rng.integers(0, 1 << 24, size=(S, 128, 128), dtype=np.int32)).cuda()
    state = rng.normal(size=(S, 10)).astype(np.float32)
    noise = rng.normal(size=(S, A)).astype(np.float32)
    st = torch.from_numpy(state).cuda()
    act, lp = torch.empty((S, A), device="cuda"), torch.empty(S, device="cuda")
    pol.act(depth, st, act, noise=torch.from_numpy(noise).cuda(), logp=lp)
    ratio = np.array([0.7, 0.9, 1.1, 1.3])[np.arange(S) % 4]
    old = (lp.cpu().numpy() - np.log(ratio)).astype(np.float32)
    adv, ret = rng.normal(size=S).astype(np.float32), 3 + rng.normal(size=S).astype(np.float32)
    g, stats = torch.empty(pol.num_params, device="cuda"), torch.empty(4, device="cuda")
    pol.ppo_gradients(depth, st, act, *(torch.from_numpy(x).cuda() for x in (old, adv, ret)), grads=g, stats=stats)
    G = OP.unpack(g.cpu().numpy(), A)
    h4 = (pol.activations(4).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    f = np.concatenate([h4, state[:, 3:10].astype(np.float64)], axis=1)
    mean, V = OP.heads(h4, state[:, 3:10], P)
    std = np.exp(P["log_std"].astype(np.float64))
    z = (act.cpu().numpy().astype(np.float64) - mean) / std
    r = np.exp((-0.5 * z * z - np.log(std)).sum(1) - 0.5 * A * np.log(2 * np.pi) - old)
    s1, s2 = r * adv, np.clip(r, 0.8, 1.2) * adv
    dl = np.where(s1 <= s2, -adv * r, 0.0) / S
    gm, gv = dl[:, None] * z / std, (V - ret) / S
    df = (gm @ P["actor.w"].astype(np.float64) + gv[:, None] * P["critic.w"].astype(np.float64))[:, :512]
    want = {"actor.w": gm.T @ f, "actor.b": gm.sum(0), "critic.w": gv @ f, "critic.b": gv.sum(keepdims=True),
            "log_std": (dl[:, None] * (z * z - 1)).sum(0) - 0.01, "fc.b": np.where(h4 > 0, df, 0.0).sum(0)}
    for name, w in want.items():
        # d4 is BF16: 2^-9 per term more for the bias of the fully connected layer
        tol = 3e-3 + (2.0 ** -8 if name == "fc.b" else 0.0)
        terms = np.linalg.norm(w) + (np.abs(gm).sum() / S ** 0.5 if name in ("actor.b", "log_std") else 0.0)
        assert np.linalg.norm(G[name] - w.reshape(G[name].shape)) <= tol * terms, name
    t = stats.cpu().numpy()
    for got, w in zip(t, (-np.minimum(s1, s2).mean(), ((V - ret) ** 2).mean(),
                          (P["log_std"] + 0.5 * (1 + np.log(2 * np.pi))).sum(), r.mean())):
        assert abs(got - w) <= 3e-3 * (1 + abs(w))
