"""Buffers at the least alignment that the entry points take: depth at any word and
colour at any byte give the bits of aligned ones; surrogate inputs at any BF16 value
give one gradient, on every run and as a replayed graph."""
import numpy as np
import pytest

from paper_2306_07552_amd import scenegen as sg
from test_gpu_surrogate import bf16_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [1, 2, 3])
@pytest.mark.parametrize("res", [[64] * 6, [8, 24, 40, 72, 104, 128]])
def test_image_buffers_at_any_address(shift, res):
    import torch
    print("case: image buffers", shift, res, flush=True)
    from paper_2306_07552_amd import gal
    cfg = sg.scaled_config(0, 6)
    scenes = sg.make_scene_set(cfg)
    scenes.res = np.asarray(res, np.int32)
    robot, consts = sg.make_robot_for(cfg), sg.config_constants(cfg)
    a = torch.from_numpy(sg.actions(cfg, 0, num_envs=6)).cuda()
    b, ref = (gal.Batch(robot, scenes, consts, color=True) for _ in range(2))
    n = b.depth_pixels
    depth = torch.full((n + 8,), 7, dtype=torch.int32, device="cuda")
    rgb = torch.full((3 * n + 16,), 7, dtype=torch.uint8, device="cuda")
    out, want = b.alloc_outputs(), ref.alloc_outputs()
    out["depth"] = depth[shift:shift + n]
    out["rgb"] = rgb[shift:shift + 3 * n].view(n, 3)
    for k in range(3):
        b.step(a, out)
        ref.step(a, want)
        torch.cuda.synchronize()
        assert torch.equal(out["depth"], want["depth"]) and torch.equal(out["rgb"], want["rgb"]), k
    # nothing around them is written
    assert torch.all(depth[:shift] == 7) and torch.all(depth[shift + n:] == 7)
    assert torch.all(rgb[:shift] == 7) and torch.all(rgb[shift + 3 * n:] == 7)
    # depth alone
    out = b.alloc_outputs()
    out["depth"] = depth[shift:shift + n]
    out.pop("rgb")
    b.step(a, out)
    ref.step(a, want)
    torch.cuda.synchronize()
    assert torch.equal(out["depth"], want["depth"])
    assert torch.all(depth[:shift] == 7) and torch.all(depth[shift + n:] == 7)


@pytest.mark.parametrize("rows", [100, 4096])
def test_unaligned_inputs_give_one_gradient(rows):
    import torch
    print("case: unaligned gradient", rows, flush=True)
    from paper_2306_07552_amd import gal
    rng = np.random.default_rng(rows)
    m = gal.Mlp(max_rows=rows, seed=2)
    x = torch.from_numpy(bf16_bits(rng.normal(size=(rows, 2112))).view(np.int16)).cuda()
    flat = torch.empty(rows * 2112 + 8, dtype=torch.int16, device="cuda")
    tx = flat[3:3 + rows * 2112].view(rows, 2112)
    tx.copy_(x)
    y = torch.from_numpy((rng.uniform(size=rows) < 0.5).astype(np.float32)).cuda()

    def gradients(x, g, loss):
        m.gradients(x, y, 3.0, grads=g, loss=loss)

    def empty():
        return torch.empty(m.num_params, device="cuda"), torch.empty(1, device="cuda")

    first, aligned = empty(), empty()
    gradients(tx, *first)
    gradients(x, *aligned)
    # the same sums, split differently: FP32 roundings of up to `rows` terms
    d = (first[0] - aligned[0]).double()
    assert d.norm() <= 1e-5 * aligned[0].double().norm()
    for _ in range(20):
        again = empty()
        gradients(tx, *again)
        assert torch.equal(again[0], first[0]) and torch.equal(again[1], first[1])
    g, loss = empty()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        gradients(tx, g, loss)
    torch.cuda.current_stream().wait_stream(stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gradients(tx, g, loss)
    for _ in range(4):
        g.zero_()
        other = empty()
        gradients(x, *other)   # own work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g, first[0]) and torch.equal(loss, first[1])
