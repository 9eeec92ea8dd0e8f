"""One workgroup per item, more items than are resident at once: the items are
started in the order of their times in the step before, which must change no
bit, with and without graph replay, after a state reset and with split items."""
import pytest

from paper_2306_07552_amd import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,color,tuning", [
    (600, False, {}),              # 512 resident
    (300, True, {"graph": 1}),     # 256 resident
    (200, False, {"region": 64, "split": 50, "graph": 1}),   # 4 or 16 items per env
])
def test_measured_order_keeps_the_bits(n, color, tuning):
    import torch
    print("case: item order", n, color, tuning, flush=True)
    from paper_2306_07552_amd import gal
    cfg = sg.scaled_config(0, n)
    scenes = sg.make_scene_set(cfg)
    robot, consts = sg.make_robot_for(cfg), sg.config_constants(cfg)
    b = gal.Batch(robot, scenes, consts, color=color)
    ref = gal.Batch(robot, scenes, consts, color=color)
    b.set_tuning(**tuning)
    ref.set_tuning(persistent=1, order=0)
    out, want = b.alloc_outputs(), ref.alloc_outputs()
    acts = torch.empty((n, 9), device="cuda")
    for k in range(5):
        acts.copy_(torch.from_numpy(sg.actions(cfg, k, num_envs=n)))
        b.step(acts, out)
        ref.step(acts, want)
        torch.cuda.synchronize()
        for name in want:
            assert torch.equal(out[name], want[name]), (k, name)
