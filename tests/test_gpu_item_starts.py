"""One workgroup per item, more items than are resident at once: the setting
`order` chooses whether the items are started by their times in the step before
(1, a new batch's) or in the static order (0), which must change no bit: with
graph replay, colour, split items and after resets, each case with a launch that
is asserted to follow the times."""
import numpy as np
import pytest

from paper_2306_07552_amd import scenegen as sg

pytestmark = pytest.mark.gpu


def make(n, color):
    from paper_2306_07552_amd import gal
    cfg = sg.scaled_config(0, n)
    scenes = sg.make_scene_set(cfg)
    return cfg, gal.Batch(sg.make_robot_for(cfg), scenes, sg.config_constants(cfg), color=color)


@pytest.mark.parametrize("n,color,tuning", [
    (1300, False, {}),
    (1300, True, {"graph": 1}),
    (1000, False, {"region": 64, "split": 400, "graph": 1}),   # one item per env, four of a split one
    (700, True, {"region": 32, "block": 256}),                 # four items per env
])
def test_items_started_by_their_times(n, color, tuning):
    import torch
    print("case: item starts", n, color, tuning, flush=True)
    cfg, b = make(n, color)
    _, ref = make(n, color)
    b.set_tuning(**tuning)
    ref.set_tuning(**dict(tuning, graph=0, order=0))
    info, plain = b.launch_info(color), ref.launch_info(color)
    assert info["items"] == plain["items"] > info["resident"] > 0, info
    assert info["by_time"] == 1 and plain["by_time"] == 0
    out, want = b.alloc_outputs(), ref.alloc_outputs()
    acts = torch.empty((n, 9), device="cuda")
    mask = torch.from_numpy((np.arange(n) % 3 == 0).astype(np.uint8)).cuda()
    for k in range(6):
        if k == 2:
            b.reset(mask)
            ref.reset(mask)
        if k == 4:
            b.reset()
            ref.reset()
        acts.copy_(torch.from_numpy(sg.actions(cfg, k, num_envs=n)))
        b.step(acts, out)
        ref.step(acts, want)
        torch.cuda.synchronize()
        for name in want:
            assert torch.equal(out[name], want[name]), (k, name)


def test_order_setting():
    """What each setting launches: the times are followed by the queue at any
    number of items, by one workgroup per item above the resident ones."""
    import torch  # noqa: F401
    print("case: order setting", flush=True)
    _, b = make(1300, False)
    _, few = make(40, False)
    for persistent in (0, 1):
        for order in (0, 1):
            for batch, more in ((b, True), (few, False)):
                batch.set_tuning(persistent=persistent, order=order)
                info = batch.launch_info()
                assert (info["items"] > info["resident"]) == more
                assert info["by_time"] == (order if more or persistent else 0)
    with pytest.raises(RuntimeError):
        b.launch_info(color=True)


@pytest.mark.parametrize("n,lanes", [(4096, 64), (8192, 32)])
def test_ordering_is_hidden_beside_the_robot_step(n, lanes):
    """The sort of the items' times runs in one workgroup beside the robot step's
    and the raster waits for it: at thousands of items it may not lengthen the
    robot stage by more than 15 us (about 0.5 of its 31 and 62 us; a sort of 14 ns
    an item took 46 and 92 us more).  The shortest of 40 steps of each, in turn."""
    import torch
    print("case: ordering hidden", n, lanes, flush=True)
    cfg, b = make(n, False)
    out = b.alloc_outputs()
    acts = torch.from_numpy(sg.actions(cfg, 0, num_envs=n)).cuda()
    best = [1e9, 1e9]
    for k in range(43):
        for order in (0, 1):
            b.set_tuning(order=order, robot_lanes=lanes)
            assert b.launch_info()["by_time"] == order
            b.profile(True)
            b.step(acts, out)
            torch.cuda.synchronize()
            b.profile(False)
            _, robot, _, _ = b.profile_read_stages()
            if k >= 3:
                best[order] = min(best[order], robot)
    print("robot stage, ms: static %.4f, by time %.4f" % tuple(best), flush=True)
    assert best[1] - best[0] < 0.015


@pytest.mark.parametrize("n,items", [(513, 8208), (2048, 32768), (2049, 32784)])
def test_items_by_the_ten_thousand(n, items):
    """More items than the sort keeps in registers, its largest count, and one env
    more, which keeps the static order."""
    import torch
    from paper_2306_07552_amd import gal
    print("case: items by the ten thousand", n, flush=True)
    cfg = sg.scaled_config(0, n)
    scenes = sg.make_scene_set(cfg)
    scenes.res = np.full(n, 128, np.int32)
    robot, consts = sg.make_robot_for(cfg), sg.config_constants(cfg)
    b, ref = gal.Batch(robot, scenes, consts), gal.Batch(robot, scenes, consts)
    b.set_tuning(region=32)
    info = b.launch_info()
    assert info["items"] == items and info["by_time"] == (items <= 32768)
    out, want = b.alloc_outputs(), ref.alloc_outputs()
    for k in range(3):
        acts = torch.from_numpy(sg.actions(cfg, k, num_envs=n)).cuda()
        b.step(acts, out)
        ref.step(acts, want)
        torch.cuda.synchronize()
        for name in want:
            assert torch.equal(out[name], want[name]), (k, name)
