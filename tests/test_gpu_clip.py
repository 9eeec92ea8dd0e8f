"""Clipping parity: triangle soups around the camera, most of whose triangles
cross the near plane or the guard band, many of them several planes at once (so
that a cluster holds more than one group of eight, and polygons of up to eight
vertices occur), bit for bit against the oracle, depth and winners."""
import numpy as np
import pytest

from paper_2306_07552_amd import scenegen as sg
from parity_util import compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tuning", [{}, {"block": 1024, "persistent": 1}, {"region": 32, "small_max": 64},
                                    {"lane_max": 0, "occlusion": 0}])
def test_clipped_triangle_soup(tuning):
    import torch
    print("case: clipped soup", tuning, flush=True)
    from oracle import oracle as O
    from paper_2306_07552_amd import gal
    cfg = sg.scaled_config(0, 10)
    scenes = sg.make_scene_set(cfg)
    rng = np.random.default_rng(12)
    verts, tris, rgb = [], [], []
    counts = [1, 7, 8, 9, 63, 64, 65, 200, 400, 3]
    for e, n in enumerate(counts):
        at = np.array([scenes.starts[e, 0, 0], scenes.starts[e, 0, 1], 1.1])
        # centres up to 3 m from the camera, sizes from 5 cm to 20 m
        c = at + rng.normal(size=(n, 1, 3)) * rng.uniform(0.05, 3.0, size=(n, 1, 1))
        v = c + rng.normal(size=(n, 3, 3)) * np.exp(rng.uniform(np.log(0.05), np.log(20.0), size=(n, 1, 1)))
        verts.append(v.reshape(-1, 3).astype(np.float32))
        tris.append(np.arange(3 * n, dtype=np.int32).reshape(n, 3))
        rgb.append(rng.integers(0, 256, size=(n, 3), dtype=np.uint8))
    scenes.verts, scenes.tris = np.concatenate(verts), np.concatenate(tris)
    scenes.tri_rgb, scenes.tri_plane = np.concatenate(rgb), None
    scenes.tri_offset = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    scenes.vert_offset = 3 * scenes.tri_offset
    robot, consts = sg.make_robot_for(cfg), sg.config_constants(cfg)
    b = gal.Batch(robot, scenes, consts, color=True)
    b.set_tuning(**tuning)
    b.counters(True)
    ob = O.OracleBatch(robot, scenes, consts, color=True)
    out = b.alloc_outputs()
    for k in range(4):
        a = sg.actions(cfg, k, num_envs=10)
        b.step(torch.from_numpy(a).cuda(), out)
        torch.cuda.synchronize()
        compare_step(b, ob, out, ob.step(a), label=f"step {k}")
    assert b.counters_read()["tris_clipped"] > 400
