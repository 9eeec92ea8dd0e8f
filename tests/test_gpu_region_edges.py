"""Triangles over the edges of their image or region, at every width of the
last double tile, in a batch whose regions are halved (few items), one whose
regions are halved twice and one whose regions stay: neither the spans of a bbox row nor the right half of a tile
may touch another pixel.  Bit for bit against the oracle, depth and winners."""
import numpy as np
import pytest

from paper_2306_07552_amd import scenegen as sg
from parity_util import compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("repeat", [1, 15, 26])
@pytest.mark.parametrize("res,tuning", [
    ([8, 16, 24, 40, 56, 72, 88, 104, 120, 128], {}),
    ([8, 16, 24, 32, 8, 16, 24, 32, 64, 128], {"region": 32, "persistent": 1}),
    ([8, 24, 40, 56, 72, 88, 104, 120, 112, 48], {"small_max": 1, "lane_max": 0}),
    ([8, 24, 40, 56, 72, 88, 104, 120, 112, 48], {"small_max": 65536}),
])
def test_triangles_over_region_edges(res, tuning, repeat):
    import torch
    print("case: region edges", res, tuning, repeat, flush=True)
    res = res * repeat
    from oracle import oracle as O
    from paper_2306_07552_amd import gal
    cfg = sg.scaled_config(0, len(res))
    scenes = sg.make_scene_set(cfg)
    scenes.res = np.asarray(res, np.int32)
    rng = np.random.default_rng(21)
    verts, tris, rgb, counts = [], [], [], [600 if e < 10 else 60 for e in range(len(res))]
    for e, n in enumerate(counts):
        # all around the camera, at any distance: slivers, single pixels, halves of the image
        d = rng.normal(size=(n, 1, 3))
        d /= np.linalg.norm(d, axis=-1, keepdims=True)
        dist = np.exp(rng.uniform(np.log(0.3), np.log(8.0), size=(n, 1, 1)))
        at = np.array([scenes.starts[e, 0, 0], scenes.starts[e, 0, 1], 1.1])
        size = dist * np.exp(rng.uniform(np.log(0.003), np.log(0.8), size=(n, 1, 1)))
        v = at + d * dist + rng.normal(size=(n, 3, 3)) * size
        verts.append(v.reshape(-1, 3).astype(np.float32))
        tris.append(np.arange(3 * n, dtype=np.int32).reshape(n, 3))
        rgb.append(rng.integers(0, 256, size=(n, 3), dtype=np.uint8))
    scenes.verts, scenes.tris = np.concatenate(verts), np.concatenate(tris)
    scenes.tri_rgb, scenes.tri_plane = np.concatenate(rgb), None
    scenes.tri_offset = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    scenes.vert_offset = 3 * scenes.tri_offset
    robot, consts = sg.make_robot_for(cfg), sg.config_constants(cfg)
    for color in (False, True):
        b = gal.Batch(robot, scenes, consts, color=color)
        b.set_tuning(**tuning)
        ob = O.OracleBatch(robot, scenes, consts, color=color)
        out = b.alloc_outputs()
        for k in range(2):
            a = sg.actions(cfg, k, num_envs=len(res))
            b.step(torch.from_numpy(a).cuda(), out)
            torch.cuda.synchronize()
            compare_step(b, ob, out, ob.step(a), label=f"color {color} step {k}")
