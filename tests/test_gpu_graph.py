"""Step graphs that replace each other while their launches are still queued
(training calls without stats do not wait): the same weights as eager steps,
bit for bit (every region of the small tables has one workgroup)."""
import numpy as np
import pytest

from tests.gpu_common import make_pair
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("streams", [1, 2])
def test_graphs_replaced_without_waits(streams):
    print(f"graphs replaced, streams {streams}", flush=True)
    frames, box = tiny_scene()
    out = []
    for graph in (0, 2):
        g, _, a = make_pair(4, 16, 200, 12, 32, 64, frames, box, use_graph=graph, streams=streams)
        b = g.add_object(2, box["t"], box["yaw"], box["half"])
        for cam, rgb, mask, depth in frames:
            g.add_keyframe(cam, rgb, np.where(mask == 1, 2, mask), depth)
        for i in (a, b):
            g.set_params(i, random_params(g.object_info(i).n_grid_params, 8, seed=i).astype(np.float32))
        for steps in (8, 2, 1, 9, 3, 40, 2):
            g.train(steps, [a, b], stats=False)
        g.train(8, [a, b], [150, 90], stats=False)
        g.train(4, [b], [300], stats=False)
        out.append([g.get_params(i) for i in (a, b)])
        assert g.object_info(a).step == 73 and g.object_info(b).step == 77
    for x, y in zip(*out):
        assert np.isfinite(x).all() and np.array_equal(x, y)
