"""Work tables kept from one call for the next of the same shape: a context
that runs calls of other shapes, kinds, bin capacities and occupancy in
between gives the results of a context that runs each call alone."""
import numpy as np
import pytest
import torch

from tests.gpu_common import make_pair
from tests.tiny import random_params, tiny_scene
from paper_2304_05735_amd import GRAD

pytestmark = pytest.mark.gpu


def _calls(gid, rays):
    def loss(n, cap):
        def run(g):
            g.debug_bin_capacity(cap)
            l = g.loss_and_grad([gid], [n])
            return [np.asarray(l), g.get_params(gid, GRAD)]
        return run

    def forward(n):
        def run(g):
            out = g.field_forward(gid, rays[:n].contiguous())
            g.sync()
            return [x.cpu().numpy() for x in out]
        return run

    def backward(n):
        def run(g):
            one = torch.ones(n, 3, device="cuda")
            r = rays[:n].contiguous()
            torch.cuda.synchronize()
            out = g.field_backward(gid, r, one, None, one[:, 0].contiguous())
            g.sync()
            return [out.cpu().numpy()]
        return run
    return dict(l64=loss(64, 0), l130=loss(130, 0), l64c=loss(64, 1 << 20), f50=forward(50),
                f200=forward(200), b50=backward(50), b200=backward(200))


@pytest.mark.parametrize("use_graph", [0, 2])
def test_alternating_shapes(use_graph):
    print(f"alternating shapes graph {use_graph}", flush=True)
    frames, box = tiny_scene()

    def make():
        g, _, gid = make_pair(4, 16, 200, 12, 32, 64, frames, box, use_graph=use_graph)
        g.other = g.add_object(box["instance"] + 1, box["t"], box["yaw"], box["half"])
        for cam, rgb, mask, depth in frames:
            g.add_keyframe(cam, rgb, np.where(mask == box["instance"], mask + 1, mask), depth)
        return g, _, gid

    rng = np.random.default_rng(2)
    o = rng.normal(size=(200, 3))
    o = 1.5 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-1, 1, (200, 3)) * np.asarray(box["half"]) - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = torch.from_numpy(np.concatenate([o, d, np.full((200, 1), 0.9), np.full((200, 1), 2.1)],
                                           1).astype(np.float32)).cuda()
    g, _, gid = make()
    p = random_params(g.object_info(gid).n_grid_params, 8, seed=1).astype(np.float32)
    calls = _calls(gid, rays)
    bits = np.packbits(np.arange(262144) % 3 == 0, bitorder="little")
    alone = {}
    for occ in (None, bits):
        for name, run in calls.items():
            h, _, hid = make()
            h.set_params(hid, p)
            if occ is not None:
                h.set_occupancy(hid, occ)
            alone[name, occ is not None] = run(h)
    order = [("l64", 0), ("l64", 0), ("l130", 0), ("l64", 0), ("b50", 0), ("f50", 0), ("f50", 1), ("b50", 1),
             ("l64", 1), ("l64", 0), ("b200", 0), ("l64", 0), ("f200", 0), ("l64c", 0), ("l64", 0),
             ("f200", 0), ("b50", 0), ("b200", 0), ("l130", 1), ("l130", 0)]
    g.set_params(gid, p)
    for i, (name, occ) in enumerate(order):
        g.set_occupancy(gid, bits if occ else None)
        for a, b in zip(alone[name, bool(occ)], calls[name](g)):
            assert np.array_equal(a, b), (i, name, occ)
        if i % 7 == 3:
            g.train(3, [g.other])  # tables of another object's training in between
