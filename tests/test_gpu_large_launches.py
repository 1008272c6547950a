"""Calls whose kernels run over their work in several launches or rounds
(2^26 points of a density query, 2^28 samples of the live masks): the same
results as calls on parts, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2304_05735_amd as pk
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


def test_query_beyond_one_launch():
    print("large query", flush=True)
    s = torch.cuda.Stream()
    g = pk.Context(pk.default_config(n_levels=1, log2_table_size=10), stream=s)
    i = g.add_object(1, np.zeros(3), 0.0, np.array([0.4, 0.3, 0.35]))
    g.set_params(i, random_params(g.object_info(i).n_grid_params, 2, seed=1).astype(np.float32))
    n = (1 << 26) + 65
    with torch.cuda.stream(s):
        xyz = torch.rand(n, 3, device="cuda").sub_(0.5)
        sig = g.query_density(i, xyz)
        for a, b in ((0, 1000), (n - 1065, n - 64), (n - 66, n)):
            assert torch.equal(sig[a:b], g.query_density(i, xyz[a:b].contiguous())), (a, b)
        assert bool((sig > 0).all()) and sig[-300:].unique().numel() > 100


def test_live_masks_beyond_one_round():
    print("large live masks", flush=True)
    frames, box = tiny_scene()
    n, k = 1 << 20, 3  # 3 x 2^27 samples
    g = pk.Context(pk.default_config(n_levels=1, log2_table_size=10, samples_per_ray=128,
                                     rays_per_step=n, autotune=0))
    ids = [g.add_object(1 + j, box["t"], box["yaw"], box["half"]) for j in range(k)]
    for j in range(k):
        cam, rgb, mask, depth = frames[j]
        g.add_keyframe(cam, rgb, np.where(mask == 1, 1 + j, 0), depth)
    cells = np.arange(262144)
    for j in ids:
        g.set_params(j, random_params(g.object_info(j).n_grid_params, 2, seed=j).astype(np.float32))
        g.set_occupancy(j, np.packbits((cells // (5 + j)) % 3 > 0, bitorder="little"))
    together = g.loss_and_grad(ids)
    apart = np.concatenate([g.loss_and_grad([j]) for j in ids])
    assert np.isfinite(together).all() and np.unique(together).size == k
    assert np.array_equal(together, apart), (together, apart)
