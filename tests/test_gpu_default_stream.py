"""A context made with torch's default stream (whose handle is NULL): calls on
device tensors follow the torch work queued before them and precede the torch
work queued after them, without a wait of the host, also when the work tables
are in place from the call before."""
import numpy as np
import pytest
import torch

import paper_2304_05735_amd as pk
from paper_2304_05735_amd.field import RomapFieldFn
from tests.tiny import random_params

pytestmark = pytest.mark.gpu


def _late(x, big):
    """x, ready only after some milliseconds of other work on torch's stream."""
    y = big
    for _ in range(8):
        y = torch.mm(y, big)
    return x + torch.where(torch.isnan(y[:1, :1]), 0.0, 0.0).reshape([1] * x.dim())


def test_default_stream_is_ordered():
    print("default stream", flush=True)
    g = pk.Context(pk.default_config(n_levels=8, max_res=256, log2_table_size=14, samples_per_ray=64,
                                     autotune=0), stream=torch.cuda.default_stream())
    i = g.add_object(1, np.zeros(3), 0.2, np.array([0.4, 0.3, 0.35]))
    p0 = torch.from_numpy(random_params(g.object_info(i).n_grid_params, 16, seed=1).astype(np.float32)).cuda()
    rng = np.random.default_rng(3)
    n = 300
    o = rng.normal(size=(n, 3))
    o = 1.5 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-0.3, 0.3, (n, 3)) - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = torch.from_numpy(np.concatenate([o, d, np.full((n, 1), 0.9), np.full((n, 1), 2.1)],
                                           1).astype(np.float32)).cuda()
    xyz = torch.from_numpy((rng.uniform(-0.3, 0.3, (5000, 3))).astype(np.float32)).cuda()
    big = torch.full((4096, 4096), 1.0 / 4096, device="cuda")

    def pass_(slow):
        def late(x):
            return _late(x, big) if slow else x
        p = late(p0).detach().requires_grad_(True)
        r = late(rays)
        rgb, depth, tend = RomapFieldFn.apply(p, r, g, i)
        total = late(rgb).pow(2).sum(1) + depth - tend  # reads the outputs, and makes the adjoints late
        if not slow:
            torch.cuda.synchronize()
        total.sum().backward()
        g.set_params(i, p0.cpu().numpy())
        sig = g.query_density(i, late(xyz))
        out = [x.detach().clone() for x in (rgb, depth, tend, total, p.grad, sig)]
        torch.cuda.synchronize()
        return out
    ref = pass_(False)
    assert ref[4].abs().max() > 0 and ref[5].max() > 0
    for k in range(3):
        for a, b in zip(ref[:4] + ref[5:], (x := pass_(True))[:4] + x[5:]):
            assert torch.equal(a, b), k
        # overfull bins add in any order: the gradient to a sum's FP32 rounding
        assert (ref[4] - x[4]).abs().max() <= 1e-5 * ref[4].abs().max(), k
