"""Densities at points (four waves to 64 points, levels and units shared among
them) against the oracle, at the edges of a block, of the levels' quarters and
of each network depth, with the bars of the density parity test; and boxes
whose size the division by a stored reciprocal does and does not cover: scaled
by a power of two, box and points have the same unit positions, so the same
densities bit for bit."""
import numpy as np
import pytest

import oracle
from tests.gpu_common import assert_fwd_close, make_pair
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,layers", [(1, 1), (3, 2), (5, 3), (8, 1), (9, 2), (16, 1)])
def test_density_blocks(L, layers):
    frames, box = tiny_scene()
    g, o, gid = make_pair(L, 16, 300, 11, 32, 16, frames, box, mlp_layers=layers)
    ob = o.objects[gid]
    p = random_params(oracle.grid_params(ob.lv), 2 * L, seed=L, layers=layers).astype(np.float32)
    g.set_params(gid, p)
    ob.params[:] = p.astype(np.float64)
    rng = np.random.default_rng(L)
    for n in (1, 63, 64, 65, 200):
        print(f"density L {L} layers {layers} n {n}", flush=True)
        xyz = (rng.uniform(-1.1, 1.1, (n, 3)) * box["half"]).astype(np.float32)
        assert_fwd_close(g.query_density(gid, xyz), o.query_density(gid, xyz), what=f"sigma {n}")


@pytest.mark.parametrize("k", [-80, -62, -59, 57, 61, 80])
def test_box_scales(k):
    print(f"box scale 2^{k}", flush=True)
    half = np.array([0.4375, 0.3, 0.7], np.float32)
    rng = np.random.default_rng(5)
    xyz = (rng.uniform(-1.1, 1.1, (500, 3)) * half).astype(np.float32)
    out = []
    for scale in (1.0, 2.0 ** k):
        h = (half * np.float32(scale)).astype(np.float32)
        box = dict(instance=1, t=(0.0, 0.0, 0.0), yaw=0.0, half=h)
        g, _, gid = make_pair(6, 16, 300, 11, 32, 16, [], box)
        g.set_params(gid, random_params(g.object_info(gid).n_grid_params, 12, seed=3).astype(np.float32))
        out.append(g.query_density(gid, (xyz * np.float32(scale)).astype(np.float32)))
    assert np.unique(out[0]).size > 100
    assert np.array_equal(out[0], out[1])
