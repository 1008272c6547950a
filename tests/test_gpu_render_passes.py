"""A view of more than 2^20 pixels, which is rendered in two passes over one
ray buffer, equals its crops bit for bit on both sides of the boundary."""
import numpy as np
import pytest

import paper_2304_05735_amd as pk
import scenes
from tests.tiny import random_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,f", [(pk.PREC_FP32, 1000.0), (pk.PREC_BF16, 5000.0)])
def test_view_of_two_passes(prec, f):
    print(f"two passes, prec {prec}", flush=True)
    W, H = 1063, 1001
    assert W * H > 1 << 20
    g = pk.Context(pk.default_config(n_levels=4, base_res=16, max_res=64, log2_table_size=12,
                                     samples_per_ray=32, precision=prec))
    gid = g.add_object(1, np.zeros(3), 0.3, np.array([0.4, 0.3, 0.35]))
    g.set_params(gid, random_params(g.object_info(gid).n_grid_params, 8, seed=3).astype(np.float32))
    # the object across the lower edge, so that the last rows hit it
    cam = scenes.camera(scenes.look_at((1.2, 0.3, 0.2), (0, 0, 0)), W, H, f)
    cam = dict(cam, cy=cam["cy"] + 400.0 if f < 2000 else cam["cy"])
    full = g.render(gid, cam)
    assert (full[2][988:] > 0).any()  # in the second pass
    for x0, y0, w, h in ((0, 970, W, 31), (500, 0, 67, H), (996, 900, 67, 101)):
        crop = g.render(gid, dict(cam, W=w, H=h, cx=cam["cx"] - x0, cy=cam["cy"] - y0))
        for a, b in zip(full, crop):
            assert np.array_equal(a[y0:y0 + h, x0:x0 + w], b), (x0, y0)
