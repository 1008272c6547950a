"""Rendering over the hit rays alone: a view equals its crops bit for bit
(a pixel's outputs do not depend on which rays share its launch), where the
hits fill several launches, leave a ragged last one, or none at all; device
outputs equal host ones, with any of them left out."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2304_05735_amd as pk
import scenes
from tests.tiny import random_params

pytestmark = pytest.mark.gpu


def _ctx(N, prec):
    g = pk.Context(pk.default_config(n_levels=4, base_res=16, max_res=64, log2_table_size=12,
                                     samples_per_ray=N, precision=prec))
    gid = g.add_object(1, np.zeros(3), 0.3, np.array([0.4, 0.3, 0.35]))
    g.set_params(gid, random_params(g.object_info(gid).n_grid_params, 8, seed=3).astype(np.float32))
    return g, gid


def _cam(W, H, f, eye=(1.2, 0.3, 0.2), at=(0, 0, 0)):
    return scenes.camera(scenes.look_at(eye, at), W, H, f)


@pytest.mark.parametrize("W,H,N,f,prec", [
    (200, 180, 128, 1500.0, pk.PREC_FP32),  # every pixel hits: 36000 rays, two launches
    (301, 133, 64, 180.0, pk.PREC_BF16), (64, 3, 32, 40.0, pk.PREC_FP32)])
def test_view_equals_its_crops(W, H, N, f, prec):
    print(f"render {W}x{H} N {N}", flush=True)
    g, gid = _ctx(N, prec)
    cam = _cam(W, H, f)
    full = g.render(gid, cam)
    assert full[2].max() > 0.0
    step = 67
    for x0 in range(0, W, step):
        w = min(step, W - x0)
        crop = g.render(gid, dict(cam, W=w, cx=cam["cx"] - x0))
        for a, b in zip(full, crop):
            assert np.array_equal(a[:, x0:x0 + w], b), x0


def test_no_hit_and_device_outputs():
    print("render no hit, device outputs", flush=True)
    g, gid = _ctx(64, pk.PREC_FP32)
    for x in g.render(gid, _cam(37, 21, 30.0, at=(2.4, 0.6, 0.4))):
        assert not x.any()
    cam = _cam(41, 30, 60.0)
    rgb, depth, opac = g.render(gid, cam)
    c = pk.make_camera(cam)
    dev = [torch.full(s, float("nan"), device="cuda") for s in ((30, 41, 3), (30, 41), (30, 41))]
    torch.cuda.synchronize()
    for keep in ((1, 1, 1), (0, 1, 0), (0, 0, 1), (1, 0, 0)):
        ptr = [C.c_void_p(t.data_ptr()) if k else None for t, k in zip(dev, keep)]
        assert pk.lib().romap_render(g.h, gid, C.byref(c), *ptr, 1) == pk.ROMAP_OK
        g.sync()
        for t, k, ref in zip(dev, keep, (rgb, depth, opac)):
            if k:
                assert np.array_equal(t.cpu().numpy(), ref)
                t.fill_(float("nan"))
        torch.cuda.synchronize()
