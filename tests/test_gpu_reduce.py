"""MLP gradient summed over one to hundreds of work items of a call: n equal
rays give n times the gradient of one.  A ray's terms are the same in every
copy, so only the float32 sums differ: below 1e-4 of n times the largest
component, while one item lost or taken twice moves it by 1/300 or more."""
import numpy as np
import pytest
import torch

from tests.gpu_common import make_pair
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,layers", [(32, 1), (64, 2), (128, 3)])
@pytest.mark.parametrize("n", [4, 5, 252, 257, 1028, 2300])
def test_record_sums(n, N, layers):
    print(f"record sums {n} N {N} layers {layers}", flush=True)
    frames, box = tiny_scene()
    g, _, gid = make_pair(3, 16, 128, 10, N, 16, frames, box, mlp_layers=layers)
    info = g.object_info(gid)
    g.set_params(gid, random_params(info.n_grid_params, 6, seed=n, layers=layers).astype(np.float32))
    ray = np.array([[0.9, 0.7, 1.1, -0.55, -0.45, -0.7, 0.2, 3.0]], np.float32)
    ray[0, 3:6] /= np.linalg.norm(ray[0, 3:6])

    def mlp_grad(k):
        rays = torch.from_numpy(np.repeat(ray, k, 0)).cuda()
        d_rgb = torch.tensor([[0.3, -0.2, 0.5]]).repeat(k, 1).cuda()
        d_depth, d_tend = torch.full((k,), 0.1).cuda(), torch.full((k,), -0.4).cuda()
        torch.cuda.synchronize()
        out = g.field_backward(gid, rays, d_rgb, d_depth, d_tend)
        g.sync()
        return out[info.n_grid_params:].double().cpu().numpy()

    one, many = mlp_grad(1), mlp_grad(n)
    assert np.abs(one).max() > 0
    assert np.abs(many - n * one).max() <= 1e-4 * n * np.abs(one).max()
