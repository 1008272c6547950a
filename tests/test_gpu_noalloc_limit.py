"""The most rays that the allocation-free forward takes: all but small tables
of its 64 MiB hold rays and encodings, one ray more is refused, and the results
are those of the allocating forward, with and without skipped samples."""
import numpy as np
import pytest
import torch

import paper_2304_05735_amd as pk
from tests.gpu_common import make_pair
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,L,occ", [(32, 1, True), (64, 2, False), (64, 16, True), (128, 1, True)])
def test_noalloc_limit(N, L, occ):
    print(f"noalloc limit N {N} L {L}", flush=True)
    frames, box = tiny_scene()
    g, _, gid = make_pair(L, 16, 64, 12, N, 64, frames, box)
    g.set_params(gid, random_params(g.object_info(gid).n_grid_params, 2 * L, seed=N).astype(np.float32))
    if occ:
        g.set_occupancy(gid, np.packbits(np.arange(262144) % 5000 < 2000, bitorder="little"))
    per = 64 + 8 * L * N
    hi = (64 << 20) // per + 1
    rng = np.random.default_rng(N)
    o = rng.normal(size=(hi, 3))
    o = 1.5 * o / np.linalg.norm(o, axis=1, keepdims=True)
    d = rng.uniform(-1, 1, (hi, 3)) * np.asarray(box["half"]) - o
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    rays = torch.from_numpy(np.concatenate([o, d, np.full((hi, 1), 0.9), np.full((hi, 1), 2.1)],
                                           1).astype(np.float32)).cuda()
    same = [torch.full(s, float("nan"), device="cuda") for s in ((hi, 3), (hi,), (hi,))]
    torch.cuda.synchronize()
    for n in range(hi, 0, -1):
        try:
            g.field_forward_noalloc(gid, rays[:n], *[x[:n] for x in same])
            break
        except pk.RomapError as e:
            assert e.code == pk.ROMAP_E_INVALID_ARG
    assert n < hi and (64 << 20) - n * per < (72 << 10) + per  # weight images: 60 KiB
    g.sync()
    out = g.field_forward(gid, rays[:n])
    g.sync()
    for a, b in zip(out, same):
        assert torch.equal(a, b[:n]) and bool(torch.isnan(b[n:]).all())
