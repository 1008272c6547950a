"""The BF16 MLP's backward over rays with skipped blocks of 16 samples (with one
hidden layer it takes blocks in pairs, one of which may be dead) against the
oracle's BF16 mode, scratch of an earlier call filled with NaN first."""
import numpy as np
import pytest

import oracle
import paper_2304_05735_amd as pk
from tests.gpu_common import assert_bf16_close, bf16_reference, make_pair
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,layers", [(32, 1), (64, 1), (128, 1), (64, 2)])
def test_dead_blocks_bf16(N, layers):
    print(f"dead blocks BF16 N {N} layers {layers}", flush=True)
    frames, box = tiny_scene()
    L, B = 6, 131
    g, o, gid = make_pair(L, 16, 200, 12, N, B, frames, box, precision=pk.PREC_BF16, mlp_layers=layers,
                          bf16_oracle=True)
    ob = o.objects[gid]
    p = random_params(oracle.grid_params(ob.lv), 2 * L, seed=N, layers=layers).astype(np.float32)
    g.set_params(gid, np.full_like(p, np.nan))
    g.loss_and_grad([gid])
    g.set_params(gid, p)
    ob.params[:] = p.astype(np.float64)
    c = np.arange(64)
    s = (c[:, None, None] + c[:, None] + c).reshape(-1)
    bits = np.packbits((s >= 80) & (s < 110), bitorder="little")  # a slab: long dead runs around a live one
    g.set_occupancy(gid, bits)
    o.set_occupancy(gid, bits)
    gl = g.loss_and_grad([gid])[0]
    assert_bf16_close(gl, g.get_params(gid, pk.GRAD), bf16_reference(o, gid, 0, B), what=f"N {N}")
