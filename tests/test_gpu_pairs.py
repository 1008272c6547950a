"""Gradient records of the fine hashed levels (x-pairs of corners) against the
oracle, where the rule that chooses them changes: tables smaller than,
as large as and larger than a region of 2^11 entries, resolutions around the
finest one whose pairs stay in a region (2047 | 2048), a cell row whose
indices carry through every low bit, and bins so small that most records
overflow to the gradient's atomics.  FP32 bars of the gradient parity tests."""
import numpy as np
import pytest

import oracle
import paper_2304_05735_amd as pk
from tests.gpu_common import assert_fwd_close, assert_grad_close, make_pair, oracle_grad, tensor_cuts
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nmin,nmax,log2T,N,cap", [
    (33, 2047, 8, 32, 0), (2047, 2048, 11, 32, 0), (2047, 2048, 14, 64, 0), (65, 1023, 12, 64, 0),
    (129, 1024, 13, 128, 0), (128, 512, 9, 32, 0), (40, 2047, 13, 32, 4), (40, 65536, 12, 64, 16)])
def test_pair_records(nmin, nmax, log2T, N, cap):
    print(f"pair records {nmin}..{nmax} 2^{log2T} N {N} cap {cap}", flush=True)
    frames, box = tiny_scene()
    L, B = 3, 150
    g, o, gid = make_pair(L, nmin, nmax, log2T, N, B, frames, box)
    ob = o.objects[gid]
    p = random_params(oracle.grid_params(ob.lv), 2 * L, seed=log2T).astype(np.float32)
    g.set_params(gid, p)
    ob.params[:] = p.astype(np.float64)
    g.debug_bin_capacity(cap)
    gl = g.loss_and_grad([gid])[0]
    gg = g.get_params(gid, pk.GRAD)
    ol, og, mass, allow, _ = oracle_grad(o, gid, 0, B)
    assert_fwd_close([gl], [ol], rtol=1e-5, what="loss")
    assert_grad_close(gg, og, mass, allow, what="gradient", cuts=tensor_cuts(o, gid))
