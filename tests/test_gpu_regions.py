"""Region sizes of the gradient accumulation (2^9, 2^10 or 2^11 table entries,
by how many regions a launch has) against the oracle: with each size the
finest resolution whose x-pairs stay in a region and the next, a dense level
whose last region is partial, tables smaller than a region, bins so small that
records overflow, and several objects of different tables in one launch.  FP32
bars of the gradient parity tests."""
import numpy as np
import pytest

import oracle
import paper_2304_05735_amd as pk
from tests.gpu_common import assert_fwd_close, assert_grad_close, make_pair, oracle_grad, tensor_cuts
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nmin,nmax,log2T,N,cap", [
    (16, 511, 14, 32, 0), (511, 512, 13, 64, 0), (16, 512, 8, 32, 8),    # 2^9
    (16, 1023, 17, 64, 0), (1023, 1024, 17, 32, 0), (65, 1024, 17, 32, 8),  # 2^10
    (2047, 2048, 18, 64, 0), (16, 2047, 19, 128, 0)])                     # 2^11
def test_region_sizes(nmin, nmax, log2T, N, cap):
    print(f"regions {nmin}..{nmax} 2^{log2T} N {N} cap {cap}", flush=True)
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
