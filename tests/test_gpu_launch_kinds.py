"""Launches of several objects: each object's losses, gradients and weights are
those of calls on it alone, bit for bit, whichever call's work tables were in
place before (one object, all in one launch, two concurrent halves, one launch
per object, other ray counts and orders, capped bins); and objects of different
table sizes in one launch, whose regions have one size, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2304_05735_amd as pk
from tests.gpu_common import assert_fwd_close, assert_grad_close, oracle_grad, tensor_cuts
from tests.tiny import random_params, tiny_scene

pytestmark = pytest.mark.gpu


def _objects(log2Ts, layers=1, with_oracle=False, **kw):
    frames, box = tiny_scene()
    cfg = pk.default_config(**{"autotune": 0, "rays_per_step": 64, **kw})
    g = pk.Context(cfg)
    o = None
    if with_oracle:
        o = oracle.OracleContext(oracle.make_config(
            L=cfg.n_levels, nmin=cfg.base_res, nmax=cfg.max_res, log2T=cfg.log2_table_size,
            N=cfg.samples_per_ray, lambda_depth=float(cfg.lambda_depth),
            lambda_density=float(cfg.lambda_density)))
    for j, lt in enumerate(log2Ts):
        i = g.add_object(j + 1, box["t"], box["yaw"], box["half"], lt)
        p = random_params(g.object_info(i).n_grid_params, 2 * cfg.n_levels, seed=j).astype(np.float32)
        g.set_params(i, p)
        if o:
            assert o.add_object(j + 1, box["t"], box["yaw"], box["half"], lt) == i
            o.objects[i].params[:] = p.astype(np.float64)
    for j in range(len(log2Ts)):  # each object has the views to itself (99: an unregistered occluder)
        for cam, rgb, mask, depth in frames:
            m = np.where(mask == 1, j + 1, np.where(mask == 2, 99, 0)).astype(np.int32)
            g.add_keyframe(cam, rgb, m, depth)
            if o:
                o.add_keyframe(cam, rgb, m, depth)
    return (g, o) if with_oracle else g


@pytest.mark.parametrize("mode,graph", [(pk.BATCH_ALL, 0), (pk.BATCH_ALL, 2), (pk.BATCH_PER_OBJECT, 0)])
def test_kinds_in_turn(mode, graph):
    print(f"kinds in turn, mode {mode} graph {graph}", flush=True)
    kw = dict(n_levels=4, max_res=200, samples_per_ray=32, use_graph=graph)
    both = _objects([12, 10], batch_mode=mode, **kw)
    alone = [_objects([12, 10], batch_mode=mode, **kw) for _ in range(2)]
    train = [((0, 1), (64, 64), 2), ((0,), (64,), 1), ((0, 1), (64, 64), 2), "loss", ((0, 1), (64, 64), 1),
             ((1,), (40,), 3), "loss", "capped", ((1, 0), (64, 64), 1), ((0, 1), (30, 90), 4),
             ((0, 1), (64, 64), 5), "loss", ((1,), (64,), 1), "capped", ((0, 1), (64, 64), 1)]
    for k, what in enumerate(train):
        if what == "loss":
            l = both.loss_and_grad([0, 1])
            for i in (0, 1):
                assert l[i] == alone[i].loss_and_grad([i])[0], k
                assert np.array_equal(both.get_params(i, pk.GRAD), alone[i].get_params(i, pk.GRAD)), k
        elif what == "capped":  # most records overflow: the sums in another order
            l = both.loss_and_grad([0])
            full = both.get_params(0, pk.GRAD)
            both.debug_bin_capacity(4)
            assert both.loss_and_grad([0]) == l, k
            capped = both.get_params(0, pk.GRAD)
            assert not np.array_equal(capped, full), k
            assert np.abs(capped - full).max() <= 1e-4 * np.abs(full).max(), k
            both.debug_bin_capacity(0)
            assert both.loss_and_grad([0]) == l, k
            assert np.array_equal(both.get_params(0, pk.GRAD), full), k
        else:
            ids, rays, steps = what
            both.train(steps, ids, rays)
            for i, n in zip(ids, rays):
                alone[i].train(steps, [i], [n])
            for i in ids:
                assert np.array_equal(both.get_params(i), alone[i].get_params(i)), (k, i)


@pytest.mark.parametrize("log2Ts,nmax,cap", [
    ((8, 12, 19), 2047, 0), ((19, 8), 2048, 8),        # regions of 2^11 entries
    ((10, 14, 17), 1023, 0), ((17, 9), 1024, 8),       # 2^10
    ((9, 11, 13), 511, 0), ((13, 9, 11), 512, 8)])     # 2^9
def test_tables_of_several_sizes(log2Ts, nmax, cap):
    print(f"tables {log2Ts} to {nmax} cells, cap {cap}", flush=True)
    B = 120
    g, o = _objects(log2Ts, with_oracle=True, n_levels=3, base_res=16, max_res=nmax, samples_per_ray=64,
                    rays_per_step=B)
    ids = list(range(len(log2Ts)))
    g.debug_bin_capacity(cap)
    losses = g.loss_and_grad(ids)
    for i in ids:
        ol, og, mass, allow, _ = oracle_grad(o, i, 0, B)
        assert_fwd_close([losses[i]], [ol], rtol=1e-5, what="loss")
        assert_grad_close(g.get_params(i, pk.GRAD), og, mass, allow, what=f"gradient 2^{log2Ts[i]}",
                          cuts=tensor_cuts(o, i))
