"""Precision of the x-pair gradient records, entry by entry, on one hashed
level whose corners are all written as pairs.  Only entries that a single
corner of a single sample touches are compared, so that each holds one term:
s A or (1 - s) A of a pair, whose ratio the sample's position gives exactly."""
import numpy as np
import pytest
import torch

import paper_2304_05735_amd as pk
from tests.tiny import random_params

pytestmark = pytest.mark.gpu

N, T, NS = 300, 1 << 14, 32
HALF = np.array([0.4, 0.3, 0.35], np.float32)


def _setup(n, seed):
    g = pk.Context(pk.default_config(n_levels=1, base_res=N, max_res=N, log2_table_size=14,
                                     samples_per_ray=NS, autotune=0), stream=torch.cuda.Stream())
    i = g.add_object(1, np.zeros(3), 0.2, HALF)
    g.set_params(i, random_params(g.object_info(i).n_grid_params, 2, seed=seed).astype(np.float32))
    rng = np.random.default_rng(seed)
    # within the first cell in x, where the position in the cell has all of
    # float32's bits, from a point of one face in y to one of the other
    o, e = rng.uniform(-0.95, 0.95, (n, 3)) * HALF, rng.uniform(-0.95, 0.95, (n, 3)) * HALF
    o[:, 1], e[:, 1] = -HALF[1], HALF[1]
    for q in (o, e):
        q[:, 0] = (rng.uniform(0.02, 0.98, n) * 2 / N - 1) * HALF[0]
    length = np.linalg.norm(e - o, axis=1, keepdims=True)
    rays = np.concatenate([o, (e - o) / length, 0 * length, length], 1).astype(np.float32)
    return g, i, rays, rng.normal(size=(n, 3)).astype(np.float32)


def _pairs(rays):
    """(entry of the smaller weight, of the larger, s) of the 4 x-pairs of every
    sample, positions in float32 as the library takes them, and of each pair
    whether nothing else touches its two entries."""
    f4 = np.float32
    o, d, tn, tf = rays[:, None, :3], rays[:, None, 3:6], rays[:, 6], rays[:, 7]
    delta = (tf - tn) / f4(NS)
    di = tn[:, None] + (np.arange(NS, dtype=f4) + f4(0.5)) * delta[:, None]
    x = (o + di[..., None] * d).reshape(-1, 3)
    p = np.clip((x + HALF) / (HALF + HALF), f4(0), f4(1))
    gr = p * f4(N)
    c = np.clip(np.floor(gr), 0, N - 1)
    f = (gr - c)[:, 0].astype(np.float64)
    c = c.astype(np.uint32)
    up = f > 0.5
    small, large = [], []
    for q in range(4):
        h = ((c[:, 1] + np.uint32(q & 1)) * np.uint32(2654435761)) ^ ((c[:, 2] + np.uint32(q >> 1)) * np.uint32(805459861))
        near, far = (c[:, 0] ^ h) & (T - 1), ((c[:, 0] + np.uint32(1)) ^ h) & (T - 1)
        small.append(np.where(up, near, far))
        large.append(np.where(up, far, near))
    small, large = np.stack(small, 1), np.stack(large, 1)
    hits = np.bincount(np.concatenate([small, large]).reshape(-1), minlength=T)
    alone = (hits[small] == 1) & (hits[large] == 1)
    return small, large, np.where(up, 1 - f, f)[:, None].repeat(4, 1), alone


def _grad(g, i, rays, adj):
    r, a = torch.from_numpy(rays).cuda(), torch.from_numpy(adj).cuda()
    torch.cuda.synchronize()
    out = g.field_backward(i, r, a, None, None)
    g.sync()
    return out[:2 * T].cpu().numpy().astype(np.float64).reshape(T, 2)


def test_overflow_takes_the_whole_split():
    """Records beyond a bin's capacity are added as float32 products of the
    unrounded split: s A / (1 - s) A is off by at most the roundings of 1 - s
    and of the two products, 3 x 2^-24.  The 32 bins hold 4 records each, so at
    most 128 pairs may show the records' own rounding (2^-19 + 2^-21 for each)."""
    print("overflow split", flush=True)
    g, i, rays, adj = _setup(60, 7)
    small, large, s, alone = _pairs(rays)
    g.debug_bin_capacity(4)
    grad = _grad(g, i, rays, adj)
    ok = alone & (s > 1e-4)
    a, b, r = grad[small[ok]], grad[large[ok]], (s / (1 - s))[ok][:, None]
    some = (a != 0).all(1) & (b != 0).all(1)
    err = np.abs(a[some] / b[some] / r[some] - 1).max(1)
    off = int((err > 3.01 * 2.0 ** -24).sum())
    print(f"  {err.size} pairs, {off} beyond the product's rounding, largest {err.max():.2e}")
    assert err.size > 500
    assert err.max() < 2.01 * (2.0 ** -19 + 2.0 ** -21)
    assert off <= 128


def test_sums_hold_38_bits_below_the_largest_term():
    """A region's fixed-point sums keep each term to half a unit of 2^-38 of the
    power of two at or below the entry's largest term.  Three equal rays with
    adjoints 1, -1 and 2^-34 leave 2^-34 of a single ray's value: the large
    terms round alike and cancel, so the small one's rounding is all that is
    off (the records and products scale exactly with a power of two)."""
    print("fixed-point bits", flush=True)
    g, i, rays, adj = _setup(60, 11)
    small, large, _, alone = _pairs(rays)
    one = _grad(g, i, rays, adj)
    k = 2.0 ** -34
    three = _grad(g, i, rays.repeat(3, 0),
                  np.stack([adj, -adj, adj * np.float32(k)], 1).reshape(-1, 3))
    e = np.concatenate([small[alone], large[alone]])
    e = e[(one[e] != 0).all(1)]
    unit = 2.0 ** (np.floor(np.log2(np.abs(one[e]).max(1))) - 38)
    err = np.abs(three[e] - k * one[e]).max(1) / unit
    print(f"  {e.size} entries, off by up to {err.max():.3f} units, {int((err > 0.5).sum())} by more than half")
    assert e.size > 1000
    assert err.max() <= 0.5
