"""A box whose full size overflows float32 (half extents above 1.7e38): unit
positions are 0 there, also where a point plus the half extent overflows."""
import numpy as np
import pytest

import paper_2304_05735_amd as pk
from tests.tiny import random_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half", [(3e38, 3e38, 3e38), (0.5, 2e38, 0.5)])
def test_size_beyond_float32(half):
    print("box overflow", half, flush=True)
    g = pk.Context(pk.default_config(n_levels=3, max_res=100, log2_table_size=10))
    i = g.add_object(1, np.zeros(3), 0.0, np.asarray(half, np.float32))
    g.set_params(i, random_params(g.object_info(i).n_grid_params, 6, seed=1).astype(np.float32))
    h = np.asarray(half, np.float32)
    rng = np.random.default_rng(2)
    x = (rng.uniform(-1, 1, (500, 3)) * h.astype(np.float64)).astype(np.float32)
    x[0], x[1] = h, -h
    x[2] = np.inf
    x[3] = np.nan
    with np.errstate(over="ignore", invalid="ignore"):
        p = np.fmin(np.fmax((x + h) / (h + h), np.float32(0)), np.float32(1))  # a NaN gives 0
    huge = ~np.isfinite(h + h)
    assert huge.any() and not p[:, huge].any()
    # the same unit positions in a box of ordinary size
    unit = pk.Context(pk.default_config(n_levels=3, max_res=100, log2_table_size=10))
    j = unit.add_object(1, np.zeros(3), 0.0, np.full(3, 0.5, np.float32))
    unit.set_params(j, g.get_params(i))
    y = np.where(huge, np.float32(-0.5), x).astype(np.float32)
    sig = g.query_density(i, x)
    assert np.isfinite(sig).all()
    assert np.array_equal(sig, unit.query_density(j, y))
