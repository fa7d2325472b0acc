"""Field evaluation of many points (corner values moved by whole waves) against the evaluation
of few (each lane its own), bit for bit, and against the oracle's field at a sample: ragged
counts, odd grids, positions on vertices, at the wrap of each axis and many periods out."""
import numpy as np
import pytest

import crp_inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("shape,n", [((16, 16, 16), 65536), ((5, 7, 6), 70001), ((2, 3, 2), 65599),
                                     ((40, 6, 33), 131072 + 63)])
def test_many_points_equal_few(oracle_lib, shape, n, dtype, mode):
    from paper_1307_2643_amd import crp as P
    O = oracle_lib
    rng = np.random.default_rng(n)
    grid = (rng.standard_normal(shape + (3,)) * 1e-13).astype(dtype)
    cell, origin = 100 * I.KPC_M, (3e20, -7e21, 1e22)
    pos = (rng.random((n, 3)) * 7 - 3) * np.array(shape)          # several periods, in cells
    k = n // 4
    pos[:k] = np.floor(pos[:k])                                   # on vertices
    pos[k:2 * k, 2] = shape[2] - rng.random(k)                    # the cell that wraps in z
    pos[2 * k:2 * k + 50] += 3e9                                  # beyond 2^31 cells
    pos = np.asarray(origin) + pos * cell
    with P.Context(P.Params(precision=P.MIX)) as ctx:
        ctx.set_field_grid(grid, cell, origin)
        many = ctx.eval_field(pos, mode)
        few = np.concatenate([ctx.eval_field(pos[i:i + 5000], mode) for i in range(0, n, 5000)])
        again = ctx.eval_field_noalloc(pos[::-1].copy(), mode)[::-1]
    assert np.array_equal(many, few) and np.array_equal(many, again)
    pick = np.concatenate([rng.choice(n, 500, replace=False), np.arange(2 * k, 2 * k + 50)])
    ref = O.eval_field(O.GridRef(grid, cell, origin), pos[pick], O.MIX if mode else O.FP64)
    assert np.array_equal(many[pick], ref)
