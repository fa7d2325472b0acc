"""Reuse of a lane's corner record between the stages of an attempt, the position it moves to and
the next candidate: runs whose steps stay inside one cell, cross a few, or jump many per stage,
on small and odd grids, against the oracle."""
import dataclasses

import numpy as np
import pytest

import crp_inputs as I
from parity_helpers import compare_records, make_ctx, run_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    from paper_1307_2643_amd import crp
    return crp


def _grid(shape, dtype, seed=5):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal(shape + (3,)) * 1e-13).astype(dtype)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape,step_cells", [((4, 4, 4), 0.05), ((5, 7, 6), 0.05),
                                              ((5, 7, 6), 0.9), ((8, 16, 4), 3.0),
                                              ((3, 2, 9), 40.0)])
def test_record_reuse_matches_oracle(P, oracle_lib, shape, step_cells, precision, dtype, layout):
    O = oracle_lib
    cell = I.W_SMALL.spacing_m
    w = dataclasses.replace(I.W_SMALL, tables="full", hmin_m=0.02 * step_cells * cell,
                            hmax_m=step_cells * cell, lmax_m=60 * step_cells * cell)
    grid, tables = _grid(shape, dtype), w.make_tables()
    inj = I.inject_mixed(150, 17, lmax_m=w.lmax_m)
    inj.lmax[:] = w.lmax_m * (0.1 + 0.9 * np.arange(150) / 150)
    cfg = O.config_for(w, O.MIX if precision else O.FP64)
    fo, no, co, _ = O.propagate(cfg, O.GridRef(grid, w.spacing_m), O.TablesRef(tables), inj)
    with make_ctx(P, w, grid, tables, P.MIX if precision else P.FP64) as ctx:
        ctx.set_launch(block=128, blocks_per_cu=1, refill=1,
                       layout=P.LAYOUT_CORNER if layout else P.LAYOUT_LINEAR)
        _, fin, neu, cnt = run_gpu(ctx, inj)
    # the same operations in the same order on both sides: bit for bit
    assert compare_records(fin, fo, f"{shape} step {step_cells} layout {layout}").all()
    for k in ("steps", "attempts", "rejects", "finished", "events"):
        assert cnt[k] == co[k], k
