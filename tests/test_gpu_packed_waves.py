"""Full waves against the oracle, bit for bit: batches of one and a half times the launch's lanes
(so every lane holds an injected candidate, and takes another when it ends), with open channels
(secondaries among them), every layout, grid type and precision form, and the refill thresholds.
On odd and even grids, steps inside a cell, across a few and across many, so that lanes of one wave
keep and fetch records in the same gather."""
import dataclasses

import numpy as np
import pytest

import crp_inputs as I
from parity_helpers import (compare_counts, compare_neutral, compare_records, make_ctx, run_gpu,
                            say)

pytestmark = pytest.mark.gpu

# one block per compute unit of 256: 32768 lanes with blocks of 128, 65536 of 256
N = 49_177
CELL = I.W_SMALL.spacing_m
SHAPES = {"in-cell": ((4, 4, 4), 0.05), "few": ((5, 7, 6), 0.9), "many": ((8, 16, 4), 3.0)}


@pytest.fixture(scope="module")
def P():
    from paper_1307_2643_amd import crp
    crp.load()
    return crp


def _batch(n, lmax, box):
    rng = np.random.default_rng(41)
    inj = I.inject_mixed(n, 43, lmax_m=lmax, e1=1e19, e2=1e21)
    inj.pos[:] = (rng.random((n, 3)) * 3.0 - 1.0) * box
    inj.lmax[:] = lmax * (0.1 + 0.9 * rng.random(n))
    return inj


def _compare(P, O, shape, precision, dtype, layout, refill, patches=(), block=128, n=None):
    dims, step = SHAPES[shape]
    w = dataclasses.replace(I.W_SMALL, tables="full", hmin_m=0.02 * step * CELL,
                            hmax_m=step * CELL, lmax_m=max(25 * step * CELL, I.MPC_M))
    rng = np.random.default_rng(5)
    grid = (rng.standard_normal(dims + (3,)) * 1e-13).astype(dtype)
    tables = w.make_tables()
    full = n is None
    n = N * block // 128 if full else n
    inj = _batch(n, w.lmax_m, np.array(dims) * CELL)
    say(f"packed {shape} precision {precision} {np.dtype(dtype).name} layout {layout} "
        f"refill {refill} patches {len(patches)}")
    with make_ctx(P, w, grid, tables, precision, qcap=1 << 18, ncap=1 << 18) as ctx:
        if patches:
            ctx.set_field_patches(patches)
        ctx.set_launch(block=block, blocks_per_cu=1, refill=refill, layout=layout)
        done, fin, neu, cnt = run_gpu(ctx, inj)
    assert done and cnt["pending"] == 0
    fo, no, co, _ = O.propagate(O.config_for(w, precision=O.MIX if precision else O.FP64),
                                O.GridRef(grid, w.spacing_m, patches=list(patches)),
                                O.TablesRef(tables), inj, fin_cap=4 * n, neu_cap=4 * n)
    # (a spread batch has a sixty-fourth of the lanes busy)
    assert not full or cnt["attempts"] > 0.2 * cnt["lane_slots"]
    assert co["charged_sec"] > 500 and co["neutral_sec"] > 100
    assert compare_records(fin, fo, shape).all()
    compare_neutral(neu, no, shape, fo)
    compare_counts(cnt, co, shape)


@pytest.mark.parametrize("refill", [1, 16, 64])
@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("precision,dtype", [(0, np.float64), (1, np.float64), (0, np.float32),
                                             (1, np.float32)],
                         ids=["fp64-f64", "mix-f64", "fp64-f32", "mix-f32"])
def test_packed_corner_records(P, oracle_lib, precision, dtype, shape, refill):
    _compare(P, oracle_lib, shape, precision, dtype, P.LAYOUT_CORNER, refill)


@pytest.mark.parametrize("shape,refill", [("in-cell", 16), ("few", 1), ("many", 64)])
@pytest.mark.parametrize("precision,dtype", [(0, np.float64), (1, np.float64), (0, np.float32),
                                             (1, np.float32)],
                         ids=["fp64-f64", "mix-f64", "fp64-f32", "mix-f32"])
def test_packed_linear(P, oracle_lib, precision, dtype, shape, refill):
    _compare(P, oracle_lib, shape, precision, dtype, P.LAYOUT_LINEAR, refill)


@pytest.mark.parametrize("lanes,more", [(40, 0), (40, 1), (64, -1)])
@pytest.mark.parametrize("precision,dtype", [(0, np.float64), (1, np.float64), (0, np.float32),
                                             (1, np.float32)],
                         ids=["fp64-f64", "mix-f64", "fp64-f32", "mix-f32"])
def test_linear_around_the_change_of_stepper(P, oracle_lib, precision, dtype, lanes, more):
    """40 lanes of each of the 512 waves (no values kept), 41 (kept), and all but one."""
    _compare(P, oracle_lib, "few", precision, dtype, P.LAYOUT_LINEAR, 4, n=512 * lanes + more)


@pytest.mark.parametrize("refill", [1, 64])
@pytest.mark.parametrize("precision,dtype,layout", [(0, np.float32, 1), (1, np.float32, 1),
                                                    (0, np.float64, 1), (1, np.float32, 0)],
                         ids=["fp64-f32-corner", "mix-f32-corner", "fp64-f64", "mix-f32-linear"])
def test_packed_patches(P, oracle_lib, precision, dtype, layout, refill):
    rng = np.random.default_rng(6)
    patches = [dict(data=(rng.standard_normal((9, 13, 7, 3)) * 2e-13).astype(dtype),
                    offset=(0, 0, 1), refine=4),
               dict(data=(rng.standard_normal((5, 5, 5, 3)) * 2e-13).astype(dtype),
                    offset=(2, 3, 2), refine=2)]
    _compare(P, oracle_lib, "few", precision, dtype, layout, refill, patches)


@pytest.mark.parametrize("precision,dtype,layout", [(0, np.float64, 1), (1, np.float32, 1),
                                                    (0, np.float64, 0)])
def test_packed_blocks_of_256(P, oracle_lib, precision, dtype, layout):
    _compare(P, oracle_lib, "few", precision, dtype, layout, 16, block=256)


@pytest.mark.parametrize("nodes", [2, 268, 269, 541, 653, 1024])
@pytest.mark.parametrize("dtype,layout,block", [(np.float64, 0, 128), (np.float64, 1, 256),
                                                (np.float32, 1, 256), (np.float32, 0, 128)])
def test_table_sizes(P, oracle_lib, dtype, layout, block, nodes):
    """Tables of 2 to 1024 nodes, which share a compute unit's LDS with the blocks' own areas:
    fewer blocks fit beyond 268 (FP64 grid, block 128), 540 (FP64, 256) and 652 nodes (FP32
    linear, 128)."""
    O = oracle_lib
    w = dataclasses.replace(I.W_SMALL, lmax_m=3 * I.MPC_M)
    e = I.table_nodes(nodes)
    full = I.tables_full()
    tables = I.Tables(e, *(np.interp(e, full.e_nodes, v) for v in
                           (full.t_pi, full.t_n, full.beta_p)))
    grid = w.make_grid().astype(dtype)
    inj = I.inject_mixed(700, 47, lmax_m=w.lmax_m, e1=1e19, e2=1e21)
    say(f"tables of {nodes} nodes, {np.dtype(dtype).name}, layout {layout}, block {block}")
    with make_ctx(P, w, grid, tables, 0) as ctx:
        ctx.set_launch(block=block, layout=layout)
        done, fin, neu, cnt = run_gpu(ctx, inj)
    assert done
    fo, no, co, _ = O.propagate(O.config_for(w), O.GridRef(grid, w.spacing_m),
                                O.TablesRef(tables), inj)
    assert compare_records(fin, fo, f"{nodes} nodes").all()
    compare_neutral(neu, no, f"{nodes} nodes", fo)
    compare_counts(cnt, co, f"{nodes} nodes")
