"""Batches around the sizes where candidates are spread over waves instead of packed 64 to a wave
(one lane per wave, several, the change to full waves), with and without open interaction
channels (secondaries take idle lanes; without channels the launch shrinks to the batch)."""
import dataclasses

import numpy as np
import pytest

import crp_inputs as I
from parity_helpers import compare_records, make_ctx, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tables", ["full", "loss"])
@pytest.mark.parametrize("n,bpc", [(1, 0), (65, 0), (1023, 0), (1025, 0), (2600, 1), (40000, 1)])
def test_small_batches_match_oracle(oracle_lib, n, bpc, tables):
    from paper_1307_2643_amd import crp as P
    O = oracle_lib
    w = dataclasses.replace(I.W_SMALL, tables=tables, lmax_m=3 * I.MPC_M)
    grid, tabs = w.make_grid(), w.make_tables()
    inj = I.inject_mixed(n, 29, lmax_m=w.lmax_m, e1=1e19)
    fo, no, co, _ = O.propagate(O.config_for(w), O.GridRef(grid, w.spacing_m), O.TablesRef(tabs),
                                inj)
    with make_ctx(P, w, grid, tabs, P.FP64, qcap=1 << 17, ncap=1 << 17) as ctx:
        ctx.set_launch(block=128, blocks_per_cu=bpc, refill=16)
        for part in range(2):      # the second batch runs on the lanes of the first
            done, fin, neu, cnt = run_gpu(ctx, inj)
            assert done and cnt["pending"] == 0
            # the same operations in the same order on both sides: bit for bit
            assert compare_records(fin, fo, f"n {n} {tables} run {part}").all()
            assert len(neu["id"]) == len(no["id"])
            for k in ("steps", "attempts", "rejects", "finished", "events", "charged_sec"):
                assert cnt[k] == (part + 1) * co[k], k
    if tables == "full" and n > 1000:
        assert co["charged_sec"] > 0
    if tables == "loss":
        assert co["events"] == 0 and np.all(fo["lineage"] == 0)
