"""Grouped lens application over row lengths: the short-row kernel (fewer than
four entries per row on average) and the eight-lanes-per-entry kernel with each
number of partial sums give, for every map, the bits of passes of at most four
maps (the last group partial, the last block of rows partial)."""
import numpy as np
import pytest

import crp_inputs as I
from oracle import lens as LN
from parity_helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_r,sky_n", [(3000, 5, 23), (6000, 3, 7), (6000, 1, 2), (60000, 1, 4),
                                         (300000, 1, 8), (1000000, 1, 12), (1000000, 1, 20)])
def test_grouped_application_over_row_lengths(n, n_r, sky_n):
    from paper_1307_2643_amd import crp as P
    w = I.W_GALBACK
    ctx = P.Context(P.params_for(w, 0, queue_capacity=1 << 20, neutral_capacity=1 << 10))
    ctx.set_field_analytic(I.GALACTIC_FIELD)
    ctx.set_tables(w.make_tables())
    ctx.inject(w.make_injection(n))
    assert ctx.propagate()
    nnz, _ = ctx.lens_build(LN.spec(10.0 ** np.linspace(16.5, 20.0, n_r + 1), sky_n=sky_n))
    rows = n_r * 6 * sky_n ** 2
    say(f"{rows} rows, {nnz / rows:.1f} entries each")
    x = np.random.default_rng(n + sky_n).uniform(-1.0, 1.0, (21, n_r, 6 * sky_n ** 2))
    y, _ = ctx.lens_apply(x)
    for k in range(0, 21, 4):
        assert np.array_equal(y[k:k + 4], ctx.lens_apply(x[k:k + 4])[0])
    ctx.close()
