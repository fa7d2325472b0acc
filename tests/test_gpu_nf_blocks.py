"""Blocks of the training kernels: four waves of one tile each while these
cover all tiles at once (32768 points with 256 CUs), eight above that, and a
second tile per wave above 65536 points; against the numpy oracle with the bars
of the other gradient tests (1e-3 relative L2 per tensor)."""
import numpy as np
import pytest

import crp_inputs as I

pytestmark = pytest.mark.gpu


def rel_l2(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-30))


@pytest.mark.parametrize("n", [1, 32768, 32769, 65600])
def test_gradient_over_block_shapes(n):
    from oracle import nf_oracle as N
    from paper_1307_2643_amd import crp as P
    w = I.W_SMALL
    prm = P.Params(precision=P.MIX, queue_capacity=1 << 12, neutral_capacity=1 << 12)
    ctx = P.Context(prm)
    ctx.set_field_grid(w.make_grid().astype(np.float32), w.spacing_m)
    ctx.set_tables(I.tables_loss_only())
    F = I.nf_frequencies()
    rng = np.random.default_rng(n)
    ws, bs = I.nf_init_weights(811)
    bs = [rng.standard_normal(b.shape).astype(np.float32) * 0.05 for b in bs]
    params = N.flatten(ws, bs).astype(np.float32)
    ctx.nf_init(F, params, I.NG_T)
    pos = rng.random((n, 3)) * 32 * w.spacing_m
    target = rng.standard_normal((n, 3)).astype(np.float32)
    print(f"gradient of {n} points", flush=True)
    out, grad, loss = ctx.nf_loss_grad(pos, target)
    xh = N.normalized_position(pos, (32, 32, 32), w.spacing_m).astype(np.float32)
    ws, bs = N.unflatten(params)
    ref_out, cache = N.forward(ws, bs, xh.astype(np.float64), F, bf16=True)
    gW, gb = N.backward(ws, cache, N.mse_grad(ref_out, target))
    # one point alone averages nothing: one feature or activation that takes
    # the neighbouring bf16 value moves a whole tensor by up to 2^-8
    bar = 1e-3 if n > 1 else 2.0 ** -8
    assert rel_l2(out, ref_out) < bar
    assert abs(loss / N.mse_loss(ref_out, target) - 1) < 2 * bar
    off = 0
    for W, b in zip(gW, gb):
        assert rel_l2(grad[off:off + W.size], W.ravel()) < bar
        off += W.size
        assert rel_l2(grad[off:off + b.size], b) < bar
        off += b.size
    ctx.close()
