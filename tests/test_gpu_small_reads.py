"""Reading records through the context's pinned memory (few records) and by
separate copies (many): the same records either way, also with columns left
out; and injection from the host through both."""
import ctypes as C

import numpy as np
import pytest

import crp_inputs as I

pytestmark = pytest.mark.gpu

N = 40000          # 128 bytes each: 5 MB, past the limit of small transfers


def run(P, pieces):
    w = I.W_SMALL
    ctx = P.Context(P.params_for(w, 0, queue_capacity=1 << 18, neutral_capacity=1 << 18))
    ctx.set_field_grid(w.make_grid(), w.spacing_m)
    ctx.set_tables(I.W_MIXED256.make_tables())
    inj = I.W_MIXED256.make_injection(N)
    inj.lmax[:] = 10 * I.MPC_M
    edges = np.linspace(0, N, pieces + 1).astype(int)
    for a, b in zip(edges[:-1], edges[1:]):
        ctx.inject(**{k: getattr(inj, k)[a:b] for k in ("id", "A", "Z", "E", "pos", "dir", "lmax")})
    assert ctx.propagate()
    return ctx


def key_order(r):
    return np.lexsort((r.get("m", r["id"] * 0), r["lineage"], r["id"]))


def parts(read, left, step):
    got = []
    while left() > 0:
        got.append(read(step))
    return {k: np.concatenate([g[k] for g in got]) for k in got[0]}


@pytest.mark.parametrize("step", [1, 777, 16000])
def test_reads_in_parts_give_the_same_records(step):
    from paper_1307_2643_amd import crp as P
    print(f"reads of {step} records", flush=True)
    one, many = run(P, 1), run(P, 40)
    fin, neu = one.read_finished(), one.read_neutral()
    if step == 1:      # leave all but 50 to reads past the limit
        first = many.read_finished(many.counts()["finished_unread"] - 50)
        rest = parts(many.read_finished, lambda: many.counts()["finished_unread"], 1)
        f2 = {k: np.concatenate([first[k], rest[k]]) for k in fin}
    else:
        f2 = parts(many.read_finished, lambda: many.counts()["finished_unread"], step)
    n2 = parts(many.read_neutral, lambda: many.counts()["neutral_unread"], max(step, 777))
    for a, b in ((fin, f2), (neu, n2)):
        oa, ob = key_order(a), key_order(b)
        assert len(oa) == len(ob)
        for k in a:
            assert np.array_equal(a[k][oa], b[k][ob]), k
    one.close()
    many.close()


def test_columns_left_out():
    from paper_1307_2643_amd import crp as P
    ctx = run(P, 1)
    ref = run(P, 1)
    rows = 100
    out = P.FinishedSoA()
    E, x, ident = np.zeros(rows), np.zeros((rows, 3)), np.zeros(rows, np.uint32)
    lin = np.zeros(rows, np.uint32)
    for name, arr in (("E", E), ("x", x), ("id", ident), ("lineage", lin)):
        setattr(out, name, C.cast(arr.ctypes.data, type(getattr(out, name))))
    n = C.c_int64(0)
    st = ctx.L.crp_read_finished(ctx.h, rows, C.byref(out), C.byref(n))
    assert st == P.EOVERFLOW and n.value == rows
    full = ref.read_finished()
    where = {(i, l): k for k, (i, l) in enumerate(zip(full["id"], full["lineage"]))}
    for k in range(rows):
        j = where[(ident[k], lin[k])]
        assert E[k] == full["E"][j] and np.array_equal(x[k], full["x"][j])
    ctx.close()
    ref.close()
