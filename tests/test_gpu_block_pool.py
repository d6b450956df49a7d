"""Device blocks that a context keeps for its next buffers: what an earlier buffer left in a block is
never read, the budget counts live buffers only, and kept blocks make room when it needs them."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


def _poison(bq, ctx, dims, nrhs):
    """Free fields full of NaN whose blocks have the sizes of the library's work fields (an FP32 field
    of 2n columns has the bytes of an FP64 field of n, and other places for its padding)."""
    bad = np.full((2 * nrhs, int(np.prod(dims)), 4, 3), np.nan + 1j * np.nan)
    made = [bq.Field(ctx, dims, bq.BQ_ODD, p, n)
            for p, n in [(bq.BQ_F32, 2 * nrhs)] * 14 + [(bq.BQ_F64, nrhs)] * 4 + [(bq.BQ_F16, nrhs)] * 3]
    for f in made:
        f.put(bad[:f.nrhs])
    for f in made:
        f.close()


@pytest.mark.parametrize("dims", [(4, 4, 6, 10), (4, 4, 4, 8)])  # a last tile that is half full, and whole tiles
def test_left_contents_are_not_read(bq, dims):
    n = 2
    U = inputs.gauge_field(dims, 0.2, seed=91)
    b = inputs.gaussian_spinor(dims, n, seed=92)
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, dims, U, -1)
    op = bq.Op(G, 0.12, 1.5, 0.0)
    fields = {(s, p): bq.Field(ctx, dims, s, p, n) for s in (bq.BQ_ODD, bq.BQ_FULL) for p in (0, 1, 2)}
    to = {k: bq.Field(ctx, dims, k[0], k[1], n) for k in fields}
    xs = [bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, n) for _ in range(2)]
    for f in fields.values():
        f.put(b)

    def everything():
        out = []
        for p in (0, 1, 2):
            for kind, sub in ((bq.BQ_OP_MHAT, bq.BQ_ODD), (bq.BQ_OP_MHATDAG_MHAT, bq.BQ_ODD), (bq.BQ_OP_MDAGM, bq.BQ_FULL)):
                op.apply(kind, fields[sub, p], to[sub, p])
                out.append(to[sub, p].get())
        op.solve_multishift(fields[bq.BQ_ODD, 0], xs, [0.0, 0.3], 1e-9)
        out += [x.get() for x in xs]
        for kw in (dict(solver=bq.BQ_SOLVER_BICGSTAB, inner_prec=bq.BQ_F64),
                   dict(solver=bq.BQ_SOLVER_BICGSTAB, inner_prec=bq.BQ_F32), dict(solver=bq.BQ_SOLVER_BLOCK_CG),
                   dict(inner_prec=bq.BQ_F32)):
            op.solve(fields[bq.BQ_FULL, 0], to[bq.BQ_FULL, 0], 1e-9, system=bq.BQ_SYS_M, **kw)
            out.append(to[bq.BQ_FULL, 0].get())
        return out

    first = everything()
    assert all(np.isfinite(o).all() for o in first)
    _poison(bq, ctx, dims, n)
    for a, c in zip(first, everything()):
        assert np.array_equal(a, c)
    # a new configuration in blocks that held others
    G2 = bq.Gauge(ctx, dims, U, -1)
    op2 = bq.Op(G2, 0.12, 1.5, 0.0)
    op2.apply(bq.BQ_OP_M, fields[bq.BQ_FULL, 0], to[bq.BQ_FULL, 0])
    got = to[bq.BQ_FULL, 0].get()
    op.apply(bq.BQ_OP_M, fields[bq.BQ_FULL, 0], to[bq.BQ_FULL, 0])
    assert np.array_equal(got, to[bq.BQ_FULL, 0].get())
    # a new field is zero whatever its block held
    assert not bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F32, 2 * n).get().any()


def test_kept_blocks_make_room(bq):
    """A budget that live fields of one size fill is there again for fields of another size."""
    dims = (8, 8, 8, 16)
    probe = bq.Context(0)
    f = bq.Field(probe, dims, bq.BQ_FULL, bq.BQ_F64, 3)
    size = probe.hbm_used()
    ctx = bq.Context(0, hbm_budget=4 * size)
    for n in (3, 2, 1, 3):
        live = []
        with pytest.raises(bq.BqError) as e:
            while len(live) < 64:
                live.append(bq.Field(ctx, dims, bq.BQ_FULL, bq.BQ_F64, n))
        assert e.value.code == bq.BQ_ERR_OOM and live
        used = ctx.hbm_used()
        assert used <= 4 * size < used + used // len(live)
        for g in live:
            g.close()
        assert ctx.hbm_used() == 0
    f.close()
