"""A column of a mixed CG solve whose step breaks down (p^dag A p not finite in the inner precision): it fails
by itself, in the same way in every kernel, and its neighbours do not notice."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [0, 2])
def test_overflow_in_one_column(bad):
    from paper_1711_03836_amd import bqhip as bq
    dims, n = (6, 4, 4, 6), 3  # 5 tiles, the last one half full
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, inputs.gauge_field(dims, 0.2, seed=81), -1), 0.12, 1.5, 0.1)
    src = inputs.gaussian_spinor(dims, n, seed=82)
    src[bad] = 2e38 * (1 + 1j)  # finite in FP32; the half spinors of its hops are not
    b, x = (bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, n) for _ in range(2))
    got = []
    # hop split (picked by size), plain and tile-shared with alpha taken by the stencil; plain with a
    # launch of its own for it (the marching kernel is asked for and the lattice has no whole planes)
    for tune in (None, (18, 1, 64), (18, 2, 64), (18, 1, 768, 0, 1), (18, 1, 64, 2)):
        if tune:
            ctx.tune_set(bq.BQ_F32, n, *tune)
        b.put(src)
        rc, info = op.solve(b, x, 1e-9, system=bq.BQ_SYS_NORMAL, inner_prec=bq.BQ_F32, raise_on_error=False)
        assert rc != bq.BQ_OK
        assert [bool(i["converged"]) for i in info] == [c != bad for c in range(n)]
        got.append((x.get(), [i["iters"] for i in info]))
    assert got[0][1][bad] == 0 and not got[0][0][bad].any()
    for a in got[1:]:
        assert a[1] == got[0][1] and np.array_equal(a[0], got[0][0])
    # the neighbours alone
    keep = [c for c in range(n) if c != bad]
    b2, x2 = (bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, n - 1) for _ in range(2))
    b2.put(src[keep])
    _, info2 = op.solve(b2, x2, 1e-9, system=bq.BQ_SYS_NORMAL, inner_prec=bq.BQ_F32)
    assert [i["iters"] for i in info2] == [got[0][1][c] for c in keep]
    assert np.array_equal(x2.get(), got[0][0][keep])
