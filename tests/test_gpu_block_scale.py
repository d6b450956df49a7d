"""Block CG on sources so small that the products of its Gram matrices lie below the smallest normal number."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5])
def test_subnormal_gram_matrices(n):
    from paper_1711_03836_amd import bqhip as bq
    dims, tol, scale = (6, 4, 4, 6), 1e-4, 1e-157  # |b|^2 about 1e-310, at the end tol^2 of it
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, inputs.gauge_field(dims, 0.2, seed=87), -1), 0.12, 1.5, 0.0)
    src = inputs.gaussian_spinor(dims, n, seed=88)
    b, x = (bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, n) for _ in range(2))
    got = []
    for f in (1.0, scale):
        b.put(f * src)
        rc, info = op.solve(b, x, tol, system=bq.BQ_SYS_NORMAL, solver=bq.BQ_SOLVER_BLOCK_CG, raise_on_error=False)
        assert rc == bq.BQ_OK and all(i["converged"] for i in info)
        got.append(x.get() / f)
    # both stop at |r| <= tol |b| of Mhat^dag Mhat, whose condition number here is below 100
    for a, c in zip(*got):
        assert np.linalg.norm(a - c) <= 200 * tol * np.linalg.norm(a)
