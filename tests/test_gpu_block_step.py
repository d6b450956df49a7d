"""Block CG over the sizes of its N x N algebra and of its Gram products: one column, part-filled and full
16 x 16 products, one tile and many, against CG column by column and the FP64 residual."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


@pytest.mark.parametrize("dims,ncols", [((2, 4, 4, 4), (1, 4)), ((6, 4, 4, 6), (1, 3, 5, 12)), ((8, 8, 8, 16), (13, 16))],
                         ids=str)
def test_block_cg_sizes(bq, dims, ncols):
    tol = 1e-10
    U = inputs.gauge_field(dims, 0.2, seed=97)
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, dims, U, -1)
    op = bq.Op(G, 0.12, 1.5, 0.0)
    for n in ncols:
        b, x, y = (bq.Field(ctx, dims, bq.BQ_FULL, bq.BQ_F64, n) for _ in range(3))
        src = inputs.gaussian_spinor(dims, n, seed=98)
        if n > 3:
            src[2] = 0.0                    # a zero source is solved by x = 0
            src[3] = (2 - 1j) * src[0]      # a dependent one waits for its own run
        b.put(src)
        rc, info = op.solve(b, x, tol, system=bq.BQ_SYS_M, solver=bq.BQ_SOLVER_BLOCK_CG)
        assert rc == bq.BQ_OK and all(i["converged"] and i["true_rel_resid"] <= tol for i in info)
        op.solve(b, y, tol, system=bq.BQ_SYS_M)
        gx, gy = x.get(), y.get()
        # both stop at |r| <= tol |b'| of Mhat^dag Mhat, whose condition number here is below 100
        for c in range(n):
            assert np.linalg.norm(gx[c] - gy[c]) <= 200 * tol * max(np.linalg.norm(gy[c]), 1e-300)
        if n > 3:
            assert not gx[2].any()
