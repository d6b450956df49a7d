"""Multishift CG where the vector kernels sum the partials themselves (up to 1024 tiles) and where a
launch of its own does: the base shift's solution does not depend on the other shifts, odd chunks end in
the second set of states, and every shift reaches its FP64 residual."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


# 3 tiles (the last part-filled), 1024 tiles (the most that are summed in place), 1088
@pytest.mark.parametrize("dims", [(6, 4, 4, 4), (16, 16, 16, 32), (16, 16, 16, 34)], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("base", [0.0, 0.02])
def test_base_shift_is_independent_of_the_others(bq, dims, base):
    tol = 1e-9
    U = inputs.gauge_field((dims[0], dims[1], dims[2], 2), 0.2, seed=95)  # repeated along t: cheap to make
    V2 = U.shape[1]
    U = np.tile(U.reshape(4, 1, V2, 3, 3), (1, dims[3] // 2, 1, 1, 1)).reshape(4, -1, 3, 3)
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, dims, U, -1)
    op = bq.Op(G, 0.12, 1.5, 0.05)
    b = bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, 2)
    b.put(inputs.gaussian_spinor(dims, 2, seed=96))
    runs = []
    for shifts, chunk in (([0.5, base, 3.0], 8), ([0.5, base, 3.0], 3), ([base], 8)):
        xs = [bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, 2) for _ in shifts]
        rc, info = op.solve_multishift(b, xs, shifts, tol, chunk=chunk)
        assert rc == bq.BQ_OK
        # the recursive residual stops at tol; the FP64 one may lie a little above it
        assert all(i["converged"] and i["true_rel_resid"] <= 1.1 * tol for k in info for i in k)
        k = shifts.index(base)
        runs.append((xs[k].get(), [i["iters"] for i in info[k]]))
    for x, it in runs[1:]:
        assert it == runs[0][1] and np.array_equal(x, runs[0][0])
