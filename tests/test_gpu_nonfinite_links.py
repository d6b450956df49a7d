"""A gauge field with one component that is not finite is refused, wherever the component lies."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu

DIMS = (6, 4, 4, 6)  # 288 sites per parity: the last 64-site tile is half full
V = int(np.prod(DIMS))
# direction, site (the first; the last of each parity), row, column, imaginary part
PLACES = [(0, 0, 0, 0, False), (3, V - 1, 2, 2, True), (2, V - 2, 1, 2, True)]


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("mu,site,row,col,imag", PLACES)
def test_refused(mu, site, row, col, imag, value):
    from paper_1711_03836_amd import bqhip as bq
    ctx = bq.Context(0)
    U = np.array(inputs.gauge_field(DIMS, 0.2, seed=85))
    bq.Gauge(ctx, DIMS, U, -1).close()
    part = (U.imag if imag else U.real).reshape(4, V, 3, 3)
    part[mu, site, row, col] = value
    with pytest.raises(bq.BqError) as e:
        bq.Gauge(ctx, DIMS, U, -1)
    assert e.value.code == bq.BQ_ERR_NONFINITE
