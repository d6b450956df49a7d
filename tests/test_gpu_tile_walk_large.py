"""Slab walks of lattices whose time slices, but not whose (x,y) planes, hold whole tiles, at the size from
which they are walked (4096 tiles), and the memory order below it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(24, 24, 24, 40), (24, 24, 24, 36)])  # 4320 tiles in slices of 108; 3888
def test_orders_are_bitwise_the_same(dims):
    from paper_1711_03836_amd import bqhip as bq
    rng = np.random.default_rng(95)
    V, n = int(np.prod(dims)), 2

    def noise(*shape):
        return (0.5 * rng.standard_normal((*shape, 2))).view(np.complex128)[..., 0]

    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, noise(4, V, 3, 3), -1), 0.1, 0.0, 0.1)  # any links: 18-real forms only
    src = noise(n, V, 4, 3)
    for prec in (bq.BQ_F64, bq.BQ_F32):
        fi, fo = bq.Field(ctx, dims, bq.BQ_ODD, prec, n), bq.Field(ctx, dims, bq.BQ_EVEN, prec, n)
        fi.put(src)
        for R, bs, lds in ((1, 768, 1), (1, 256, 0), (2, 128, 0)):
            out = []
            for order in (0, 1, 2):
                ctx.tune_set(prec, n, 18, R, bs, 0, lds, order)
                op.apply(bq.BQ_OP_K1, fi, fo)
                out.append(fo.get())
            assert out[0].any() and np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2]), (prec, R, lds)
        fi.close()
        fo.close()
