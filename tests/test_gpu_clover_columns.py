"""The clover applied to columns that share it in registers, on lattices large enough for that (FP16: 2048
tiles, FP32: 256), against FP64 and against the columns one by one."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs
from test_gpu_parity import TOL, maxrel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(16, 16, 16, 64), (12, 12, 20, 92), (16, 16, 16, 8), (6, 10, 14, 40)])
def test_shared_clover(dims):
    from paper_1711_03836_amd import bqhip as bq
    n, V = 5, int(np.prod(dims))
    short = (*dims[:3], 2)
    U = np.tile(inputs.gauge_field(short, 0.2, seed=96), (1, dims[3] // 2, 1, 1))  # t is the slowest index
    src = inputs.gaussian_spinor(dims, n, seed=97)
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, U, -1), 0.12, 1.5, 0.0)
    for kind in (bq.BQ_OP_CLOVER, bq.BQ_OP_CLOVER_INV):
        out, (si, so) = {}, bq.OP_SUBSETS[kind]
        for prec in (bq.BQ_F64, bq.BQ_F32, bq.BQ_F16):
            for cols in (n, 1):
                fi, fo = bq.Field(ctx, dims, si, prec, cols), bq.Field(ctx, dims, so, prec, cols)
                fi.put(src[:cols])
                op.apply(kind, fi, fo)
                out[prec, cols] = fo.get()
                fi.close()
                fo.close()
            assert np.array_equal(out[prec, n][0], out[prec, 1][0]), (kind, prec)
            assert out[prec, n].shape == (n, V, 4, 3)
            assert maxrel(out[prec, n], out[bq.BQ_F64, n]) < TOL[prec], (kind, prec)
