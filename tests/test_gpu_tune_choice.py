"""A stencil configuration is what the caller set: also one that earlier stood for the library's own choice
(R columns, 128 or 256 sites, nothing else); that choice has a value of its own."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu


def test_choice_and_no_choice(tmp_path):
    from paper_1711_03836_amd import bqhip as bq
    dims, n = (6, 10, 14, 18), 12  # 119 tiles: beyond the hop split in every precision
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, inputs.gauge_field(dims, 0.2, seed=75), -1), 0.12, 1.5, 0.1)
    src = inputs.gaussian_spinor(dims, n, seed=76)
    for prec, plain in ((bq.BQ_F64, (18, 2, 128)), (bq.BQ_F32, (18, 4, 128)), (bq.BQ_F16, (12, 4, 128))):
        free = ctx.tune_get(prec, n)
        assert free == (plain[0], 0, 0, 0, 0, 0)
        fi, fo = bq.Field(ctx, dims, bq.BQ_ODD, prec, n), bq.Field(ctx, dims, bq.BQ_EVEN, prec, n)
        fi.put(src)
        got = []
        for t in (free, (12, 0, 0), plain, (12, *plain[1:]), free):
            ctx.tune_set(prec, n, *t)
            assert ctx.tune_get(prec, n) == tuple(t) + (0,) * (6 - len(t))
            op.apply(bq.BQ_OP_K1, fi, fo)
            got.append(fo.get())
        assert np.array_equal(got[0], got[2]) and np.array_equal(got[0], got[4])
        assert np.array_equal(got[1], got[3])
        with pytest.raises(bq.BqError):
            ctx.tune_set(bq.BQ_F16, n, 18, 0, 0)  # no such link form
        for bad in ((0, 64), (1, 0), (0, 0, 2), (0, 0, 0, 1), (0, 0, 0, 0, 1)):
            with pytest.raises(bq.BqError):
                ctx.tune_set(prec, n, plain[0], *bad)
        assert ctx.tune_get(prec, n) == free
    with pytest.raises(bq.BqError):
        ctx.tune_set(bq.BQ_F64, 0, 18, 0, 0)
    # through a file: no choice stays none, a choice stays one
    ctx.tune_set(bq.BQ_F32, n, 18, 4, 128)
    ctx.save_tuning(tmp_path / "t.json", [(bq.BQ_F64, n), (bq.BQ_F32, n)])
    other = bq.Context(0)
    other.load_tuning(tmp_path / "t.json")
    assert other.tune_get(bq.BQ_F64, n) == (18, 0, 0, 0, 0, 0) and other.tune_get(bq.BQ_F32, n) == (18, 4, 128, 0, 0, 0)


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (16, 16, 16, 16)])  # hop split; tile-shared
def test_autotuned_entry_names_its_kernel(dims):
    from paper_1711_03836_amd import bqhip as bq
    n = 12
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, inputs.gauge_field(dims, 0.2, seed=77), -1), 0.12, 1.5, 0.1)
    op.autotune(bq.BQ_F32, n)
    t = ctx.tune_get(bq.BQ_F32, n)
    ctx.tune_set(bq.BQ_F32, n, *t)
    assert ctx.tune_get(bq.BQ_F32, n) == t
    assert t[1:] == (0,) * 5 or t[1] > 0 and t[2] >= 64
    if np.prod(dims) // 128 * n > 1024:  # beyond the hop split every kernel has a name
        assert t[1] > 0


@pytest.mark.parametrize("prec,recon,R,bs", [(0, 18, 1, 768), (1, 18, 1, 1024), (1, 12, 2, 768), (2, 12, 1, 576)])
def test_tile_shared_with_one_column_group(prec, recon, R, bs):
    """As many columns as a thread has: nothing to share, so the plain kernel runs, within its 512 threads."""
    from paper_1711_03836_amd import bqhip as bq
    dims = (6, 10, 14, 18)  # 119 tiles: not a multiple of the 8 of a workgroup
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, inputs.gauge_field(dims, 0.2, seed=78), -1), 0.12, 1.5, 0.1)
    fi, fo = bq.Field(ctx, dims, bq.BQ_ODD, prec, R), bq.Field(ctx, dims, bq.BQ_ODD, prec, R)
    fi.put(inputs.gaussian_spinor(dims, R, seed=79))
    got = []
    for t in ((recon, 1, 64), (recon, R, bs, 0, 1)):
        ctx.tune_set(prec, R, *t)
        op.apply(bq.BQ_OP_MHATDAG_MHAT, fi, fo)
        got.append(fo.get())
    assert np.array_equal(*got)
