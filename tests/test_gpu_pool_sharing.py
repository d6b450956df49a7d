"""Device blocks kept for the next buffers, where others want the memory too: other sizes, other allocators,
other contexts, threads, and streams that still work on a field when it is freed."""
import re
import threading

import numpy as np
import pytest
import torch

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu

MIB = 1 << 20
DIMS = (32, 32, 32, 32)  # an odd FP64 field: 96 MiB a column


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


def _free():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _pass_through(bq, ctx, n):
    bq.Field(ctx, DIMS, bq.BQ_ODD, bq.BQ_F64, n).close()


def test_full_pool_takes_new_sizes(bq):
    """Eight blocks' worth of an old size does not keep a new size out: what is held in the end is the new one."""
    ctx = bq.Context(0, hbm_budget=8 << 30)  # the pool holds up to 1 GiB
    warm = bq.Field(ctx, (4, 4, 4, 4), bq.BQ_ODD, bq.BQ_F64, 1)
    before = _free()
    _pass_through(bq, ctx, 6)   # 576 MiB
    _pass_through(bq, ctx, 10)  # 960 MiB: no room beside the other
    held = (before - _free()) / MIB
    assert 900 < held < 1024
    _pass_through(bq, ctx, 11)  # 1056 MiB: larger than the pool may be, changes nothing
    assert abs((before - _free()) / MIB - held) < 64
    warm.close()


def test_memory_goes_back(bq):
    ctx, other = bq.Context(0), bq.Context(0)
    warm = [bq.Field(c, (4, 4, 4, 4), bq.BQ_ODD, bq.BQ_F64, 1) for c in (ctx, other)]
    before = _free()
    _pass_through(bq, ctx, 10)
    assert (before - _free()) / MIB > 900
    ctx.trim()
    assert abs(before - _free()) / MIB < 64
    ctx.trim()
    # a context without a budget of its own counts the blocks that others keep as free
    _pass_through(bq, ctx, 10)
    _pass_through(bq, other, 9)
    assert (before - _free()) / MIB > 1800
    with pytest.raises(bq.BqError) as e:
        bq.Field(bq.Context(0), DIMS, bq.BQ_ODD, bq.BQ_F64, 5000)  # 480 GiB: beyond any budget
    assert e.value.code == bq.BQ_ERR_OOM
    budget = int(re.search(r"of (\d+) in use", str(e.value)).group(1))
    assert abs(budget - 0.9 * before) / MIB < 64
    for f in warm:
        f.close()


def test_field_freed_under_a_stream(bq):
    dims, n = (16, 16, 16, 32), 4
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, inputs.gauge_field(dims, 0.2, seed=91), -1), 0.12, 1.5, 0.1)
    fi = bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F64, n)
    fi.put(inputs.gaussian_spinor(dims, n, seed=92))
    stream = torch.cuda.Stream()
    for _ in range(3):
        out = bq.Field(ctx, dims, bq.BQ_EVEN, bq.BQ_F64, n)
        for _ in range(100):  # no work fields: returns at once
            op.apply(bq.BQ_OP_K1, fi, out, stream=stream)
        out.close()
        fresh = bq.Field(ctx, dims, bq.BQ_EVEN, bq.BQ_F64, n)  # the same block
        stream.synchronize()
        assert not fresh.get().any()
        fresh.close()


def test_threads_and_trims(bq):
    """Two threads with a context each, while a third gives their blocks back and makes contexts."""
    dims, n = (8, 8, 8, 16), 2
    U, src = inputs.gauge_field(dims, 0.2, seed=93), inputs.gaussian_spinor(dims, n, seed=94)
    errors, left = [], [2]
    ctxs = [bq.Context(0) for _ in range(2)]

    def work(ctx):
        try:
            op = bq.Op(bq.Gauge(ctx, dims, U, -1), 0.12, 1.5, 0.1)
            first = None
            for k in range(40):
                fi, fo = (bq.Field(ctx, dims, bq.BQ_ODD, bq.BQ_F32, n) for _ in range(2))
                fi.put(src)
                op.apply(bq.BQ_OP_MHATDAG_MHAT, fi, fo)
                got = fo.get()
                first = got if first is None else first
                assert np.array_equal(got, first), k
                fi.close()
                fo.close()
        except Exception as e:  # noqa: BLE001  handed to the main thread
            errors.append(e)
        finally:
            left[0] -= 1

    threads = [threading.Thread(target=work, args=(c,)) for c in ctxs]
    for t in threads:
        t.start()
    for _ in range(2000):
        if left[0] == 0:
            break
        for c in ctxs:
            c.trim()
        bq.Context(0).close()
    for t in threads:
        t.join()
    assert not errors, errors
