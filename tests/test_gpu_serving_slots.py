"""Server sessions with free slots, and holes among those in use: stencils cover the slots in use only, in the
kernel that their number picks, and every column's result is bitwise that of any kernel and of its request alone."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu

DIMS = (6, 10, 14, 18)  # 119 tiles, the last 8 sites full
SLOTS = 16
# columns, kappa, tolerance; the third is sent when the first has left
REQS = [(3, 0.121, 1e-3), (9, 0.122, 1e-9), (2, 0.119, 1e-8)]


def _serve(bq, ctx, G, which, prec, tunes):
    for p in {prec, bq.BQ_F64}:
        ctx.tune_set(p, SLOTS, *tunes)
    srv = bq.Server(ctx, SLOTS, 8)
    tickets, out = {}, {}

    def send(i):
        n, kappa, tol = REQS[i]
        tickets[srv.submit(G, inputs.gaussian_spinor(DIMS, n, seed=60 + i), kappa, 1.5, 0.0, tol, prec)] = i

    for i in which:
        if i < 2 or len(which) == 1:
            send(i)
    while len(out) < len(which):
        for t in srv.step():
            out[tickets[t]] = srv.result(t)
            if tickets[t] == 0 and 2 in which:
                assert 1 not in out  # its nine columns are still in slots 3 to 11
                send(2)
    srv.close()
    return out


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_slots_in_use(prec):
    from paper_1711_03836_amd import bqhip as bq
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, DIMS, inputs.gauge_field(DIMS, 0.2, seed=59), -1)
    free = (12, 0, 0)
    want = _serve(bq, ctx, G, (0, 1, 2), prec, free)
    for i, (n, _, tol) in enumerate(REQS):
        rc, info, _ = want[i]
        assert rc == bq.BQ_OK and len(info) == n and all(c["true_rel_resid"] <= tol for c in info)
    runs = [((0, 1, 2), t) for t in ((12, 1, 64), (12, 2, 128), (12, 1, 768, 0, 1, 0), (12, 1, 512, 0, 1, 2))]
    runs += [((i,), free) for i in range(3)] + [((1,), (12, 1, 768, 0, 1, 1))]
    for which, tunes in runs:
        got = _serve(bq, ctx, G, which, prec, tunes)
        for i in which:
            assert got[i][0] == want[i][0]
            assert [c["iters"] for c in got[i][1]] == [c["iters"] for c in want[i][1]]
            assert np.array_equal(got[i][2], want[i][2]), (which, tunes, i)
