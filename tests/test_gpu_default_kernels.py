"""The kernel that a launch's size picks when no configuration was chosen (hop-split, plain or
tile-shared) against the plain kernel with one column per wave: bitwise, for every operator kind,
precision and link form, at the sizes where the choice changes and on lattices with a part-filled tile."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu

# tiles per parity: 1 (8 of 64 sites), 2 (96 of 128), 8, 119 (the last 8 sites full), 162
SMALL = [(2, 2, 2, 2), (6, 4, 4, 4), (4, 8, 4, 8), (6, 10, 14, 18), (12, 12, 12, 12)]
# columns whose (tiles x columns) lie at and beyond one round of hop-split workgroups (512 FP64, 1024 else)
COLS = {(2, 2, 2, 2): (1, 16), (6, 4, 4, 4): (3,), (4, 8, 4, 8): (2, 13), (6, 10, 14, 18): (4, 5, 8, 9),
        (12, 12, 12, 12): (3, 4, 6, 7)}


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


@pytest.mark.parametrize("dims", SMALL, ids=lambda d: "x".join(map(str, d)))
def test_picked_kernel_is_bitwise_the_plain_one(bq, dims):
    U = inputs.gauge_field(dims, 0.2, seed=71)
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, dims, U, -1)
    op = bq.Op(G, 0.12, 1.5, 0.1)
    for n in COLS[dims]:
        b = inputs.gaussian_spinor(dims, n, seed=72)
        for prec in (bq.BQ_F64, bq.BQ_F32, bq.BQ_F16):
            ins = {s: bq.Field(ctx, dims, s, prec, n) for s in (bq.BQ_EVEN, bq.BQ_ODD, bq.BQ_FULL)}
            outs = {s: bq.Field(ctx, dims, s, prec, n) for s in ins}
            for f in ins.values():
                f.put(b)
            d = ctx.tune_get(prec, n)
            assert d[3:] == (0, 0, 0)
            for recon in ((12,) if prec == bq.BQ_F16 else (12, 18)):
                for kind, (si, so) in bq.OP_SUBSETS.items():
                    got = []
                    for R, bs in ((d[1], d[2]), (1, 64)):  # the default's shape: the library picks; plain
                        ctx.tune_set(prec, n, recon, R, bs)
                        op.apply(kind, ins[si], outs[so])
                        got.append(outs[so].get())
                    assert np.array_equal(got[0], got[1]), (dims, n, prec, recon, kind)
            ctx.tune_set(prec, n, *d)


@pytest.mark.parametrize("dims,n", [((6, 4, 4, 6), 2), ((6, 10, 14, 18), 3)])
def test_solves_are_bitwise_the_plain_kernels(bq, dims, n):
    """Norm partials and the fused residual update of the picked kernels, through whole solves."""
    U = inputs.gauge_field(dims, 0.2, seed=73)
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, dims, U, -1)
    op = bq.Op(G, 0.12, 1.5, 0.1)
    b, x = (bq.Field(ctx, dims, bq.BQ_FULL, bq.BQ_F64, n) for _ in range(2))
    b.put(inputs.gaussian_spinor(dims, n, seed=74))
    runs = [dict(inner_prec=p, system=s) for p in (0, 1, 2) for s in (bq.BQ_SYS_M,)]
    runs += [dict(inner_prec=1, system=bq.BQ_SYS_M, **kw) for kw in (dict(chunk=1), dict(chunk=3), dict(use_graph=True))]
    runs += [dict(inner_prec=1, system=bq.BQ_SYS_M, maxiter=7, raise_on_error=False)]
    runs += [dict(inner_prec=0, system=bq.BQ_SYS_FULL_NORMAL),
             dict(inner_prec=1, system=bq.BQ_SYS_M, solver=bq.BQ_SOLVER_BICGSTAB)]
    got = []
    for plain in (False, True):
        if plain:
            for p in (0, 1, 2):
                ctx.tune_set(p, n, 12 if p == 2 else 18, 1, 64)
        for kw in runs:
            rc, info = op.solve(b, x, 1e-10, **kw)
            got.append((x.get(), [i["iters"] for i in info], [i["true_rel_resid"] for i in info]))
    for a, c in zip(got[:len(runs)], got[len(runs):]):
        assert np.array_equal(a[0], c[0]) and a[1:] == c[1:]
