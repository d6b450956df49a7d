"""Taking up a gauge configuration: links into every storage form, clover term and inverse in every
precision, plaquette, on lattices whose last tile is part-filled, against the oracle and bitwise
between the forms."""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2, 2), (2, 4, 2, 6), (6, 4, 4, 6), (4, 6, 8, 2), (6, 10, 4, 10)]
KAPPA, CSW, MU = 0.12, 1.5, 0.1


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("on_device", [False, True])
def test_configuration(bq, dims, on_device):
    import torch
    U = inputs.gauge_field(dims, 0.3, seed=85)
    ref = orc.Operator(dims, U, KAPPA, CSW, mu=MU)
    b = inputs.gaussian_spinor(dims, 2, seed=86)
    ctx = bq.Context(0)
    G = bq.Gauge(ctx, dims, torch.from_numpy(U).to("cuda:0") if on_device else U, -1)
    assert abs(G.plaquette() - orc.plaquette(dims, U)) <= 1e-14
    assert G.su3_deviation() <= 1e-14
    op = bq.Op(G, KAPPA, CSW, MU)
    res = {}
    # FP64: 12 terms of the clover and 48 of the hop per component, each to an ulp; FP32: its rounding of
    # links, clover and spinor and as many terms; FP16: the bound the parity tests state
    for prec, tol in ((bq.BQ_F64, 1e-13), (bq.BQ_F32, 2e-5), (bq.BQ_F16, 2e-2)):
        fi, fo = (bq.Field(ctx, dims, bq.BQ_FULL, prec, 2) for _ in range(2))
        ei, eo = (bq.Field(ctx, dims, bq.BQ_EVEN, prec, 2) for _ in range(2))
        fi.put(b)
        ei.put(b)
        for recon in ((12,) if prec == bq.BQ_F16 else (18, 12)):  # both link forms hold the same field
            ctx.tune_set(prec, 2, recon, 1, 64)
            op.apply(bq.BQ_OP_M, fi, fo)
            for c in range(2):
                want = ref.M(b[c])
                assert np.abs(fo.get()[c] - want).max() <= tol * np.abs(want).max(), (prec, recon)
        op.apply(bq.BQ_OP_CLOVER, fi, fo)
        op.apply(bq.BQ_OP_CLOVER_INV, ei, eo)
        res[prec] = (fo.get(), eo.get())
        for c in range(2):
            want = orc.clover_apply(dims, ref.T, b[c])
            assert np.abs(res[prec][0][c] - want).max() <= tol * np.abs(want).max()
            want = ref.even(orc.clover_apply(dims, ref.Tinv, b[c]))
            assert np.abs(ref.even(res[prec][1][c]) - want).max() <= tol * np.abs(want).max()
    # a field that is SU(3) to FP32 but not to FP64 keeps the two-row forms of FP32 and FP16 only
    V = U.copy()
    V[1, 0] *= 1 + 1e-9
    G2 = bq.Gauge(ctx, dims, V, -1)
    assert 1e-9 < G2.su3_deviation() < 1e-8
    op2 = bq.Op(G2, KAPPA, CSW, MU)
    for prec in (bq.BQ_F64, bq.BQ_F32, bq.BQ_F16):
        fi, fo = (bq.Field(ctx, dims, bq.BQ_FULL, prec, 2) for _ in range(2))
        fi.put(b)
        ctx.tune_set(prec, 2, 12, 1, 64)
        op2.apply(bq.BQ_OP_M, fi, fo)
        assert np.isfinite(fo.get()).all()
