"""Slab walks of the stencils' tiles: lattices whose time slices, but not whose (x,y) planes, hold whole
tiles, and planes cut in y as well as z."""
import importlib

import numpy as np
import pytest

from paper_1711_03836_amd import inputs
from oracle import oracle as orc
from test_gpu_parity import TOL, maxrel, oracle_apply

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(8, 8, 24, 4), (12, 12, 8, 4), (16, 32, 16, 4), (8, 6, 10, 6)])
@pytest.mark.parametrize("prec,recon,R,bs,lds", [(0, 18, 1, 768, 1), (1, 18, 1, 768, 1), (1, 12, 1, 256, 1), (2, 12, 1, 768, 1),
                                                  (0, 18, 2, 128, 0)])
def test_slab_walks_bitwise(dims, prec, recon, R, bs, lds):
    """Orders 1 and 2 on slices of 12 tiles (four slabs of 3), slices of 9 (one slab), planes of 4 tiles
    (cut into slabs of 1 tile by 8 planes) and slices of no whole tiles visit the work items of order 0 and do
    each site's arithmetic in the same order: bitwise equal, and the oracle's result."""
    bq = importlib.import_module("paper_1711_03836_amd.bqhip")
    nrhs = 12
    U = inputs.gauge_field(dims, 0.3, seed=71)
    ctx = bq.Context(0)
    op = bq.Op(bq.Gauge(ctx, dims, U, -1), 0.124, 1.5, 0.1)
    ref = orc.Operator(dims, U, 0.124, 1.5, mu=0.1)
    psi = inputs.gaussian_spinor(dims, nrhs, seed=72)
    for name in ("K1", "MHATDAG_MHAT", "MDAG"):
        kind = getattr(bq, "BQ_OP_" + name)
        si, so = bq.OP_SUBSETS[kind]
        out = {}
        for order in (0, 1, 2):
            ctx.tune_set(prec, nrhs, recon, R, bs, 0, lds, order)
            fi, fo = bq.Field(ctx, dims, si, prec, nrhs), bq.Field(ctx, dims, so, prec, nrhs)
            fi.put(psi)
            op.apply(kind, fi, fo)
            out[order] = fo.get()
        assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2]), name
        mask = {bq.BQ_EVEN: ref.parity == 0, bq.BQ_ODD: ref.parity == 1, bq.BQ_FULL: np.ones(ref.V, bool)}[so]
        want = oracle_apply(ref, kind, bq, psi[nrhs - 1])
        assert maxrel(out[1][nrhs - 1][mask], want[mask]) < TOL[prec], name
