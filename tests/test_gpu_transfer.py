"""Fields into the library's layout and back: every site of the subset, part-filled last tiles, both
parities at once and one alone, and nothing outside the subset."""
import numpy as np
import pytest

from paper_1711_03836_amd import inputs

pytestmark = pytest.mark.gpu

# tiles per parity: a part of one, one and a part, 3 (odd: a workgroup's second tile is past the end), 119
DIMS = [(2, 2, 2, 2), (6, 4, 4, 4), (6, 4, 4, 2), (4, 4, 4, 6), (6, 10, 14, 18)]


@pytest.fixture(scope="module")
def bq():
    from paper_1711_03836_amd import bqhip
    return bqhip


@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("on_device", [False, True])
def test_round_trip(bq, dims, on_device):
    import torch
    ctx = bq.Context(0)
    V = int(np.prod(dims))
    odd = np.sum(inputs.coords(dims), axis=1) % 2 == 1
    for n in (1, 3):
        a = inputs.gaussian_spinor(dims, n, seed=81)
        a[0, V // 2] = 0.0  # an FP16 site of scale zero
        for prec in (bq.BQ_F64, bq.BQ_F32, bq.BQ_F16):
            if prec == bq.BQ_F64:
                want, tol = a, 0.0
            elif prec == bq.BQ_F32:
                want, tol = a.astype(np.complex64).astype(np.complex128), 0.0
            else:  # binary16 of each value over its site's largest component (FP32)
                tol = 2.0**-11 + 2.0**-22
                want = a
            for subset, held in ((bq.BQ_FULL, np.ones(V, bool)), (bq.BQ_ODD, odd), (bq.BQ_EVEN, ~odd)):
                f = bq.Field(ctx, dims, subset, prec, n)
                out = np.full_like(a, 7.0 - 3.0j)
                if on_device:
                    f.put(torch.from_numpy(a).to("cuda:0"))
                    t = torch.from_numpy(out).to("cuda:0")
                    f.get(out=t)
                    out = t.cpu().numpy()
                else:
                    f.put(a)
                    f.get(out=out)
                assert np.all(out[:, ~held] == 7.0 - 3.0j)
                if tol == 0.0:
                    assert np.array_equal(out[:, held], want[:, held])
                else:
                    x = out[:, held].view(np.float64).reshape(n, -1, 24)
                    y = want[:, held].view(np.float64).reshape(n, -1, 24)
                    scale = np.abs(y).max(axis=2, keepdims=True)
                    assert np.all(np.abs(x - y) <= tol * scale)
