"""Remap: layer counts at the edges of the 16 chunks of target layers a column
is cut into (chunks left empty, the last one short, the largest LDS), columns
that leave a block of 16 ragged, and a tracer listed twice (remapped once).  Bars of the remap parity
tests."""
import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_remap import _bars, _run_pair, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz,precision,coef", [
    (0, 9, 5, "fp64", "sigma"), (0, 9, 7, "fp64", "hybrid"), (0, 9, 8, "mixed", "hybrid"), (0, 33, 17, "fp64", "hybrid"), (0, 8, 16, "fp64", "hybrid"),
    (1, 12, 64, "mixed", "sigma"), (0, 10, 127, "fp64", "hybrid"), (0, 10, 128, "fp64", "hybrid")])
def test_chunks(fv3, orc, kind, n, nz, precision, coef):  # noqa: F811
    errs, *_ = _run_pair(fv3, orc, kind, n, nz, precision, coef=coef)
    bar = _bars(precision)
    for k, e in errs.items():
        assert e <= bar(k), (k, e)


def test_field_given_twice(fv3):  # noqa: F811
    import torch

    n, nz, H = 16, 9, 3
    init = fi.periodic_state(n=n, nz=nz, nq=3)
    init["delp"] = fi.deform_layers(init["delp"], seed=2)
    g = fv3.Grid(0, n, nz)
    ak, bk = fi.hybrid_coefficients(nz, g.ptop)
    out = []
    for order in ((0, 1, 2, 0), (0, 1, 2)):
        s = fv3.State.allocate(g)
        s.load(init)
        qd = [g.upload(q, nz) for q in init["q"]]
        fv3.remap(s, g, ak, bk, [qd[m] for m in order])
        torch.cuda.synchronize()
        out.append([g.download(q, nz)[..., H:H + n, H:H + n] for q in qd])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
