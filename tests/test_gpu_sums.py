"""Mass sums in groups of six fields: one to three groups, a single level and
levels that leave a remainder of the four loaded ahead, against exact
rational sums of the same products; and that a sum does not depend on the
other fields of its call.  The compensated sums of the blocks and their
combination are accurate to a few units in the last place (bar 4 eps of the
sum of magnitudes, as for the conservation tests)."""
import math

import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_parity import H, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz,nq,precision", [(0, 9, 1, 0, "fp64"), (0, 66, 5, 4, "mixed"), (0, 20, 6, 5, "fp64"),
                                                    (1, 10, 3, 11, "mixed"), (0, 8, 7, 16, "fp64")])
def test_groups(fv3, kind, n, nz, nq, precision):  # noqa: F811
    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz, nq=1)
    g = fv3.Grid(kind, n, nz, precision=precision)
    s = fv3.State.allocate(g)
    s.load(init)
    rng = np.random.default_rng(n)
    qs = [g.upload(rng.standard_normal(init["delp"].shape) * 10.0 ** m, nz) for m in range(nq)]
    got = fv3.mass_sums(g, s.f["delp"], s.f["pt"], qs)
    sl = (Ellipsis, slice(H, H + n), slice(H, H + n))
    area = g.metric("area")[sl][:, None]
    m = g.download(s.f["delp"], nz)[sl] * area
    for k, f in enumerate([None, s.f["pt"]] + qs):
        x = m if f is None else g.download(f, nz)[sl] * m
        ref, mag = math.fsum(x.ravel()), math.fsum(np.abs(x).ravel())
        assert abs(got[k] - ref) <= 4 * np.finfo(float).eps * mag, (k, got[k], ref)
    if nq > 1:
        alone = fv3.mass_sums(g, s.f["delp"], s.f["pt"], [qs[-1]])
        assert alone[2] == got[1 + nq] and alone[0] == got[0]
