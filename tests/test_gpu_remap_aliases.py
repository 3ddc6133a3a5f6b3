"""Remap with fields listed more than once: a tracer repeated further apart
than the fields of one launch, state fields among the tracers, and delp itself
among them.  Bit for bit what the call without the repetition gives."""
import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_remap import H, fv3  # noqa: F401

pytestmark = pytest.mark.gpu
STATE = ("u", "v", "w", "delp", "pt", "delz")


def _start(fv3, kind, n, nz, precision, nq):  # noqa: F811
    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz, nq=nq)
    init["delp"] = fi.deform_layers(init["delp"], seed=2)
    g = fv3.Grid(kind, n, nz, precision=precision)
    s = fv3.State.allocate(g)
    s.load(init)
    return g, s, [g.upload(q, nz) for q in init["q"]], fi.hybrid_coefficients(nz, g.ptop)


def _fields(g, s, qd, n, nz, names=STATE):
    sl = (Ellipsis, slice(H, H + n), slice(H, H + n))
    return [s.get(k)[sl] for k in names] + [g.download(q, nz)[sl] for q in qd]


@pytest.mark.parametrize("kind,n,nz,precision", [(0, 16, 9, "fp64"), (1, 8, 20, "mixed")])
@pytest.mark.parametrize("order", [(0, 1, 2, 3, 4, 0), (0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 0, 5, 11), ("pt", 0, 1, 2, 3, 4, 5, "w", "delz")])
def test_listed_again(fv3, kind, n, nz, precision, order):  # noqa: F811
    import torch

    out = []
    for again in (True, False):
        g, s, qd, (ak, bk) = _start(fv3, kind, n, nz, precision, 12)
        lst = order if again else [m for q, m in enumerate(order) if not isinstance(m, str) and m not in order[:q]]
        fv3.remap(s, g, ak, bk, [s.f[m] if isinstance(m, str) else qd[m] for m in lst])
        torch.cuda.synchronize()
        assert fv3.check_status(g) == 0
        out.append(_fields(g, s, qd, n, nz))
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("kind,n,nz,precision", [(0, 16, 9, "mixed"), (1, 8, 20, "fp64")])
@pytest.mark.parametrize("nq", [0, 6])
def test_delp_listed(fv3, kind, n, nz, precision, nq):  # noqa: F811
    """Every other field is remapped with the layers the call was given; delp
    takes the reference thickness of the surface pressure that its own remapped
    values add up to."""
    import torch

    out = []
    for listed in (True, False):
        g, s, qd, (ak, bk) = _start(fv3, kind, n, nz, precision, nq + 1)
        extra = s.f["delp"] if listed else qd[nq].copy_(s.f["delp"])
        fv3.remap(s, g, ak, bk, [extra] + qd[:nq])
        torch.cuda.synchronize()
        out.append(_fields(g, s, qd[:nq], n, nz, ("u", "v", "w", "pt", "delz")))
        sl = (Ellipsis, slice(H, H + n), slice(H, H + n))
        if listed:
            got = s.get("delp")[sl]
        else:
            x = g.download(qd[nq], nz)[sl]
            ps = np.full_like(x[:, 0], g.ptop)
            for k in range(nz):
                ps = ps + x[:, k]
            pe = ak[:, None, None, None] + bk[:, None, None, None] * ps[None]
            want = np.moveaxis(np.diff(pe, axis=0), 0, 1)
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
    # three roundings of interface pressures of 1e5 Pa, then that of the field
    assert np.abs(got - want).max() <= 4 * 2.0 ** -53 * 1.1e5 + (2.0 ** -24 * want.max() if precision == "mixed" else 0.0)
