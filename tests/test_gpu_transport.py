"""Marching transport: widths at the edges of a strip (58 columns) and of its
halo, single-column remainders, and the tracer transport's groups (up to four
fields a launch, one given twice, an odd and an even number of sub-cycles,
the edge-flux fix-up).  Bars of the single-stage and ten-substep parity
tests (1e-13 after one d_sw, 1e-11 for the tracers); the accumulators carry
the error of the C-grid winds, an absolute one from the pressure gradient, so
without the mean wind of 10 m/s their relative bar grows by the ratio of the
largest winds with and without it."""
import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_parity import H, _compare, _int, _pair, _relerr, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz", [(0, 57, 2), (0, 58, 2), (0, 59, 2), (0, 61, 1), (1, 58, 1), (1, 59, 2),
                                       (0, 116, 1), (0, 117, 1), (0, 8, 3), (1, 8, 2)])
def test_widths(fv3, orc, kind, n, nz):  # noqa: F811
    init = fi.periodic_state(n=n, nz=nz, temp_noise=1.0) if kind == 0 else fi.cube_state(n=n, nz=nz)
    full = max(np.abs(init["u"]).max(), np.abs(init["v"]).max())
    if kind == 0:   # both signs of the Courant numbers
        for k in ("u", "v"):
            init[k] = init[k] - 10.0
    grow = full / max(np.abs(_int(init["u"], n, "Y")).max(), np.abs(_int(init["v"], n, "X")).max())
    g, s, og, os_ = _pair(fv3, orc, kind, n, nz, init)
    dt = 0.4 if kind == 0 else 100.0
    fields = ("u", "v", "delp", "pt", "w", "mfx", "mfy", "cx", "cy", "delz")
    fv3.acoustic_substeps(s, g, dt, 1, stop_stage=7)
    orc.acoustic_substeps(og, os_, dt, 1, stop_stage=7)
    tol = {k: 1e-13 * (grow if k in ("mfx", "mfy", "cx", "cy") else 1.0) for k in fields}
    _compare(s, os_, n, fields, tol, f"width kind{kind} n{n}")


@pytest.mark.parametrize("kind,n,nz,nq,nsplt,opts", [
    (0, 20, 3, 1, 1, {}), (0, 20, 3, 5, 2, {}), (1, 12, 3, 4, 3, {}), (1, 12, 2, 3, 2, dict(edge_fix=True)),
    (0, 59, 1, 2, 1, dict(hord_tr=7)), (0, 20, 2, 6, 1, dict(hord_tr=5))])
def test_tracer_groups(fv3, orc, kind, n, nz, nq, nsplt, opts):  # noqa: F811
    import torch

    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz, nq=nq)
    g = fv3.Grid(kind, n, nz, **opts)
    s = fv3.State.allocate(g)
    s.load(init)
    og = orc.Grid(kind, n, nz, delta=1000.0, **opts)
    os_ = orc.new_state(og, init)
    dt = 0.4 if kind == 0 else 100.0
    fv3.acoustic_substeps(s, g, 2 * dt, 2)
    orc.acoustic_substeps(og, os_, 2 * dt, 2)
    qd, qh = [g.upload(q, nz) for q in init["q"]], [q.copy() for q in init["q"]]
    fv3.tracer_transport(qd, s, g, nsplt=nsplt)
    orc.tracer_transport(og, qh, os_["dp0"], os_["mfx"], os_["mfy"], os_["cx"], os_["cy"], nsplt=nsplt)
    torch.cuda.synchronize()
    for m, (a, b) in enumerate(zip(qd, qh)):
        e = _relerr(_int(g.download(a, nz), n, "C"), _int(b, n, "C"))
        assert e <= 1e-11, (m, e)


def test_tracer_given_twice(fv3):  # noqa: F811
    """A field listed twice is transported twice, as by two calls."""
    import torch

    n, nz = 16, 2
    init = fi.periodic_state(n=n, nz=nz, nq=2)
    g = fv3.Grid(0, n, nz)
    s = fv3.State.allocate(g)
    s.load(init)
    fv3.acoustic_substeps(s, g, 0.8, 2)
    a = [g.upload(q, nz) for q in init["q"]]
    b = [g.upload(q, nz) for q in init["q"]]
    fv3.tracer_transport([a[0], a[1], a[0]], s, g, nsplt=1)
    fv3.tracer_transport(b, s, g, nsplt=1)
    fv3.tracer_transport([b[0]], s, g, nsplt=1)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        np.testing.assert_array_equal(g.download(x, nz)[..., H:H + n, H:H + n], g.download(y, nz)[..., H:H + n, H:H + n])
