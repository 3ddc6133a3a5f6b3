"""Marching kernels in mixed precision: strips in c_sw (58 of n + 3 points),
the transports (58 of n) and nh_p_grad (58 of n + 1), one, two and three of
them, and the tracer transport in groups of one to four fields, an odd and an
even number of sub-cycles, with the edge-flux fix-up and every order.  Against
the FP64 oracle at the mixed-precision bars (1e-4 of the largest value, w
1e-2): the states carry grid-scale noise of a tenth of the wind, so a
neighbour taken from the wrong lane or strip stands far above them."""
import pytest

import fv3_inputs as fi
from test_gpu_parity import _compare, _int, _relerr, fv3  # noqa: F401

pytestmark = pytest.mark.gpu
FIELDS = ("u", "v", "w", "delp", "pt", "delz", "uc", "vc", "mfx", "mfy", "cx", "cy", "pfull", "phi")
TOL = {k: 1e-2 if k == "w" else 1e-4 for k in FIELDS}


def _run(fv3, orc, kind, n, nz, ns, nq=0, **opts):  # noqa: F811
    init = fi.periodic_state(n=n, nz=nz, nq=nq, temp_noise=1.0) if kind == 0 else fi.cube_state(n=n, nz=nz, nq=nq)
    g = fv3.Grid(kind, n, nz, precision="mixed", **opts)
    s = fv3.State.allocate(g)
    s.load(init)
    og = orc.Grid(kind, n, nz, delta=1000.0, **opts)
    os_ = orc.new_state(og, init)
    dt = 0.4 if kind == 0 else 100.0
    fv3.acoustic_substeps(s, g, ns * dt, ns)
    orc.acoustic_substeps(og, os_, ns * dt, ns)
    return init, g, s, og, os_


@pytest.mark.parametrize("kind,n,nz,opts", [
    (0, 55, 2, {}), (0, 56, 2, {}), (0, 59, 3, {}), (0, 117, 2, {}), (1, 57, 2, {}), (1, 59, 2, {}), (1, 117, 1, {}),
    (0, 59, 2, dict(hord=5)), (1, 59, 2, dict(hord=6)), (1, 59, 2, dict(edge_fix=True)),
    (1, 59, 2, dict(edge_interp=True)), (1, 12, 66, {})])
def test_substeps(fv3, orc, kind, n, nz, opts):  # noqa: F811
    _, g, s, og, os_ = _run(fv3, orc, kind, n, nz, 2, **opts)
    assert fv3.check_status(g) == 0
    _compare(s, os_, n, FIELDS, TOL, f"mixed kind{kind} n{n} nz{nz} {opts}")


@pytest.mark.parametrize("kind,n,nz,nq,nsplt,opts", [
    (0, 59, 2, 1, 1, {}), (0, 59, 2, 2, 2, {}), (1, 12, 3, 3, 1, {}), (1, 59, 1, 4, 2, {}), (0, 117, 1, 4, 3, {}),
    (1, 12, 2, 5, 2, {}), (0, 20, 2, 7, 1, {}), (1, 12, 2, 4, 2, dict(edge_fix=True)), (1, 12, 3, 3, 1, dict(edge_fix=True)),
    (0, 59, 2, 4, 1, dict(hord_tr=7)), (1, 12, 2, 4, 2, dict(hord_tr=5)), (0, 61, 1, 2, 1, dict(hord_tr=6))])
def test_tracer_groups(fv3, orc, kind, n, nz, nq, nsplt, opts):  # noqa: F811
    import torch

    init, g, s, og, os_ = _run(fv3, orc, kind, n, nz, 2, nq=nq, **opts)
    qd, qh = [g.upload(q, nz) for q in init["q"]], [q.copy() for q in init["q"]]
    fv3.tracer_transport(qd, s, g, nsplt=nsplt)
    orc.tracer_transport(og, qh, os_["dp0"], os_["mfx"], os_["mfy"], os_["cx"], os_["cy"], nsplt=nsplt)
    torch.cuda.synchronize()
    for m, (a, b) in enumerate(zip(qd, qh)):
        e = _relerr(_int(g.download(a, nz), n, "C"), _int(b, n, "C"))
        print(f"q{m} {e:.2e}", flush=True)
        assert e <= 1e-4, (m, e)
