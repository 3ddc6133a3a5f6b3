"""Tracer transport with fields listed more than once, in one group of a launch
and in several, through several sub-cycles: each sub-cycle takes the list in
order, so the second mention of a field is transported after the first within
every sub-cycle.  Against the oracle on the same list; bar of the ten-substep
parity tests (1e-11; in mixed precision 1e-4)."""
import pytest

import fv3_inputs as fi
from test_gpu_parity import _int, _relerr, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz,order,nsplt,opts", [
    (0, 20, 3, (0, 1, 0), 2, {}), (0, 20, 2, (0, 0), 3, {}), (1, 12, 3, (0, 1, 2, 3, 4, 0, 2), 2, {}),
    (1, 12, 2, (0, 1, 1), 3, dict(edge_fix=True)), (1, 12, 2, (0, 1, 0), 2, dict(edge_ppm=True)),
    (0, 16, 3, (0, 1, 2, 3, 4, 5, 6, 7, 0), 2, dict(precision="mixed"))])
def test_repeated_fields(fv3, orc, kind, n, nz, order, nsplt, opts):  # noqa: F811
    import torch

    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz, nq=max(order) + 1)
    g = fv3.Grid(kind, n, nz, **opts)
    s = fv3.State.allocate(g)
    s.load(init)
    og = orc.Grid(kind, n, nz, delta=1000.0, **{k: v for k, v in opts.items() if k != "precision"})
    os_ = orc.new_state(og, init)
    dt = 0.4 if kind == 0 else 100.0
    fv3.acoustic_substeps(s, g, 2 * dt, 2)
    orc.acoustic_substeps(og, os_, 2 * dt, 2)
    qd, qh = [g.upload(q, nz) for q in init["q"]], [q.copy() for q in init["q"]]
    fv3.tracer_transport([qd[m] for m in order], s, g, nsplt=nsplt)
    orc.tracer_transport(og, [qh[m] for m in order], os_["dp0"], os_["mfx"], os_["mfy"], os_["cx"], os_["cy"], nsplt=nsplt)
    torch.cuda.synchronize()
    bar = 1e-4 if opts.get("precision") == "mixed" else 1e-11
    for m, (a, b) in enumerate(zip(qd, qh)):
        e = _relerr(_int(g.download(a, nz), n, "C"), _int(b, n, "C"))
        print(f"q{m} {e:.2e}", flush=True)
        assert e <= bar, (m, e)
