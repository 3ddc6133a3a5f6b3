"""c_sw: widths at the edges of a strip (58 of the n + 3 points a row), layer
counts that leave wavefronts of a block idle, the smallest cube, and the
one-sided edge interpolation, on the C-grid winds after the half step.  The
bars are those of the single-stage parity tests (1e-13 of the largest wind;
with the edge stencils the same)."""
import pytest

import fv3_inputs as fi
from test_gpu_parity import _compare, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz,opts", [
    (0, 55, 1, {}), (0, 56, 2, {}), (0, 8, 5, {}), (1, 55, 1, {}), (1, 56, 2, {}), (1, 113, 1, {}), (1, 114, 1, {}),
    (1, 8, 3, {}), (1, 8, 2, dict(edge_interp=True)), (1, 55, 1, dict(edge_interp=True))])
def test_csw_widths(fv3, orc, kind, n, nz, opts):  # noqa: F811
    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz)
    g = fv3.Grid(kind, n, nz, **opts)
    s = fv3.State.allocate(g)
    s.load(init)
    og = orc.Grid(kind, n, nz, delta=1000.0, **opts)
    os_ = orc.new_state(og, init)
    dt = 0.4 if kind == 0 else 100.0
    fv3.acoustic_substeps(s, g, dt, 1, stop_stage=2)
    orc.acoustic_substeps(og, os_, dt, 1, stop_stage=2)
    _compare(s, os_, n, ("uc", "vc"), {k: 1e-13 for k in ("uc", "vc")}, f"csw kind{kind} n{n} nz{nz} {opts}")
