"""nh_p_grad: widths at the edges of a strip (58 of the n + 1 corners a row),
layer counts that leave wavefronts of a block idle, grids large enough for two
layers a wavefront (even and odd counts), and the edge stencils.  The bars are
those of the single-stage parity tests (1e-13 of the largest wind)."""
import pytest

import fv3_inputs as fi
from test_gpu_parity import _compare, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz,opts", [
    (0, 57, 1, {}), (0, 58, 5, {}), (0, 8, 3, {}), (1, 57, 2, {}), (1, 58, 3, {}), (1, 8, 127, {}), (1, 8, 129, {}),
    (1, 8, 130, {}), (1, 58, 65, {}), (1, 8, 3, dict(edge_interp=True)), (1, 8, 129, dict(edge_interp=True))])
def test_nhgrad_widths(fv3, orc, kind, n, nz, opts):  # noqa: F811
    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz)
    g = fv3.Grid(kind, n, nz, **opts)
    s = fv3.State.allocate(g)
    s.load(init)
    og = orc.Grid(kind, n, nz, delta=1000.0, **opts)
    os_ = orc.new_state(og, init)
    dt = 0.4 if kind == 0 else 100.0
    fv3.acoustic_substeps(s, g, dt, 1, stop_stage=10)
    orc.acoustic_substeps(og, os_, dt, 1, stop_stage=10)
    _compare(s, os_, n, ("u", "v"), {k: 1e-13 for k in ("u", "v")}, f"nhgrad kind{kind} n{n} nz{nz} {opts}")
