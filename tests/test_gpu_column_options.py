"""Column solves with their options at depth: off-centring, the cubic interface
perturbation and humidity together, where chunks have neighbours on both sides
(11 to 163 layers: a last chunk of one layer, whose neighbour above reads two
layers on; the most of the short chunks; the long ones), and each precision.

Bars: those of the plain solve at depth (1e-13, w 3e-11, times nz / 6), times
4: the cubic interface value weighs the layers' errors by at most 16 / 12, the
off-centred scan divides by beta = 0.75 and adds (1 - beta) / beta of P*, a
third.  In mixed precision the mixed bars (1e-4, w 1e-2)."""
import pytest

import fv3_inputs as fi
from test_gpu_parity import W_BAR, _compare, _humid, fv3  # noqa: F401

pytestmark = pytest.mark.gpu
FIELDS = ("w", "delz", "pfull", "phi", "delp", "pt")


@pytest.mark.parametrize("kind,n,nz,precision,opts,moist", [
    (1, 8, 11, "fp64", dict(beta=0.75, pp_order=4), True), (0, 9, 16, "fp64", dict(beta=0.75, pp_order=4), True),
    (1, 8, 81, "fp64", dict(beta=0.75, pp_order=4), True), (0, 9, 160, "fp64", dict(beta=0.75, pp_order=4), True),
    (0, 9, 163, "fp64", dict(beta=0.75, pp_order=4), True), (1, 8, 177, "fp64", dict(beta=0.75, pp_order=4), True),
    (1, 8, 16, "fp64", dict(pp_order=4), False), (0, 9, 21, "fp64", dict(beta=0.75), False), (0, 9, 1, "fp64", dict(beta=0.75, pp_order=4), True),
    (0, 9, 2, "fp64", dict(beta=0.75, pp_order=4), True), (0, 9, 6, "fp64", dict(beta=0.75, pp_order=4), False),
    (1, 8, 16, "mixed", dict(beta=0.75, pp_order=4), True), (0, 9, 81, "mixed", dict(beta=0.75, pp_order=4), True),
    (1, 8, 163, "mixed", dict(beta=0.75, pp_order=4), True), (0, 9, 170, "mixed", {}, False)])
def test_depths(fv3, orc, kind, n, nz, precision, opts, moist):  # noqa: F811
    init = (fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz)
    if moist:
        init = _humid(init, n, 70 + n)
    g = fv3.Grid(kind, n, nz, precision=precision, **opts)
    s = fv3.State.allocate(g)
    s.load(init)
    og = orc.Grid(kind, n, nz, **opts)
    os_ = orc.new_state(og, init)
    dt = 0.4 if kind == 0 else 100.0
    fv3.acoustic_substeps(s, g, dt, 1, stop_stage=8)
    assert orc.acoustic_substeps(og, os_, dt, 1, stop_stage=8) == 0
    grow = 4.0 * max(1.0, nz / 6.0)
    if precision == "mixed":
        tol = {k: 1e-2 if k == "w" else 1e-4 for k in FIELDS}
    else:
        tol = {k: (W_BAR if k == "w" else 1e-13) * grow for k in FIELDS}
    _compare(s, os_, n, FIELDS, tol, f"options kind{kind} nz{nz} {precision} {opts} moist{moist}")
