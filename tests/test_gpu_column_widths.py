"""Column solves and interface heights: columns per block from 16 to 256, as
the depth and the number of columns choose them (one chunk of up to five
layers with 256 columns, two with 128, four with 64, blocks left partial).
Bars of the single stages; the C-grid winds, through which the first solve
shows, carry its geopotential's error phi (bar 1e-13 of the largest) into the
half step's pressure gradient, dt / 2 phi / dx, which at these resolutions is
more than the 1e-13 of the wind itself: the bar is the sum of both."""
import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_parity import H, STAG, W_BAR, _compare, _int, _pair, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz", [(0, 368, 1), (0, 363, 5), (0, 260, 6), (0, 257, 8), (0, 260, 10), (0, 200, 18),
                                       (1, 150, 4), (0, 130, 20), (0, 9, 3)])
def test_wide(fv3, orc, kind, n, nz):  # noqa: F811
    init = fi.periodic_state(n=n, nz=nz) if kind == 0 else fi.cube_state(n=n, nz=nz)
    g, s, og, os_ = _pair(fv3, orc, kind, n, nz, init)
    dt = 0.4 if kind == 0 else 100.0
    grow = max(1.0, nz / 6.0)
    fv3.acoustic_substeps(s, g, dt, 1, stop_stage=8)
    orc.acoustic_substeps(og, os_, dt, 1, stop_stage=8)
    tol = {k: 1e-13 * grow for k in ("delp", "pt", "delz", "pfull", "phi", "uc", "vc")}
    tol["w"] = W_BAR * grow
    dx = np.abs(g.metric("dxc")[:, H:H + n, H:H + n]).min()
    for k in ("uc", "vc"):
        tol[k] += 0.5 * dt * tol["phi"] * np.abs(os_["phi"]).max() / dx / np.abs(_int(os_[k], n, STAG[k])).max()
    _compare(s, os_, n, tuple(tol), tol, f"wide kind{kind} n{n} nz{nz}")
