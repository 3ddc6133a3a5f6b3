"""The halo of delz after a call: the exchange at the start of the last substep
(stage 1 of the substep covers every cell field), alone, stopped after a stage,
and in an ensemble.  Bit for bit, against the halo exchange of the thicknesses
that substep starts from."""
import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_parity import H, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


def _state(fv3, kind, n, nz, precision):  # noqa: F811
    g = fv3.Grid(kind, n, nz, precision=precision)
    s = fv3.State.allocate(g)
    s.load((fi.periodic_state if kind == 0 else fi.cube_state)(n=n, nz=nz))
    return g, s


@pytest.mark.parametrize("kind,n,nz,precision,stop", [(0, 9, 3, "fp64", 0), (0, 9, 3, "mixed", 1), (1, 8, 4, "mixed", 0),
                                                      (1, 10, 2, "fp64", 1), (1, 8, 6, "fp64", -1), (0, 20, 2, "mixed", -1)])
def test_delz_halo(fv3, kind, n, nz, precision, stop):  # noqa: F811
    import torch

    dt = 0.4 if kind == 0 else 100.0
    g, s = _state(fv3, kind, n, nz, precision)
    fv3.acoustic_substeps(s, g, dt, 1)
    ref = s.f["delz"]
    fv3.halo_fill(g, [ref], nz, fp64=True)
    g2, s2 = _state(fv3, kind, n, nz, precision)
    if stop < 0:
        fv3.acoustic_substeps_batched([s2], [g2], 2 * dt, 2)
    else:
        fv3.acoustic_substeps(s2, g2, 2 * dt, 2, stop_stage=stop)
    torch.cuda.synchronize()
    N = n + 2 * H
    halo = np.ones((N, N), dtype=bool)
    halo[H:H + n, H:H + n] = False
    if kind == 1:   # corner blocks of the cube hold nothing
        for a in (slice(0, H), slice(H + n, N)):
            for b in (slice(0, H), slice(H + n, N)):
                halo[a, b] = False
    a, b = g2.download(s2.f["delz"], nz)[..., :N, :N][..., halo], g.download(ref, nz)[..., :N, :N][..., halo]
    assert np.all(b != 0.0)
    np.testing.assert_array_equal(a, b)
