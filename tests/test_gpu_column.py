"""Column solves in chunks of layers: depths at the edges of a chunk (5
layers), of the short-chunk kernel (160 layers) and beyond, column counts that
leave a partial block, terrain, and an ensemble of members on both sides of the depth limit.

Bars against the oracle, as for the single stages at small depth (1e-13;
w 3e-11): an error of the equation of state moves w by the inverse of the
layer mass, so w's bar grows with the number of layers over the 6 it was
derived for; the interface sums add one rounding per layer, so the other
fields' bar grows the same way."""
import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_parity import W_BAR, _compare, _pair, fv3  # noqa: F401

pytestmark = pytest.mark.gpu
H = 3


@pytest.mark.parametrize("kind,n,nz", [(0, 9, 1), (0, 9, 2), (0, 9, 5), (0, 17, 6), (1, 8, 11), (0, 9, 80),
                                       (1, 8, 81), (0, 9, 160), (0, 9, 161), (1, 8, 163)])
def test_depths(fv3, orc, kind, n, nz):  # noqa: F811
    init = fi.periodic_state(n=n, nz=nz) if kind == 0 else fi.cube_state(n=n, nz=nz)
    g, s, og, os_ = _pair(fv3, orc, kind, n, nz, init)
    dt = 0.4 if kind == 0 else 300.0
    grow = max(1.0, nz / 6.0)
    fv3.acoustic_substeps(s, g, dt, 1, stop_stage=8)
    orc.acoustic_substeps(og, os_, dt, 1, stop_stage=8)
    tol = {k: 1e-13 * grow for k in ("delp", "pt", "delz", "pfull", "phi", "uc", "vc")}
    tol["w"] = W_BAR * grow
    _compare(s, os_, n, tuple(tol), tol, f"depth kind{kind} n{n} nz{nz}")


@pytest.mark.parametrize("kind,n,nz", [(0, 10, 7), (1, 12, 9)])
def test_terrain(fv3, orc, kind, n, nz):  # noqa: F811
    """Surface heights with the neighbour tiles' values in the halo."""
    init = fi.periodic_state(n=n, nz=nz) if kind == 0 else fi.cube_state(n=n, nz=nz)
    rng = np.random.default_rng(3)
    phis = 9.80665 * 200.0 * rng.random(init["phis"].shape)[:, None]
    orc.halo_fill(orc.Grid(kind, n, 1), phis, "C")
    init["phis"] = np.ascontiguousarray(phis[:, 0])
    g, s, og, os_ = _pair(fv3, orc, kind, n, nz, init)
    dt = 0.2 if kind == 0 else 60.0
    fv3.acoustic_substeps(s, g, 2 * dt, 2, stop_stage=8)
    orc.acoustic_substeps(og, os_, 2 * dt, 2, stop_stage=8)
    tol = {k: 1e-11 for k in ("delp", "pt", "delz", "pfull", "phi", "uc", "vc", "w")}
    _compare(s, os_, n, tuple(tol), tol, f"terrain kind{kind}")


def test_ensemble_across_the_depth_limit(fv3):  # noqa: F811
    """Members of 12 and 170 layers in one ensemble compute what they compute
    alone, bit for bit."""
    import torch

    dims = [(16, 12), (9, 170)]

    def make():
        gs = [fv3.Grid(0, n, nz) for n, nz in dims]
        ss = []
        for g, (n, nz) in zip(gs, dims):
            ss.append(fv3.State.allocate(g))
            ss[-1].load(fi.periodic_state(n=n, nz=nz, seed=n))
        return gs, ss

    ga, sa = make()
    fv3.acoustic_substeps_batched(sa, ga, 0.4, 2)
    gb, sb = make()
    for g, s in zip(gb, sb):
        fv3.acoustic_substeps(s, g, 0.4, 2)
    torch.cuda.synchronize()
    for a, b, (n, _) in zip(sa, sb, dims):
        for k in ("u", "v", "w", "delp", "pt", "delz"):
            sl = (Ellipsis, slice(H, H + n), slice(H, H + n))
            np.testing.assert_array_equal(a.get(k)[sl], b.get(k)[sl])
