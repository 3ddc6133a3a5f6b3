"""The network at the edges of its tiles: widths that leave 16 of the 32
padded columns, single inputs and outputs, row counts around 32 and 64, after
a larger call that left non-finite activations behind; the row limit; column
features and the correction on rows and levels that fill no tile.  Bars of
test_gpu_mlp.py (2e-3 of the largest magnitude per array; 1e-6 and 1e-13 for
the element kernels)."""
import numpy as np
import pytest

import fv3_inputs as fi
from oracle import mlp as omlp
from test_gpu_mlp import _dev, _norm_arrays, _params, _rel, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(7, 16, 48, 5), (1, 32, 16, 1), (33, 80, 64, 32), (64, 64, 96, 70)])
@pytest.mark.parametrize("rows", [1, 31, 33, 64, 65, 257])
def test_sizes(fv3, sizes, rows):  # noqa: F811
    import torch

    ps = _params(11, sizes)
    rng = np.random.default_rng(rows)
    net = fv3.MLP(ps, maxrows=300)
    bad = _dev(np.full((300, sizes[0]), np.nan))
    net.gradients(bad, _dev(np.zeros((300, sizes[3]))))   # leaves NaN in every activation row
    X = rng.standard_normal((rows, sizes[0])).astype(np.float32)
    T = rng.standard_normal((rows, sizes[3])).astype(np.float32)
    P = [p.astype(np.float64) for p in ps]
    Y = torch.empty((rows, sizes[3]), dtype=torch.float32, device="cuda")
    net.forward(_dev(X), Y)
    torch.cuda.synchronize()
    want, _ = omlp.forward(P, X.astype(np.float64), bf=True)
    assert _rel(Y.cpu().numpy(), want) <= 2e-3
    got = net.gradients(_dev(X), _dev(T))
    loss, grads, _ = omlp.loss_grad(P, X.astype(np.float64), T.astype(np.float64), bf=True)
    for k, (g, w) in enumerate(zip(got, grads)):
        assert g.shape == w.shape and _rel(g, w) <= 2e-3, k
    assert abs(net.train_step(_dev(X), _dev(T), want_loss=True) - loss) <= 2e-3 * loss


def test_row_limit(fv3):  # noqa: F811
    """Up to the next multiple of 16 above maxrows, and no further."""
    net = fv3.MLP(_params(1, (4, 16, 16, 2)), maxrows=20)
    net.gradients(_dev(np.zeros((32, 4))), _dev(np.zeros((32, 2))))
    with pytest.raises(fv3.FV3Error):
        net.gradients(_dev(np.zeros((33, 4))), _dev(np.zeros((33, 2))))


@pytest.mark.parametrize("n,nz", [(9, 13), (11, 33)])
def test_element_tiles(fv3, n, nz):  # noqa: F811
    import torch

    init = fi.cube_state(n=n, nz=nz, seed=5, nq=0)
    g = fv3.Grid(1, n, nz)
    s = fv3.State.allocate(g)
    s.load(init)
    F = omlp.features(init, n)
    mean, std = _norm_arrays(F)
    # the normalisation the call is given, FP32 (a uniform delp has std 1e-6:
    # the rounding of its mean is what remains of it)
    mean32, inv32 = mean.astype(np.float32), (1.0 / std).astype(np.float32)
    X = torch.full(F.shape, float("nan"), dtype=torch.float32, device="cuda")
    fv3.column_features(s, g, _dev(mean32), _dev(inv32), X)
    torch.cuda.synchronize()
    Z = (F - mean32.astype(np.float64)) * inv32.astype(np.float64)
    assert np.abs(X.cpu().numpy() - Z).max() <= 1e-6 * max(1.0, np.abs(Z).max())
    rng = np.random.default_rng(n)
    Y = rng.standard_normal((6 * n * n, 3 * nz)).astype(np.float32)
    ym, ys = (rng.standard_normal(3 * nz).astype(np.float32) * 1e-4 for _ in range(2))
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    pt0 = s.get("pt")[..., 3:3 + n, 3:3 + n]
    fv3.apply_correction(s, g, _dev(Y), _dev(ym), _dev(ys), 600.0, flag)
    torch.cuda.synchronize()
    d = Y.astype(np.float64)[:, 2 * nz:] * ys[2 * nz:].astype(np.float64) + ym[2 * nz:].astype(np.float64)
    want = pt0 + 600.0 * d.reshape(6, n, n, nz).transpose(0, 3, 1, 2)
    assert np.abs(s.get("pt")[..., 3:3 + n, 3:3 + n] - want).max() <= 1e-13 * np.abs(want).max()
    assert int(flag.item()) == 0
