"""Mass sums over many blocks: counts of block partials at the edges of the
batches they are combined in (256: one batch exactly, one more, many), with
values of both signs spread over ten decades, against exact rational sums (bar
4 eps of the sum of magnitudes); and the allocation-free call gives the same
bits."""
import math

import numpy as np
import pytest

from test_gpu_parity import H, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,precision", [(0, 8, "fp64"), (0, 256, "fp64"), (0, 260, "mixed"), (0, 1030, "fp64"),
                                              (1, 130, "mixed"), (1, 257, "fp64")])
def test_many_partials(fv3, kind, n, precision):  # noqa: F811
    import torch

    g = fv3.Grid(kind, n, 1, precision=precision)
    gen = torch.Generator("cuda").manual_seed(n)
    f = []
    for q in range(3):
        b = g.new_field(1)
        x = torch.randn(g.view(b, 1).shape, generator=gen, device="cuda", dtype=torch.float64)
        x *= 10.0 ** (10.0 * torch.rand(x.shape, generator=gen, device="cuda", dtype=torch.float64) - 5.0)
        g.view(b, 1).copy_(x)
        f.append(b)
    got = fv3.mass_sums(g, f[0], f[1], [f[2]])
    dev = torch.zeros(3, dtype=torch.float64, device="cuda")
    fv3.mass_sums_noalloc(g, f[0], f[1], [f[2]], dev)
    assert np.array_equal(got, dev.cpu().numpy())
    sl = (Ellipsis, slice(H, H + n), slice(H, H + n))
    m = g.download(f[0], 1)[sl] * g.metric("area")[sl][:, None]
    for k, q in enumerate([None, f[1], f[2]]):
        x = m if q is None else g.download(q, 1)[sl] * m
        ref, mag = math.fsum(x.ravel()), math.fsum(np.abs(x).ravel())
        print(k, abs(got[k] - ref) / mag, flush=True)
        assert abs(got[k] - ref) <= 4 * np.finfo(float).eps * mag, (k, got[k], ref)
