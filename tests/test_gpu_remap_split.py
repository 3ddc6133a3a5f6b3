"""Remap: every split of a block between columns and chunks of layers (256
columns and one chunk to 16 and 16), at the layer counts where it changes (5,
10, 20, 40 layers a chunk count), one column more than a block holds, and grids
of fewer blocks than the split asks for.  Bars of the remap parity tests."""
import pytest

from test_gpu_remap import _bars, _run_pair, fv3  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,nz,precision,coef", [
    (0, 182, 5, "fp64", "sigma"), (0, 183, 5, "mixed", "sigma"), (0, 129, 6, "fp64", "sigma"), (0, 130, 10, "fp64", "hybrid"),
    (0, 129, 11, "mixed", "hybrid"), (0, 91, 20, "fp64", "hybrid"), (0, 65, 21, "mixed", "hybrid"), (1, 27, 40, "fp64", "hybrid"),
    (0, 47, 41, "fp64", "hybrid"), (1, 10, 80, "mixed", "hybrid"), (1, 20, 81, "fp64", "sigma"), (0, 8, 5, "fp64", "sigma"),
    (0, 50, 9, "mixed", "hybrid")])
def test_splits(fv3, orc, kind, n, nz, precision, coef):  # noqa: F811
    errs, *_ = _run_pair(fv3, orc, kind, n, nz, precision, coef=coef)
    bar = _bars(precision)
    for k, e in errs.items():
        assert e <= bar(k), (k, e)
