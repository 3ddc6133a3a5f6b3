"""Members of an ensemble share the options of the column solves: a member that
differs from the first in off-centring, interface order or humidity is refused
with FV3_EUNSUPPORTED, whichever combination the others have; members that
agree are accepted."""
import itertools

import numpy as np
import pytest

import fv3_inputs as fi
from test_gpu_parity import fv3  # noqa: F401

pytestmark = pytest.mark.gpu
CASES = [(beta, ppo, moist) for beta in (1.0, 0.75) for ppo in (2, 4) for moist in (False, True)]


@pytest.mark.parametrize("nz", [4, 165])
def test_column_options_shared(fv3, nz):  # noqa: F811
    n = 8
    init = fi.periodic_state(n=n, nz=nz)
    made = []
    for beta, ppo, moist in CASES:
        pair = []
        for _ in range(2):
            g = fv3.Grid(0, n, nz, beta=beta, pp_order=ppo)
            s = fv3.State.allocate(g)
            s.load(dict(init, qv=np.full_like(init["pt"], 0.01)) if moist else init)
            pair.append((g, s))
        made.append(pair)
    for (a, pa), (b, pb) in itertools.product(zip(CASES, made), repeat=2):
        (ga, sa), (gb, sb) = pa[0], pb[1]
        try:
            fv3.acoustic_substeps_batched([sa, sb], [ga, gb], 0.1, 1)
            got = 0
        except fv3.FV3Error as e:
            got = e.status
        assert got == (0 if a == b else -8), (a, b, got)
