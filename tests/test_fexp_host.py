"""The column solves' FP64 exponential (csrc/flog.hpp), compiled for the host
with hipcc and run on the CPU: within one ulp of the host library's exp over
the arguments of the equation of state and the whole normal range, +inf on
overflow, 0 for -inf, NaN for NaN."""
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2205_04148_amd", "csrc")
DRIVER = r"""
#include "flog.hpp"
#include <cstdio>
#include <cstdlib>
int main()
{
    char buf[64];
    while (std::scanf("%63s", buf) == 1) std::printf("%a\n", fv3::fexp(std::strtod(buf, nullptr)));
    return 0;
}
"""


@pytest.fixture(scope="module")
def fexp(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("fexp")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    subprocess.run([hipcc, "-O2", "-x", "hip", "--offload-arch=gfx950", "-I", CSRC, "-o", str(exe), str(src)],
                   check=True, capture_output=True)

    def run(xs):
        out = subprocess.run([str(exe)], input="\n".join(float(x).hex() for x in xs), capture_output=True,
                             text=True, check=True).stdout.split()
        return np.array([float.fromhex(o) for o in out])

    return run


def test_within_one_ulp(fexp):
    rng = np.random.default_rng(8)
    xs = np.concatenate([rng.uniform(-12.0, 12.0, 60000), rng.uniform(-700.0, 700.0, 20000),
                         rng.uniform(-1e-3, 1e-3, 10000), 0.5 * math.log(2.0) * np.arange(-40, 41), [0.0, -0.0]])
    got, ref = fexp(xs), np.exp(xs)
    err = np.abs(got - ref) / np.spacing(ref)
    print("max ulp", err.max(), "share off by one ulp", (err > 0.5).mean())
    assert err.max() <= 1.0, xs[err.argmax()]
    assert got[-1] == 1.0 and got[-2] == 1.0


def test_special_arguments(fexp):
    got = fexp([1000.0, math.inf, -math.inf, -1e5, math.nan])
    assert got[0] == math.inf and got[1] == math.inf and got[2] == 0.0 and got[3] == 0.0 and math.isnan(got[4])
