"""The network's parameter transfers on the device the network lives on: with
another HIP device current, fv3_mlp_get_params and fv3_mlp_set_params launch on
the network's device and leave the caller's device current, and a launch that
fails is reported instead of returning what an earlier call left behind.  Runs
without a GPU: a small library stands in for the HIP calls and records the
device that is current at each launch."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2205_04148_amd", "libfv3.so")
FAKE = r"""
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
int current = 0, launches = 0, launch_error = 0, seen[64];
int hipGetDevice(int *d) { *d = current; return 0; }
int hipSetDevice(int d) { current = d; return 0; }
int hipMalloc(void **p, size_t n) { *p = malloc(n ? n : 1); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipGetLastError(void) { return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t l, void *s)
{
    (void)f; (void)g; (void)b; (void)a; (void)l; (void)s;
    if (launches < 64) seen[launches] = current;
    launches++;
    return launch_error;
}
"""
SCRIPT = textwrap.dedent("""
    import ctypes as C, sys
    fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
    lib = C.CDLL(sys.argv[2])
    current, launches, error = (C.c_int.in_dll(fake, k) for k in ("current", "launches", "launch_error"))
    seen = (C.c_int * 64).in_dll(fake, "seen")
    count = 5 * 16 + 16 + 16 * 16 + 16 + 16 * 3 + 3
    p = (C.c_float * count)(*range(count))
    net = C.c_void_p()
    assert lib.fv3_mlp_create(5, 16, 16, 3, 20, p, C.byref(net)) == 0
    assert launches.value >= 1 and all(seen[q] == 0 for q in range(launches.value))
    for call in (lib.fv3_mlp_get_params, lib.fv3_mlp_set_params):
        current.value, launches.value = 1, 0
        assert call(net, p) == 0
        assert launches.value >= 1, "no launch seen"
        assert all(seen[q] == 0 for q in range(launches.value)), "launched on another device than the network's"
        assert current.value == 1, "the caller's device was not restored"
        error.value = 1
        assert call(net, p) == -4, "a failed launch was not reported"
        error.value = 0
        assert current.value == 1
    assert lib.fv3_mlp_free(net) == 0
    print("ok")
""")


def test_parameters_with_another_device_current(tmp_path):
    gcc = shutil.which("gcc")
    if gcc is None or not os.path.exists(LIB):
        pytest.skip("gcc or the built library not available")
    src, so = tmp_path / "fake.c", tmp_path / "fake.so"
    src.write_text(FAKE)
    subprocess.run([gcc, "-shared", "-fPIC", "-O1", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", SCRIPT, str(so), LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr
