"""Counter rows of the present kernels map to the launch names of the timing
hooks: every kernel symbol of the built library has a name, the marching
transports go by their kind (not their PPM order or number of fields), the
column solves by their site (not the length of their chunks), the remap by what
it remaps, and every name under which the sources time a launch is reached."""
import glob
import os
import re

import pytest

from paper_2205_04148_amd import pmc

PKG = os.path.dirname(os.path.abspath(pmc.__file__))


@pytest.fixture(scope="module")
def symbols():
    lib = os.path.join(PKG, "libfv3.so")
    if not os.path.exists(lib):
        pytest.skip("library not built")
    with open(lib, "rb") as f:
        found = {s.decode() for s in re.findall(rb"_ZN3fv3(?:12_GLOBAL__N_1)?\d+k_\w+", f.read())}
    return sorted(s for s in found if "k_multi" not in s and not re.match(r"_ZN3fv35k_one(?!ITnDa)", s))


def test_kinds_and_sites(symbols):
    seen = {}
    for s in symbols:
        seen.setdefault(pmc.launch_name(s), []).append(s)
    assert None not in seen
    for kind, name in enumerate(("k_march_mass", "k_march_wind", "k_march_height", "k_march_tracer")):
        assert seen[name], name
        for s in seen[name]:   # template: type, kind, fields, order
            assert re.search(rf"7k_marchI[fd]Li{kind}ELi[1-4]ELi[5-8]EE", s), s
    for site, name in enumerate(("k_column_c", "k_column_3")):
        bodies = {re.search(rf"(k_column|k_column_any)I[fd]Li{site}E", s).group(1) for s in seen[name]}
        assert bodies == {"k_column", "k_column_any"}, (name, bodies)
    for name in ("k_layer", "k_wgrad", "k_features", "k_remap_cells", "k_remap_winds", "k_remap_delp"):
        assert name in seen, name


def test_timed_names_are_reached(symbols):
    """Names given to the launch hooks in the sources (the corner halo runs the
    scalar halo's kernel; copies are told apart by their types)."""
    names = {pmc.launch_name(s) for s in symbols}
    timed = set()
    for path in glob.glob(os.path.join(PKG, "csrc", "*.hip")):
        with open(path) as f:
            text = f.read()
        timed |= set(re.findall(r"timed\(\"(k_\w+)\"", text))
        timed |= set(re.findall(r"launch_fn<[^;]*?>\(\s*\"(k_[\w<>]+)\"", text, re.S))
        timed |= set(re.findall(r"launch2d(?:_s)?\((k_\w+(?:<B>)?),", text))
    assert len(timed) > 20
    missing = timed - names - {"k_halo_corner"}
    if any(n.startswith("k_copy<") for n in names):
        missing.discard("k_copy")
    assert not missing, missing
