"""CPU: the cut of a batched field's planes into units and slabs (csrc/cut.hpp, the functions that
the host and the kernels share), compiled here with overflow checks: on every lattice that the entry
points accept, the units follow one another from 0 to nx, each of 1 to 16 planes, and the slabs hold
whole units, at most sixteen, and no more planes than asked for."""
import ctypes
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2604_25876_amd" / "csrc"

DRIVER = """
#include "cut.hpp"
using namespace skyr;
extern "C" {
int u_start(int k, int nx, int units) { return unit_start(k, nx, units, 0); }
int u_start_len(int k, int nx, int units, int len) { return unit_start(k, nx, units, len); }
int u_default(int nx) { return default_units(nx, 16); }
int u_slab(int nx, int units, int cap) { return slab_units(nx, units, cap); }
int u_planes(int slab, int per, int nx, int units) { return slab_planes(slab, per, nx, units, 0); }
}
"""


@pytest.fixture(scope="module")
def cut(tmp_path_factory):
    d = tmp_path_factory.mktemp("cut")
    (d / "cut.cpp").write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-ftrapv", "-fPIC", "-shared", "-I", str(CSRC),
                           "-o", str(d / "libcut.so"), str(d / "cut.cpp")])
    return ctypes.CDLL(str(d / "libcut.so"))


# the smallest; around the units' lengths; below and above 185,352 planes, from where the last unit's
# number times the planes passes 2^31; the longest lattice of 5 x 5 rows that is accepted
@pytest.mark.parametrize("nx", list(range(1, 70)) + [124, 127, 252, 256, 257, 1000, 65535, 65536, 185351, 185352, 185400,
                                                     200000, 1342173, 2 ** 29 // 25 - 4])
def test_units_and_slabs(cut, nx):
    units = cut.u_default(nx)
    ks = range(units + 1) if units < 30000 else [k for c in (0, units // 2, units) for k in range(c - 300, c + 301)
                                                if 0 <= k <= units]
    starts = {k: cut.u_start(k, nx, units) for k in ks}
    assert starts[0] == 0 and starts[units] == nx
    for k in ks:
        assert starts[k] == k * nx // units
        if k + 1 in starts:
            assert 1 <= starts[k + 1] - starts[k] <= 16
    for cap in range(16, 257, 16):
        per = cut.u_slab(nx, units, cap)
        slabs = -(-units // per)
        assert 1 <= per <= 16 and (slabs - 1) * per < units
        for s in {0, 1, slabs // 2, slabs - 1} & set(range(slabs)):
            first, end = s * per, min(units, (s + 1) * per)
            planes = cut.u_planes(s, per, nx, units)
            assert planes == end * nx // units - first * nx // units
            assert 1 <= planes <= max(cap, 16)


# a tile that was set: slabs of the length that was set, the last one of what is left
@pytest.mark.parametrize("nx", [1, 15, 16, 17, 124, 200000, 2 ** 29 // 25 - 4])
@pytest.mark.parametrize("length", [16, 100, 1000, 2 ** 31 - 1])
def test_units_of_a_set_length(cut, nx, length):
    units = -(-nx // length)
    for k in {0, 1, units // 2, units - 1, units} & set(range(units + 1)):
        assert cut.u_start_len(k, nx, units, length) == min(nx, k * length)
