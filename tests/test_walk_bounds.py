"""walk::list_bounds (csrc/dkdv_walk.hpp, compiled for the host): which rows of a list set the dK/dV walk gives to a key block
when rows see only the keys 0 .. pos - shift, against the definition over (row, key) pairs."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HDR = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2603_17484_amd", "csrc", "dkdv_walk.hpp")
SRC = """
#include "%s"
extern "C" void bounds(int k0, int shift, int nkb, int* out) {
    const l2a::walk::ListBounds b = l2a::walk::list_bounds(k0, shift, nkb);
    out[0] = b.lo, out[1] = b.hi;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("bounds")
    (d / "b.cpp").write_text(SRC % HDR)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", str(d / "b.so"), str(d / "b.cpp")])
    return ctypes.CDLL(str(d / "b.so"))


@pytest.mark.parametrize("T,shift,f", [(1, 0, 1.0), (300, 0, 0.4), (300, 1, 0.4), (300, 64, 1.0), (321, 65, 0.2), (700, 128, 0.1),
                                       (1001, 299, 0.5), (1001, 1000, 1.0), (640, 639, 1.0)])
def test_bounds(lib, T, shift, f):
    rng = np.random.default_rng(T + shift)
    pos = np.flatnonzero(rng.random(T) < f)
    nkb = (T + 63) // 64
    first = np.array([(pos < 64 * k).sum() for k in range(nkb + 1)])
    out = (ctypes.c_int * 2)()
    for k0 in range(0, T, 128):
        lib.bounds(k0, shift, nkb, out)
        lo, hi = out
        assert 0 <= lo <= hi <= nkb
        rows = np.arange(len(pos))
        assert not (pos[rows < first[lo]] - shift >= k0).any()            # rows left out see no key of the block
        last = k0 + 127                                                   # rows from entry hi on see the whole block ...
        if last < T:                                                      # (a block past the end is masked everywhere)
            assert (pos[rows >= first[hi]] - shift >= last).all()
        if shift == 0:
            assert first[lo] == (pos < k0).sum()
