"""The decode step's division of work, replayed on the CPU: every unit that a sequence needs is taken exactly once, by
one wavefront or one workgroup, whatever is in the batch."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "decode_units_check.cpp")
HDR = os.path.join(HERE, "..", "paper_2603_17484_amd", "csrc", "decode_units.hpp")
LIB = os.path.join(HERE, "libdecode_units_check.so")


@pytest.fixture(scope="module")
def chk():
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(map(os.path.getmtime, (SRC, HDR))):
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", LIB, SRC])
    L = ctypes.CDLL(LIB)
    L.units_check.argtypes = [ctypes.c_int] * 3 + [ctypes.c_void_p] * 3 + [ctypes.c_int, ctypes.c_void_p, ctypes.c_char_p, ctypes.c_int]
    return L


def replay(chk, pos, W, T, heads, routed, do_local=1, ring=0):
    t = np.minimum(np.maximum(np.asarray(pos, dtype=np.int32), 0), T - 1).astype(np.int32)
    win = np.zeros_like(t) if ring else np.maximum(t - W, 0).astype(np.int32)
    routed = np.ascontiguousarray(routed, dtype=np.int32)
    nunits = (T + 511) // 512 + (1 if do_local and not ring else 0)
    wgs = min(512, 8 * len(t) * heads * ((nunits + 7) // 8)) // 8      # the host's grid
    alone, msg = ctypes.c_int(), ctypes.create_string_buffer(300)
    rc = chk.units_check(len(t), heads, do_local, t.ctypes.data, win.ctypes.data, routed.ctypes.data, wgs, ctypes.byref(alone), msg, 300)
    assert rc == 0, msg.value.decode()
    return alone.value


@pytest.mark.parametrize("heads", [1, 3, 8, 40])
@pytest.mark.parametrize("W", [0, 31, 511, 512, 513, 4096])
@pytest.mark.parametrize("T", [1, 512, 513, 5000])
def test_every_unit_once(chk, T, W, heads):
    rng = np.random.default_rng(T + W + heads)
    for B in (1, 2, 9, 65):
        pos = rng.integers(0, T, B)
        pos[0] = T - 1
        for do_local in (0, 1):
            replay(chk, pos, W, T, heads, rng.integers(0, heads + 1, B), do_local)
            replay(chk, pos, W, T, heads, np.full(B, heads), do_local)
        replay(chk, pos, W, T, heads, np.zeros(B))
        replay(chk, pos + 3 * T, W, T, heads, np.zeros(B), ring=1)


def test_both_walks_are_used(chk):
    """Sizes on both sides of the rule: none, some and all of the units by single wavefronts."""
    T = 131072
    assert replay(chk, [T - 1], 4096, T, 4, [0]) == 0
    pos = [T - 1 - 977 * i for i in range(8)]
    some = replay(chk, pos, 4096, T, 4, [4, 0, 0, 0, 4, 0, 0, 0])
    assert some == 2048                                   # one round of 8 x 256 wavefronts, the rest by workgroups
    every = 4 * sum(p // 512 + 1 + (p >= 4096 and (p - 4096) % 512 != 0) for p in pos)
    assert replay(chk, pos, 4096, T, 4, [4] * 8) == every  # the fourth round is nearly full
