"""The dK/dV kernel's launch order by heads and its downward Local walk, replayed on the CPU (the companion of
test_dkdv_walk.py, same header, same brute force)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from tests.test_dkdv_walk import DENSE, HDR, LIST, LOCAL, SRC as WALK_SRC, routed_positions

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "dkdv_heads_check.cpp")
LIB = os.path.join(HERE, "libdkdv_heads_check.so")


@pytest.fixture(scope="module")
def chk():
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(map(os.path.getmtime, (SRC, WALK_SRC, HDR))):
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", LIB, SRC])
    L = ctypes.CDLL(LIB)
    L.heads_launch.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_void_p]
    L.heads_jobs_check.argtypes = [ctypes.c_int] * 4 + [ctypes.c_char_p, ctypes.c_int]
    L.heads_walk_check.argtypes = [ctypes.c_int] * 6 + [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_void_p,
                                                        ctypes.c_char_p, ctypes.c_int]
    return L


def launch(chk, T, bh, W):
    out = np.zeros(5, dtype=np.int32)
    chk.heads_launch(T, bh, W, out.ctypes.data)
    return dict(zip(("nblk", "groups", "chunk", "nsplit", "jobs"), (int(x) for x in out)))


@pytest.mark.parametrize("T,bh,W,groups,nsplit", [
    (131072, 4, 4096, 0, 1), (32768, 4, 4096, 0, 1), (65536, 8, 4096, 0, 1),      # long: chunks of key blocks
    (16384, 8, 4096, 8, 1), (16384, 4, 4096, 4, 1), (16384, 4, 8192, 4, 2),       # T <= 2 W: split
    (8192, 8, 4096, 8, 2), (8192, 4, 1024, 4, 2), (4096, 8, 1024, 8, 1), (24576, 4, 4096, 0, 1), (4096, 4, 4096, 4, 4), (1, 1, 0, 1, 8), (300, 3000, 64, 0, 1)])
def test_what_the_host_launches(chk, T, bh, W, groups, nsplit):
    l = launch(chk, T, bh, min(W, T))
    assert (l["groups"], l["nsplit"]) == (groups, nsplit)
    assert l["chunk"] >= 1 and (groups == 0 or l["jobs"] >= l["nblk"] * bh * nsplit)


@pytest.mark.parametrize("nbh", [1, 2, 3, 4, 6, 8, 12, 24, 30])
@pytest.mark.parametrize("nblk", [1, 2, 7, 8, 33, 128])
@pytest.mark.parametrize("nsplit", [1, 2, 8])
def test_every_job_once(chk, nbh, nblk, nsplit):
    groups = {0: 8, 4: 4, 2: 2, 6: 2}.get(nbh % 8, 1)
    msg = ctypes.create_string_buffer(512)
    assert chk.heads_jobs_check(nblk, nbh, groups, nsplit, msg, 512) == 0, msg.value.decode()


@pytest.mark.parametrize("T", [1, 127, 129, 640, 1000])
@pytest.mark.parametrize("G", [1, 7])
@pytest.mark.parametrize("W", [0, 100, 128, 600, 1000])
def test_walks(chk, T, G, W):
    pos = routed_positions(T, G, 0.3, True, T + G + W)
    downs = 0
    for chunk in (1, 3, 64):
        for nsplit in (1, 2, 4):
            for kinds in ([LOCAL, LIST], [LOCAL], [LIST], [LOCAL, DENSE]):
                msg, n = ctypes.create_string_buffer(512), ctypes.c_int()
                k = np.asarray(kinds, dtype=np.int32)
                rc = chk.heads_walk_check(T, G, W, chunk, nsplit, len(kinds), k.ctypes.data, pos.ctypes.data, len(pos),
                                          ctypes.byref(n), msg, 512)
                assert rc == 0, f"chunk={chunk} nsplit={nsplit} sets={kinds}: {msg.value.decode()}"
                downs += n.value
    assert downs > 0 or T > W + 128
