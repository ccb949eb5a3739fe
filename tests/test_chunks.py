"""The block order of the hop launches (csrc/chunks.h, compiled here for the
host): every plan visits every site of a parity exactly once, with the right
coordinates, within the partial slots a workspace holds; and the division by
launch constants is exact."""

import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1411_5219_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("chunks") / "chunks.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(HERE, "chunk_harness.cpp"), "-o", so], check=True)
    l = ctypes.CDLL(so)
    l.fast_divide.argtypes = [ctypes.c_uint, ctypes.c_uint]
    l.fast_divide.restype = ctypes.c_uint
    return l


# planes smaller than, equal to, a multiple of and just above a chunk; rows
# longer than a chunk; 2^4; wide flat lattices whose ragged planes would
# exceed the partial slots
LATTICES = [(2, 2, 2, 2), (4, 6, 8, 2), (16, 8, 4, 2), (32, 12, 4, 6), (10, 14, 6, 4), (24, 24, 6, 4), (44, 6, 2, 4),
            (130, 2, 4, 2), (258, 2, 2, 2), (256, 2, 2, 4), (6, 66, 4, 2)]


@pytest.mark.parametrize("L", LATTICES)
def test_every_site_once(lib, L):
    Vh = int(np.prod(L)) // 2
    # slots of the workspace's partials per parity: one per x-row or per 64 sites
    slots = max((Vh + 63) // 64, L[1] * L[2] * L[3])
    Li = (ctypes.c_int * 4)(*L)
    for order in (0, 1, 2, 3, 5, 64):
        for block in (64, 128, 192, 256):
            for ygroup in (1, 2, 3, 64):
                for maxsub, idle in ((1, 16), (1, 20), (1, 40), (block // 64, 20)):
                    for p in (0, 1):
                        counts = np.zeros(Vh, dtype=np.int32)
                        nsp = ctypes.c_int()
                        bad = lib.chunk_cover(Li, order, block, ygroup, maxsub, idle, p,
                                              counts.ctypes.data_as(ctypes.POINTER(ctypes.c_int)), ctypes.byref(nsp))
                        case = (order, block, ygroup, maxsub, idle, p)
                        assert bad == 0, case
                        assert (counts == 1).all(), case
                        assert nsp.value <= slots, case


def test_fast_division(lib):
    rng = random.Random(3)
    top = (1 << 31) - 1
    for d in [1, 2, 3, 5, 7, 63, 64, 65, 127, 641, 65535, 65536, 65537, top - 1, top] + \
            [rng.randrange(1, 1 << rng.randrange(1, 32)) for _ in range(300)]:
        for n in [0, 1, d - 1, d, min(top, d + 1), top // d * d, max(0, top // d * d - 1), top] + \
                [rng.randrange(0, top + 1) for _ in range(50)]:
            assert lib.fast_divide(d, n) == n // d, (d, n)
