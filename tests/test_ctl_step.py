"""The scalar steps of a CG iteration as its kernels run them (ctl_step: a
step late, together with the next one) against the same steps one by one, and
the flag by which x takes alpha p exactly once per iteration."""

import ctypes
import os
import random
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.join(HERE, "..")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("ctl_step") / "step.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1411_5219_amd", "csrc"),
                    os.path.join(HERE, "ctl_step_harness.cpp"), "-o", so], check=True)
    l = ctypes.CDLL(so)
    d = ctypes.c_double
    l.compare.argtypes = [ctypes.POINTER(d), ctypes.c_int, d, d, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                          ctypes.POINTER(ctypes.c_int)]
    l.family.argtypes = [ctypes.POINTER(d), ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.POINTER(d),
                         ctypes.POINTER(ctypes.c_int)]
    return l


def _totals(rng, n, bad):
    """||w||^2, ||r||^2, the update's ||r||^2 and ||z||^2 of a falling residual, with a fault somewhere."""
    t, rr = [], 1.0
    for _ in range(n):
        rr *= 10 ** rng.uniform(-0.9, 0.2)
        t += [rng.uniform(0.5, 2.0), rr, rr * rng.uniform(0.9, 1.5), rng.uniform(0.5, 2.0)]
    if bad is not None:
        t[rng.randrange(len(t))] = bad
    return t


@pytest.mark.parametrize("bad", [None, 0.0, float("nan"), float("inf")])
@pytest.mark.parametrize("delta,tol_inner,window,max_stag", [(0.0, 0.0, 0, 0), (0.1, 0.0, 0, 0), (0.05, 0.1, 3, 2),
                                                             (1e-4, 0.0, 2, 1)])
def test_steps_late_are_the_steps(lib, delta, tol_inner, window, max_stag, bad):
    for seed in range(60):
        rng = random.Random(seed)
        n = 14
        tot = _totals(rng, n, bad)
        log = (ctypes.c_int * n)()
        limit = rng.choice([5, 1000])
        k = lib.compare((ctypes.c_double * len(tot))(*tot), n, delta, tol_inner, limit, window, max_stag, log)
        assert k == 0, (seed, k)
        done, ups = 0, 0
        for i in range(n):
            xdo, d, u = log[i] & 1, (log[i] >> 1) & 1, log[i] >> 2
            # x takes alpha p unless the solve had ended before, ended at alpha, or an update took it
            ended_at_alpha = d and not done and (tot[4 * i] == 0.0 or tot[4 * i] != tot[4 * i] or tot[4 * i] == float("inf"))
            assert xdo == (0 if done or ended_at_alpha or u > ups else 1), (seed, i)
            done, ups = d, u


@pytest.mark.parametrize("base", [0, 2])
def test_family(lib, base):
    n, iters = 4, 12
    sigma = [0.0, 0.3, 1.0, 4.0]
    sigma[0], sigma[base] = sigma[base], sigma[0]
    tot = []
    rr = 1.0
    for _ in range(iters):
        rr *= 0.25
        tot += [2.0 * rr, rr]
    log = (ctypes.c_int * (n * iters))()
    lib.family((ctypes.c_double * len(tot))(*tot), n, base, iters, (ctypes.c_double * n)(*sigma), log)
    for i in range(n):
        done = 0
        for k in range(iters):
            assert log[k * n + i] & 1 == 1 - done, (i, k)
            done = log[k * n + i] >> 1
        assert done
