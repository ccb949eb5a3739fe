"""The kernel a Wilson hop launch runs (csrc/hop_form.h, compiled here for the
host): whatever is chosen by size, for one launch or for the systems of a batch
together, is a kernel that is built, and its blocks cover every right-hand side."""

import ctypes
import itertools
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1411_5219_amd", "csrc")
STORAGES = [(64, 18), (64, 12), (32, 18), (32, 12), (16, 12)]
# below, at and above every wave count a form changes at; planes that fill their chunks and that do not
LATTICES = [(2, 2, 2, 2), (8, 8, 8, 4), (16, 16, 16, 8), (20, 20, 20, 8), (24, 24, 24, 6), (10, 14, 18, 22),
            (24, 24, 24, 48), (32, 32, 32, 6), (32, 32, 32, 8), (36, 36, 36, 8), (48, 48, 48, 12), (130, 2, 2, 2)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("forms") / "forms.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(HERE, "hop_form_harness.cpp"), "-o", so], check=True)
    return ctypes.CDLL(so)


def choose(lib, prec, recon, full, lattices, nrhs):
    flat = [v for L in lattices for v in L]
    out = (ctypes.c_int * 5)()
    form = lib.form_of(prec, recon, full, (ctypes.c_int * len(flat))(*flat), len(lattices), nrhs, out)
    return form, dict(zip(("split", "halves", "tile", "lnt", "built"), out))


@pytest.mark.parametrize("prec,recon", STORAGES)
def test_every_choice_is_built(lib, prec, recon):
    batches = [[L] for L in LATTICES] + [list(p) for p in itertools.combinations(LATTICES, 2)] + [[(16, 16, 16, 8)] * 8]
    for lattices, full, nrhs in itertools.product(batches, (0, 1), range(1, 17)):
        form, h = choose(lib, prec, recon, full, lattices, nrhs)
        case = (lattices, full, nrhs, form, h)
        assert h["built"], case
        assert h["split"] in (0, 1, 2) and h["halves"] in (1, 2), case
        assert 1 <= h["tile"] <= 4 and h["tile"] * h["halves"] <= 4, case
        assert h["split"] == 0 or h["tile"] == 1, case
        assert h["lnt"] == (nrhs == 1 and not full), case
