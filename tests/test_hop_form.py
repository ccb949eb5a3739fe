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


def choose(lib, prec, recon, full, lattices, nrhs, rare=0):
    flat = [v for L in lattices for v in L]
    out = (ctypes.c_int * 6)()
    form = lib.form_of(prec, recon, full, (ctypes.c_int * len(flat))(*flat), len(lattices), nrhs, rare, out)
    return form, dict(zip(("split", "halves", "tile", "lnt", "next", "built"), out))


@pytest.mark.parametrize("prec,recon", STORAGES)
def test_every_choice_is_built(lib, prec, recon):
    batches = [[L] for L in LATTICES] + [list(p) for p in itertools.combinations(LATTICES, 2)] + [[(16, 16, 16, 8)] * 8]
    for lattices, full, nrhs, rare in itertools.product(batches, (0, 1), range(1, 17), (0, 1)):
        form, h = choose(lib, prec, recon, full, lattices, nrhs, rare)
        case = (lattices, full, nrhs, rare, form, h)
        assert h["built"], case
        assert h["split"] in (0, 1, 2) and h["halves"] in (1, 2), case
        assert 1 <= h["tile"] <= 4 and h["tile"] * h["halves"] <= 4, case
        assert h["split"] == 0 or h["tile"] == 1, case
        assert h["lnt"] == (nrhs == 1 and not full), case


def test_every_kernel_is_chosen(lib):
    """Kernels that are built are run: one wave per chunk, a pair and a pair with
    right-hand sides next to each other, tiles with one wave and with two."""
    seen = set()
    for (prec, recon), L, full, nrhs in itertools.product(STORAGES, LATTICES + [(48, 48, 48, 24)], (0, 1), range(1, 17)):
        _, h = choose(lib, prec, recon, full, [L], nrhs)
        seen.add((prec, recon, h["split"], h["halves"], h["lnt"], h["next"]))
    every = {(p, r, 2, 1, *k) for p, r in STORAGES for k in ((0, 0), (1, 0), (0, 1))} - {(32, 18, 2, 1, 0, 1)}
    every |= {(p, r, 0, h, 0, 0) for p, r in STORAGES for h in (1, 2)} | {(64, 18, 1, 1, 1, 0)}
    assert seen == every, seen ^ every


def test_every_block_once(lib):
    """Blocks of every tile of right-hand sides, in either order of the tiles."""
    for slots, swizzle, adjacent in itertools.product((1, 2, 7, 8, 9, 64, 100), (0, 1), (0, 1)):
        for nrhs, tile in itertools.product((1, 2, 3, 4, 5, 7, 8, 13, 16, 37), (1, 2, 3, 4)):
            ntiles = -(-nrhs // tile)
            counts = (ctypes.c_int * (ntiles * slots))()
            case = (slots, swizzle, nrhs, tile, adjacent)
            assert lib.block_cover(slots, tile, adjacent, nrhs, swizzle, counts) == 0, case
            assert set(counts) == {1}, case


def test_launches_of_many_rhs(lib):
    """Up to 65535 right-hand sides: launches of fewer than 2^32 work-items, as few
    and as even as can be."""
    items = ctypes.c_longlong()
    for slots, tile, threads, nrhs in itertools.product((1, 288, 1152, 86016, 688128), (1, 2, 3, 4), (64, 128, 256),
                                                        (1, 16, 17, 4096, 60000, 65535)):
        n = lib.parts_of(slots, tile, threads, nrhs, ctypes.byref(items))
        case = (slots, tile, threads, nrhs, n)
        assert 1 <= n <= nrhs and items.value < 2**32, case
        parts = -(-nrhs // n)
        assert n - (nrhs - (parts - 1) * n) < parts, case
        if (slots + 7) * -(-nrhs // tile) * threads < 2**32:
            assert n == nrhs, case
        else:
            assert parts == 1 or (slots + 7) * (-(-nrhs // (parts - 1)) // tile) * threads >= 2**32 - (slots + 7) * threads, case


PAIR, TILE, NEXT = 2, 3, 5


@pytest.mark.parametrize("L,prec,recon,full,nrhs,rare,form", [
    # the right-hand sides of a chunk next to each other where tiles, or one right-hand side after the other, were slower
    ((24, 24, 24, 8), 64, 18, 0, 8, 0, NEXT), ((26, 26, 26, 8), 64, 12, 0, 12, 0, NEXT), ((10, 14, 18, 22), 64, 18, 1, 8, 0, NEXT),
    ((32, 32, 32, 8), 32, 12, 0, 3, 0, NEXT), ((36, 36, 36, 8), 32, 12, 0, 8, 0, NEXT), ((24, 24, 24, 16), 32, 12, 0, 12, 0, NEXT),
    # tiles stay where the links of one round fit the LDS, on large lattices of whole planes, and for reliable updates
    ((20, 20, 20, 8), 64, 18, 0, 3, 0, TILE), ((32, 32, 32, 8), 64, 18, 0, 12, 0, TILE), ((24, 24, 24, 8), 64, 18, 0, 8, 1, TILE),
    ((32, 32, 32, 8), 32, 12, 0, 12, 0, TILE), ((24, 24, 24, 8), 32, 12, 1, 8, 0, TILE), ((48, 48, 48, 24), 16, 12, 0, 2, 0, TILE),
    # and pairs one right-hand side after the other where all of them run at once
    ((8, 8, 8, 4), 64, 18, 0, 16, 0, PAIR), ((16, 16, 16, 8), 32, 12, 0, 4, 0, PAIR),
    ((12, 12, 12, 8), 64, 12, 1, 16, 0, PAIR), ((18, 18, 18, 8), 64, 12, 1, 6, 0, NEXT)])
def test_choices(lib, L, prec, recon, full, nrhs, rare, form):
    assert choose(lib, prec, recon, full, [L], nrhs, rare)[0] == form
