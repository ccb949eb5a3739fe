"""Conversions between canonical arrays and internal fields where a block's 64
sites per parity do not divide the lattice: the planes of the FP64 fields are
checked entry by entry, the other storages by the way back."""

import math

import numpy as np
import pytest

from lattice_inputs import gauge_field, gaussian_spinor

pytestmark = pytest.mark.gpu

LATTICES = [(2, 2, 2, 2), (4, 2, 6, 2), (10, 6, 4, 2), (8, 4, 4, 2), (130, 2, 2, 2), (6, 10, 6, 4)]


@pytest.fixture(scope="module")
def mods():
    import torch
    from paper_1411_5219_amd import fields, lqcd
    assert torch.cuda.is_available()
    return torch, fields, lqcd


def _sites(L4):
    """Canonical index of site h of each parity, x fastest."""
    X, Y, Z, T = L4
    i = np.arange(X * Y * Z * T)
    par = (i % X + i // X % Y + i // (X * Y) % Z + i // (X * Y * Z)) % 2
    return [i[par == p] for p in (0, 1)]


def _planes(raw, lat, npl):
    """(2, npl, Vh) complex128 of the two parity blocks of an FP64 field."""
    v = raw.cpu().numpy().view(np.complex128).reshape(2, npl, -1)
    return v[:, :, :lat.V // 2]


@pytest.mark.parametrize("L4", LATTICES)
@pytest.mark.parametrize("nrhs", [1, 3])
def test_spinors(mods, L4, nrhs):
    torch, fields, lqcd = mods
    lat = fields.Lattice(L4, (0.0, 0.0, 0.0, math.pi))
    psi = gaussian_spinor(L4, seed=71, nrhs=nrhs)
    src = psi if nrhs > 1 else psi[0]
    print(f"\n[case] pack spinors L={L4} nrhs={nrhs}", flush=True)
    dev = lat.spinor(src)
    got = dev.cpu().numpy().reshape(nrhs, -1)
    for k in range(nrhs):
        pl = _planes(torch.from_numpy(got[k].copy()), lat, 12)
        for p, idx in enumerate(_sites(L4)):
            assert np.array_equal(pl[p], psi[k].reshape(lat.V, 12)[idx].T), (k, p)
    # 2^-24 of an entry in FP32, 2^-11 of the site's largest in FP16
    for prec, tol in ((64, 0.0), (32, 2.0 ** -24), (16, 2.0 ** -11)):
        back = lat.unpack(lat.spinor(src, prec), prec, nrhs=nrhs).reshape(nrhs, lat.V, 12)
        ref = psi.reshape(nrhs, lat.V, 12)
        big = np.maximum(np.abs(ref.real), np.abs(ref.imag)).max(axis=2, keepdims=True)
        d = back - ref
        assert (np.maximum(np.abs(d.real), np.abs(d.imag)) <= tol * big).all(), prec


@pytest.mark.parametrize("L4", LATTICES)
def test_links_and_colour(mods, L4):
    torch, fields, lqcd = mods
    lat = fields.Lattice(L4, (0.0, 0.0, 0.0, math.pi))
    U = gauge_field(L4, "haar", seed=72)
    print(f"\n[case] pack links L={L4}", flush=True)
    for recon, npl in ((18, 9), (12, 6)):
        raw = lat.gauge(U, 64, recon).cpu().numpy().view(np.complex128).reshape(4, 2, npl, -1)[..., :lat.V // 2]
        for mu in range(4):
            for p, idx in enumerate(_sites(L4)):
                assert np.array_equal(raw[mu, p], np.asarray(U[mu]).reshape(lat.V, 9)[idx][:, :npl].T), (recon, mu, p)
    rng = np.random.default_rng(73)
    chi = rng.normal(size=(lat.V, 3)) + 1j * rng.normal(size=(lat.V, 3))
    assert np.array_equal(lat.unpack_colour(lat.colour(chi)).reshape(lat.V, 3), chi)
