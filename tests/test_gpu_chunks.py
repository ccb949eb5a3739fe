"""The hop kernels at the edges of their blocks: planes smaller than a chunk of
64 sites, ragged last chunks, x-rows longer than a chunk, a wide flat lattice
that runs in memory order, and right-hand sides that fill, split and leave
part of a block."""

import math

import pytest

from gpu_util import site_rel_err
from lattice_inputs import gauge_field, gaussian_spinor
from oracle import staggered as S
from oracle import wilson as W

pytestmark = pytest.mark.gpu

# the bounds of test_gpu_dslash.py: FP64 rounding of about 1000 operations per
# site; FP32 the same at 6e-8; FP16 storage 2^-11 of a site's largest value
TOL = {64: 1e-13, 32: 1e-5, 16: 1e-2}
LATTICES = [(10, 6, 4, 2), (24, 24, 2, 2), (44, 6, 2, 4), (130, 2, 2, 2), (258, 2, 2, 2)]


@pytest.fixture(scope="module")
def mods():
    import torch
    from paper_1411_5219_amd import fields, lqcd
    assert torch.cuda.is_available()
    return torch, fields, lqcd


@pytest.mark.parametrize("L4", LATTICES)
@pytest.mark.parametrize("prec,recon", [(64, 18), (64, 12), (32, 12), (16, 12)])
@pytest.mark.parametrize("nrhs", [1, 2, 5, 8])
def test_block_edges(mods, L4, prec, recon, nrhs):
    torch, fields, lqcd = mods
    theta, kappa, mu = (0.2, 0.0, -0.4, math.pi), 0.14, 0.03
    print(f"\n[case] block edges L={L4} prec={prec}/{recon} nrhs={nrhs}", flush=True)
    U = gauge_field(L4, "exp", eps=0.4, seed=41)
    psi = gaussian_spinor(L4, seed=42, nrhs=nrhs)
    lat = fields.Lattice(L4, theta)
    o = lqcd.op(kappa, mu, prec, recon)
    Ud = lat.gauge(U, prec, recon)
    src = psi if nrhs > 1 else psi[0]
    full = lat.spinor(src, prec)
    out = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec, nrhs=nrhs)
    lqcd.dslash_apply(lat.g, o, Ud, full, out, dagger=1, nrhs=nrhs)
    got = lat.unpack(out, prec, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    sch = lat.zeros(lqcd.FIELD_SPINOR_PARITY, prec, nrhs=nrhs)
    lqcd.dslash_eo_apply(lat.g, o, Ud, lat.parity_view(full, 0, prec, nrhs), sch, 0, lqcd.OP_SCHUR, 0, nrhs,
                         lat.workspace(o))
    pb = lat.nbytes(lqcd.FIELD_SPINOR_PARITY, prec)
    f = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec, nrhs=nrhs)
    f.view(nrhs, 2, pb)[:, 0, :] = sch.view(nrhs, pb)
    even = lat.unpack(f, prec, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    ev = W.parity(L4) == 0
    for k in range(nrhs):
        ref = W.apply_M(U, psi[k], L4, theta, kappa, mu, dagger=True)
        assert site_rel_err(got[k], ref) <= TOL[prec], ("full", k)
        ref = W.schur(U, W.mask(psi[k], L4, 0), L4, theta, kappa, mu)
        assert site_rel_err(even[k][ev], ref[ev]) <= TOL[prec], ("schur", k)


@pytest.mark.parametrize("L4", LATTICES)
@pytest.mark.parametrize("order", [0, 1])
def test_solves_at_block_edges(mods, L4, order):
    """The reductions: a solve on one and on three right-hand sides certified
    by the oracle, blocks in memory order and in planes."""
    torch, fields, lqcd = mods
    theta, kappa, mu = (0.2, 0.0, -0.4, math.pi), 0.13, 0.03
    print(f"\n[case] solves at block edges L={L4} order={order}", flush=True)
    U = gauge_field(L4, "exp", eps=0.4, seed=43)
    lat = fields.Lattice(L4, theta)
    o = lqcd.op(kappa, mu)
    Ud = lat.gauge(U)
    families = [(k, p) for k in (lqcd.KERNEL_DSLASH, lqcd.KERNEL_DSLASH_RHS) for p in (64, 32)]
    saved = {f: lqcd.lqcd_get_launch(*f) for f in families}
    try:
        for f in families:
            lqcd.lqcd_set_launch(*f, **dict(saved[f], order=order))
        for nrhs in (1, 3):
            b = gaussian_spinor(L4, seed=44, nrhs=nrhs)
            bd = lat.spinor(b if nrhs > 1 else b[0])
            x = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs)
            p = lqcd.solve_params(tol=1e-10, inner_prec=32, inner_recon=12, nrhs=nrhs)
            rc, info = lqcd.cg_solve(lat.g, o, Ud, bd, x, p, lat.workspace(o, p))
            assert rc == 0, info
            got = lat.unpack(x, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
            for k in range(nrhs):
                assert W.true_residual(U, got[k], b[k], L4, theta, kappa, mu) <= 1e-10, (nrhs, k)
    finally:
        for f in families:
            lqcd.lqcd_set_launch(*f, **saved[f])


@pytest.mark.parametrize("L4", LATTICES)
@pytest.mark.parametrize("prec,recon", [(64, 18), (32, 12)])
def test_staggered_block_edges(mods, L4, prec, recon):
    torch, fields, lqcd = mods
    import numpy as np
    theta, nrhs = (0.2, 0.0, -0.4, math.pi), 3
    print(f"\n[case] staggered block edges L={L4} prec={prec}", flush=True)
    U = gauge_field(L4, "exp", eps=0.4, seed=45)
    chi = gaussian_spinor(L4, seed=46, nrhs=nrhs)[:, :, 0, :].copy()
    lat = fields.Lattice(L4, theta)
    out = lat.zeros(lqcd.FIELD_COLOUR_FULL, prec, nrhs=nrhs)
    lqcd.stag_apply(lat.g, lqcd.stag_op(0.1, prec, recon), lat.gauge(U, prec, recon), lat.colour(chi, prec), out, 0,
                    nrhs)
    got = lat.unpack_colour(out, prec, nrhs=nrhs)
    for k in range(nrhs):
        ref = S.apply_M(U, chi[k], L4, theta, 0.1)
        err = np.linalg.norm(got[k] - ref, axis=-1)
        assert err.max() <= TOL[prec] * np.sqrt(np.mean(np.linalg.norm(ref, axis=-1) ** 2)), k


# lattices just large enough for tiles of two right-hand sides (two waves each), with ragged last chunks
@pytest.mark.parametrize("L4,prec,recon", [((44, 20, 20, 4), 64, 18), ((44, 48, 20, 4), 64, 12), ((44, 28, 20, 4), 32, 12),
                                           ((42, 30, 20, 4), 32, 18)])
@pytest.mark.parametrize("dagger", [0, 1])
def test_two_rhs_tiles(mods, L4, prec, recon, dagger):
    torch, fields, lqcd = mods
    theta, kappa, mu = (0.2, 0.0, -0.4, math.pi), 0.14, 0.03
    print(f"\n[case] two-rhs tiles L={L4} prec={prec}/{recon} dagger={dagger}", flush=True)
    psi = gaussian_spinor(L4, seed=44, nrhs=2)
    lat = fields.Lattice(L4, theta)
    o = lqcd.op(kappa, mu, prec, recon)
    Ud = lat.gauge(gauge_field(L4, "exp", eps=0.4, seed=43), prec, recon)
    pair, single = lat.spinor(psi, prec), [lat.spinor(psi[k], prec) for k in range(2)]
    out = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec, nrhs=2)
    lqcd.dslash_apply(lat.g, o, Ud, pair, out, dagger=dagger, nrhs=2)
    got = lat.unpack(out, prec, nrhs=2).reshape(2, lat.V, 4, 3)
    sch = lat.zeros(lqcd.FIELD_SPINOR_PARITY, prec, nrhs=2)
    lqcd.dslash_eo_apply(lat.g, o, Ud, lat.parity_view(pair, 0, prec, 2), sch, 0, lqcd.OP_SCHUR, dagger, 2, lat.workspace(o))
    pb = lat.nbytes(lqcd.FIELD_SPINOR_PARITY, prec)
    for k in range(2):
        # one right-hand side at a time: the kernels the other tests hold to the oracle
        one = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec)
        lqcd.dslash_apply(lat.g, o, Ud, single[k], one, dagger=dagger)
        assert site_rel_err(got[k], lat.unpack(one, prec).reshape(lat.V, 4, 3)) <= TOL[prec], ("full", k)
        f = torch.zeros(2, 2 * pb, dtype=torch.uint8, device="cuda")
        f[0, :pb] = sch.view(2, pb)[k]
        lqcd.dslash_eo_apply(lat.g, o, Ud, lat.parity_view(single[k], 0, prec), f[1, :pb], 0, lqcd.OP_SCHUR, dagger, 1,
                             lat.workspace(o))
        a, b = (lat.unpack(f[i].contiguous(), prec).reshape(lat.V, 4, 3) for i in range(2))
        ev = W.parity(L4) == 0
        assert site_rel_err(a[ev], b[ev]) <= TOL[prec], ("schur", k)


def test_two_rhs_tiles_norms(mods):
    """The reductions of such tiles: a mixed solve whose inner and outer hops both run them."""
    torch, fields, lqcd = mods
    L4, theta, kappa, mu, tol = (44, 28, 20, 4), (0.0, 0.0, 0.0, math.pi), 0.12, 0.05, 1e-10
    print(f"\n[case] two-rhs tiles, solve L={L4}", flush=True)
    U, b = gauge_field(L4, "exp", eps=0.4, seed=45), gaussian_spinor(L4, seed=46, nrhs=2)
    lat = fields.Lattice(L4, theta)
    o = lqcd.op(kappa, mu, 64, 18)
    p = lqcd.solve_params(nrhs=2, tol=tol, maxiter=500, eo=1, inner_prec=32, inner_recon=12, delta_reliable=0.01)
    x = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=2)
    rc, info = lqcd.cg_solve(lat.g, o, lat.gauge(U), lat.spinor(b), x, p, lat.workspace(o, p))
    assert rc == 0, info
    got = lat.unpack(x, 64, nrhs=2).reshape(2, lat.V, 4, 3)
    for k in range(2):
        tr = W.true_residual(U, got[k], b[k], L4, theta, kappa, mu)
        assert tr <= tol and abs(tr - info[k]["true_resid"]) <= 1e-3 * tol


def test_calls_follow_the_current_stream(mods):
    torch, fields, lqcd = mods
    s = torch.cuda.Stream()
    assert lqcd._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(s):
        assert lqcd._stream(None) == s.cuda_stream == lqcd._stream(s)
    assert lqcd._stream(None) == torch.cuda.current_stream().cuda_stream != s.cuda_stream
