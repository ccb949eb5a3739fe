"""Solves and hops on lattices large enough for each way a hop launch shares
its sites and right-hand sides among waves."""

import math

import pytest

from lattice_inputs import gauge_field, gaussian_spinor
from oracle import wilson as W

pytestmark = pytest.mark.gpu

THETA = (0.2, 0.0, -0.4, math.pi)


@pytest.fixture(scope="module")
def mods():
    import torch
    from paper_1411_5219_amd import fields, lqcd
    assert torch.cuda.is_available()
    return torch, fields, lqcd


@pytest.fixture(scope="module")
def large():
    """Planes of whole blocks, two chunks per SIMD: the FP64 hops of one right-hand side run one wave per chunk."""
    L4 = (32, 32, 32, 8)
    return L4, gauge_field(L4, "exp", eps=0.3, seed=61), gaussian_spinor(L4, seed=62)


@pytest.mark.parametrize("inner", [64, 32])
def test_batch_of_one_large_rhs(mods, large, inner):
    """A batch whose hops run one wave per chunk: set-up and the final residual
    of the full matrix, which has no such kernel, run their own."""
    torch, fields, lqcd = mods
    L4, U, b = large
    kappa, mu, tol = 0.11, 0.05, 1e-10
    print(f"\n[case] batch of one L={L4} inner={inner}", flush=True)
    lat = fields.Lattice(L4, THETA)
    o = lqcd.op(kappa, mu)
    p = lqcd.solve_params(tol=tol, maxiter=500, eo=1, nrhs=1, inner_prec=inner, inner_recon=12, delta_reliable=0.01)
    x = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64)
    ws = torch.empty(lqcd.lqcd_workspace_bytes_batch([lat.g], [o], p), dtype=torch.uint8, device="cuda")
    rc, infos = lqcd.cg_solve_batch([lat.g], [o], [lat.gauge(U)], [lat.spinor(b)], [x], p, ws)
    assert rc == 0, infos
    tr = W.true_residual(U, lat.unpack(x), b, L4, THETA, kappa, mu)
    assert tr <= tol and abs(tr - infos[0][0]["true_resid"]) <= 1e-3 * tol


# The bounds of test_gpu_dslash.py: FP64 rounding of about 1000 operations per
# site; FP32 the same at 6e-8; FP16 storage 2^-11 of a site's largest value.
TOL = {64: 1e-13, 32: 1e-5, 16: 1e-2}
A = (20, 18, 16, 8)     # 180 sites per plane: a ragged last chunk
B = (20, 14, 10, 10)    # chunks over several planes, a time extent of 10: memory order in FP64
C = (20, 14, 12, 12)    # the same where FP32/12 pairs no longer run at once
D = (24, 20, 18, 8)     # room for three such pairs is not left: they lie next to each other
P, T, N = 2, 3, 5       # FORM_PAIR, FORM_TILE, FORM_NEXT
# lattice, storage, right-hand sides, form of one parity and of both: tiles of
# three and four, with a last tile that is full and one that is not, and pairs
# with their right-hand sides next to each other
FORMS = [(A, 64, 18, 3, T, N), (A, 64, 18, 4, T, N), (A, 64, 18, 5, N, N), (A, 64, 12, 4, T, N), (A, 64, 12, 7, N, N),
         (B, 64, 18, 5, T, N), (B, 64, 12, 7, T, P),
         (A, 32, 18, 5, T, T), (A, 32, 18, 7, T, T), (A, 32, 12, 3, P, P), (A, 32, 12, 5, T, T), (A, 32, 12, 8, T, T),
         (C, 32, 12, 5, N, T), (A, 16, 12, 3, P, P), (A, 16, 12, 5, T, T), (A, 16, 12, 7, T, T), (C, 16, 12, 3, P, P),
         (D, 16, 12, 3, N, N), (D, 32, 12, 3, N, T)]


@pytest.fixture(scope="module")
def choice(tmp_path_factory):
    import ctypes
    import subprocess
    import test_hop_form as H
    so = str(tmp_path_factory.mktemp("forms") / "forms.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", H.CSRC,
                    H.os.path.join(H.HERE, "hop_form_harness.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    return lambda *a: H.choose(lib, *a)


def per_site(got, ref):
    from gpu_util import site_rel_err
    return site_rel_err(got, ref)


@pytest.mark.parametrize("L4,prec,recon,nrhs,parity,full", FORMS)
@pytest.mark.parametrize("dagger", [0, 1])
def test_several_rhs(mods, choice, L4, prec, recon, nrhs, parity, full, dagger):
    torch, fields, lqcd = mods
    kappa, mu = 0.14, 0.03
    print(f"\n[case] several rhs L={L4} prec={prec}/{recon} nrhs={nrhs} dagger={dagger}", flush=True)
    assert choice(prec, recon, 0, [L4], nrhs)[0] == parity and choice(prec, recon, 1, [L4], nrhs)[0] == full
    U = gauge_field(L4, "exp", eps=0.4, seed=63)
    psi = gaussian_spinor(L4, seed=64, nrhs=nrhs)
    lat = fields.Lattice(L4, THETA)
    o = lqcd.op(kappa, mu, prec, recon)
    Ud, src = lat.gauge(U, prec, recon), lat.spinor(psi, prec)
    out = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec, nrhs=nrhs)
    lqcd.dslash_apply(lat.g, o, Ud, src, out, dagger=dagger, nrhs=nrhs)
    got = lat.unpack(out, prec, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    sch = lat.zeros(lqcd.FIELD_SPINOR_PARITY, prec, nrhs=nrhs)
    lqcd.dslash_eo_apply(lat.g, o, Ud, lat.parity_view(src, 0, prec, nrhs), sch, 0, lqcd.OP_SCHUR, dagger, nrhs,
                         lat.workspace(o))
    pb = lat.nbytes(lqcd.FIELD_SPINOR_PARITY, prec)
    f = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec, nrhs=nrhs)
    f.view(nrhs, 2, pb)[:, 0, :] = sch.view(nrhs, pb)
    even = lat.unpack(f, prec, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    ev = W.parity(L4) == 0
    for k in range(nrhs):
        ref = W.apply_M(U, psi[k], L4, THETA, kappa, mu, dagger=bool(dagger))
        assert per_site(got[k], ref) <= TOL[prec], ("full", k)
        ref = W.schur(U, W.mask(psi[k], L4, 0), L4, THETA, kappa, mu, dagger=bool(dagger))
        assert per_site(even[k][ev], ref[ev]) <= TOL[prec], ("schur", k)


@pytest.mark.parametrize("recon,nrhs", [(18, 3), (12, 3), (18, 2)])
def test_large_tiles(mods, large, choice, recon, nrhs):
    """FP64 tiles on a lattice of whole planes: both parities, and the Schur complement."""
    torch, fields, lqcd = mods
    L4, U, b = large
    kappa, mu = 0.14, 0.03
    print(f"\n[case] large tiles L={L4} recon={recon} nrhs={nrhs}", flush=True)
    assert choice(64, recon, 1, [L4], nrhs)[0] == choice(64, recon, 0, [L4], nrhs)[0] == T
    lat = fields.Lattice(L4, THETA)
    src = lat.spinor(b).repeat(nrhs)
    scale = [1.0, -0.5, 2.0][:nrhs]
    src.view(torch.float64).view(nrhs, -1).mul_(torch.tensor(scale, dtype=torch.float64, device="cuda")[:, None])
    out = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs)
    o, Ud = lqcd.op(kappa, mu, 64, recon), lat.gauge(U, 64, recon)
    lqcd.dslash_apply(lat.g, o, Ud, src, out, dagger=1, nrhs=nrhs)
    ref = W.apply_M(U, b, L4, THETA, kappa, mu, dagger=True)
    got = lat.unpack(out, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    for k in range(nrhs):
        assert per_site(got[k], scale[k] * ref) <= TOL[64], k
    sch = lat.zeros(lqcd.FIELD_SPINOR_PARITY, 64, nrhs=nrhs)
    lqcd.dslash_eo_apply(lat.g, o, Ud, lat.parity_view(src, 0, 64, nrhs), sch, 0, lqcd.OP_SCHUR, 0, nrhs,
                         lat.workspace(o))
    f = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs)
    f.view(nrhs, 2, -1)[:, 0, :] = sch.view(nrhs, -1)
    even = lat.unpack(f, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    ref = W.schur(U, W.mask(b, L4, 0), L4, THETA, kappa, mu)
    ev = W.parity(L4) == 0
    for k in range(nrhs):
        assert per_site(even[k][ev], scale[k] * ref[ev]) <= TOL[64], ("schur", k)


@pytest.mark.parametrize("L4,inner,nrhs", [(A, 32, 5), (A, 64, 5), (A, 16, 7), (C, 32, 5), (B, 64, 5)])
def test_reductions_of_several_rhs(mods, L4, inner, nrhs):
    """Their norms: solves certified by the oracle."""
    torch, fields, lqcd = mods
    kappa, mu, tol = 0.13, 0.03, 1e-10
    print(f"\n[case] several rhs solve L={L4} inner={inner} nrhs={nrhs}", flush=True)
    U, b = gauge_field(L4, "exp", eps=0.4, seed=65), gaussian_spinor(L4, seed=66, nrhs=nrhs)
    lat = fields.Lattice(L4, THETA)
    o = lqcd.op(kappa, mu)
    p = lqcd.solve_params(nrhs=nrhs, tol=tol, maxiter=1000, eo=1, inner_prec=inner, inner_recon=12, delta_reliable=0.05)
    x = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs)
    rc, info = lqcd.cg_solve(lat.g, o, lat.gauge(U), lat.spinor(b), x, p, lat.workspace(o, p))
    assert rc == 0, info
    got = lat.unpack(x, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    for k in range(nrhs):
        tr = W.true_residual(U, got[k], b[k], L4, THETA, kappa, mu)
        assert tr <= tol and abs(tr - info[k]["true_resid"]) <= 1e-3 * tol, k


@pytest.mark.parametrize("nrhs", [2, 3, 5, 16])
def test_persistent_batch(mods, nrhs):
    """The persistent kernel's hops, one wave per chunk: planes of whole blocks,
    a ragged last chunk and chunks over several planes, right-hand sides that
    the kernel's blocks share unevenly."""
    torch, fields, lqcd = mods
    mu, tol = 0.03, 1e-10
    systems = [((32, 16, 4, 4), 0.12), ((20, 18, 4, 4), 0.13), ((6, 10, 4, 12), 0.11)]
    print(f"\n[case] persistent batch nrhs={nrhs}", flush=True)
    geoms, ops, Us, bs, xs, host = [], [], [], [], [], []
    for i, (L4, kappa) in enumerate(systems):
        U, b = gauge_field(L4, "exp", eps=0.4, seed=67 + i), gaussian_spinor(L4, seed=77 + i, nrhs=nrhs)
        lat = fields.Lattice(L4, THETA)
        host.append((L4, kappa, U, b, lat))
        geoms.append(lat.g)
        ops.append(lqcd.op(kappa, mu))
        Us.append(lat.gauge(U))
        bs.append(lat.spinor(b))
        xs.append(lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs))
    p = lqcd.solve_params(tol=tol, maxiter=1000, eo=1, nrhs=nrhs, inner_prec=32, inner_recon=12, delta_reliable=0.05,
                          persistent=1)
    ws = torch.empty(lqcd.lqcd_workspace_bytes_batch(geoms, ops, p), dtype=torch.uint8, device="cuda")
    rc, infos = lqcd.cg_solve_batch(geoms, ops, Us, bs, xs, p, ws)
    assert rc == 0 and infos[0][0]["persistent_launches"] >= 1, infos
    for (L4, kappa, U, b, lat), x, info in zip(host, xs, infos):
        got = lat.unpack(x, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
        for k in range(nrhs):
            tr = W.true_residual(U, got[k], b[k], L4, THETA, kappa, mu)
            assert tr <= tol and abs(tr - info[k]["true_resid"]) <= 1e-3 * tol, (L4, k)


@pytest.mark.parametrize("L4,prec,recon,nrhs", [(A, 64, 18, 5), (A, 32, 12, 3), (A, 16, 12, 5)])
def test_launch_fields_without_effect(mods, L4, prec, recon, nrhs):
    """rhs_tile, rhs_group and rhs_lanes change no result, whichever form the hop
    takes; the answer is the same bytes."""
    torch, fields, lqcd = mods
    print(f"\n[case] launch fields L={L4} prec={prec} nrhs={nrhs}", flush=True)
    lat = fields.Lattice(L4, THETA)
    Ud = lat.gauge(gauge_field(L4, "exp", eps=0.4, seed=69), prec, recon)
    inp = lat.spinor(gaussian_spinor(L4, seed=79, nrhs=nrhs), prec)
    op, saved = lqcd.op(0.16, 0.005, prec, recon), lqcd.lqcd_get_launch(lqcd.KERNEL_DSLASH_RHS, prec)
    outs = []
    try:
        for tile, group, lanes in [(4, 4, 1), (1, 0, 1), (2, 2, 4), (4, 16, 16)]:
            lqcd.lqcd_set_launch(lqcd.KERNEL_DSLASH_RHS, prec,
                                 **dict(saved, rhs_tile=tile, rhs_group=group, rhs_lanes=lanes))
            out = lat.zeros(lqcd.FIELD_SPINOR_FULL, prec, nrhs=nrhs)
            lqcd.dslash_apply(lat.g, op, Ud, inp, out, nrhs=nrhs)
            outs.append(out)
    finally:
        lqcd.lqcd_set_launch(lqcd.KERNEL_DSLASH_RHS, prec, **saved)
    assert outs[0].any() and all(torch.equal(outs[0], o) for o in outs[1:])
