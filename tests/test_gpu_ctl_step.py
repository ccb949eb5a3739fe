"""CG iterations whose scalar steps run inside their kernels and as launches of
their own: lattices whose partials leave no room for the copies of the control
blocks (2^4), the smallest that do, ragged blocks, several right-hand sides
and shifts; every solution by the oracle's true residual."""

import math

import numpy as np
import pytest

from lattice_inputs import gauge_field, gaussian_spinor
from oracle import staggered as S
from oracle import wilson as W

pytestmark = pytest.mark.gpu

THETA = (0.0, 0.0, 0.0, math.pi)


@pytest.fixture(scope="module")
def mods():
    import torch
    from paper_1411_5219_amd import fields, lqcd
    assert torch.cuda.is_available()
    return torch, fields, lqcd


@pytest.mark.parametrize("L4", [(2, 2, 2, 2), (4, 4, 4, 4), (6, 10, 6, 4)])
@pytest.mark.parametrize("inner,eo,nrhs", [(64, 1, 1), (64, 0, 1), (64, 1, 3), (32, 1, 1), (32, 1, 3), (16, 1, 2)])
def test_cg(mods, L4, inner, eo, nrhs):
    torch, fields, lqcd = mods
    kappa, mu, tol = 0.12, 0.05, 1e-10
    print(f"\n[case] ctl step cg L={L4} inner={inner} eo={eo} nrhs={nrhs}", flush=True)
    U = gauge_field(L4, "exp", eps=0.4, seed=61)
    b = gaussian_spinor(L4, seed=62, nrhs=nrhs)
    lat = fields.Lattice(L4, THETA)
    o = lqcd.op(kappa, mu, 64, 18)
    p = lqcd.solve_params(nrhs=nrhs, tol=tol, maxiter=2000, eo=eo, inner_prec=inner, inner_recon=18 if inner == 64 else 12,
                          delta_reliable=0.0 if inner == 64 else 0.05)
    xd = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs)
    rc, info = lqcd.cg_solve(lat.g, o, lat.gauge(U), lat.spinor(b if nrhs > 1 else b[0]), xd, p, lat.workspace(o, p))
    assert rc == 0, info
    x = lat.unpack(xd, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    for k in range(nrhs):
        tr = W.true_residual(U, x[k], b[k], L4, THETA, kappa, mu)
        assert tr <= tol and abs(tr - info[k]["true_resid"]) <= 1e-3 * tol, (k, tr, info[k])
        assert inner == 64 or info[k]["reliable_updates"] > 0


@pytest.mark.parametrize("L4,n", [((2, 2, 2, 2), 1), ((4, 4, 4, 4), 5), ((8, 8, 8, 4), 1), ((8, 8, 8, 4), 32), ((10, 6, 6, 4), 8)])
def test_multishift(mods, L4, n):
    torch, fields, lqcd = mods
    mass, tol = 0.3, 1e-10
    shifts = [0.01 * 1.3 ** i if i else 0.0 for i in range(n)][::-1]  # the base system comes last
    print(f"\n[case] ctl step multishift L={L4} n={n}", flush=True)
    U = gauge_field(L4, "exp", eps=0.4, seed=63)
    rng = np.random.default_rng(64)
    V = int(np.prod(L4))
    chi = rng.normal(size=(V, 3)) + 1j * rng.normal(size=(V, 3))
    lat = fields.Lattice(L4, THETA)
    b = S.mask(chi, L4, 0)
    o = lqcd.stag_op(mass)
    pb = lat.nbytes(lqcd.FIELD_COLOUR_PARITY, 64)
    xd = lat.zeros(lqcd.FIELD_COLOUR_PARITY, 64, nrhs=n)
    p = lqcd.solve_params(tol=tol, maxiter=2000, eo=1, inner_prec=64)
    rc, info = lqcd.stag_multishift_solve(lat.g, o, lat.gauge(U), lat.colour_parity(lat.colour(b), 0), xd, shifts, p,
                                          lat.stag_workspace(o, n))
    assert rc == 0, info
    for i, sh in enumerate(shifts):
        full = torch.zeros(2 * pb, dtype=torch.uint8, device="cuda")
        full[:pb] = xd[i * pb:(i + 1) * pb]
        x = lat.unpack_colour(full)
        res = np.linalg.norm((b - S.normal_e(U, x, L4, THETA, mass) - sh * x).ravel()) / np.linalg.norm(b.ravel())
        assert res <= tol and abs(res - info[i]["true_resid"]) <= 1e-3 * tol + 1e-15, (i, res, info[i])


@pytest.mark.parametrize("L4,n", [((16, 16, 16, 8), 7), ((18, 14, 10, 12), 6), ((6, 4, 4, 10), 32)])
def test_multishift_shares(mods, L4, n):
    """The multi-shift update in shares of the shifts: uneven ones, and one each."""
    test_multishift(mods, L4, n)


# one system much wider than the others (their blocks lie in a row), equal ones (one grid plane each), and a 2^4
# system, for which the whole batch keeps launches for its scalar steps
@pytest.mark.parametrize("lattices", [[(4, 4, 4, 4), (16, 16, 16, 4), (4, 6, 4, 2)], [(6, 6, 4, 4), (4, 6, 6, 4)],
                                      [(2, 2, 2, 2), (4, 6, 4, 4)]])
@pytest.mark.parametrize("inner,nrhs", [(64, 1), (32, 2)])
@pytest.mark.parametrize("use_graph", [0, 1])
def test_batch(mods, lattices, inner, nrhs, use_graph):
    torch, fields, lqcd = mods
    mu, tol = 0.05, 1e-10
    print(f"\n[case] ctl step batch {lattices} inner={inner} nrhs={nrhs} graph={use_graph}", flush=True)
    geoms, ops, Us, bs, xs, host = [], [], [], [], [], []
    for i, L4 in enumerate(lattices):
        kappa = 0.12 + 0.01 * i
        U, b = gauge_field(L4, "exp", eps=0.4, seed=65 + i), gaussian_spinor(L4, seed=75 + i, nrhs=nrhs)
        lat = fields.Lattice(L4, THETA)
        geoms.append(lat.g)
        ops.append(lqcd.op(kappa, mu))
        Us.append(lat.gauge(U))
        bs.append(lat.spinor(b if nrhs > 1 else b[0]))
        xs.append(lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs))
        host.append((L4, kappa, U, b, lat))
    p = lqcd.solve_params(tol=tol, maxiter=2000, nrhs=nrhs, inner_prec=inner, inner_recon=18 if inner == 64 else 12,
                          use_graph=use_graph)
    ws = torch.empty(lqcd.lqcd_workspace_bytes_batch(geoms, ops, p), dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        rc, infos = lqcd.cg_solve_batch(geoms, ops, Us, bs, xs, p, ws, stream=s)
    torch.cuda.synchronize()
    assert rc == 0, infos
    for i, (L4, kappa, U, b, lat) in enumerate(host):
        x = lat.unpack(xs[i], 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
        for k in range(nrhs):
            tr = W.true_residual(U, x[k], b[k], L4, THETA, kappa, mu)
            assert tr <= tol and abs(tr - infos[i][k]["true_resid"]) <= 1e-3 * tol, (i, k, tr)


def test_update_hops_over_many_blocks(mods):
    """A mixed solve whose update hops stride over more than four rounds of blocks: thirteen right-hand sides that need
    updates in different iterations, one of them zero."""
    torch, fields, lqcd = mods
    L4, nrhs, kappa, mu, tol = (24, 20, 24, 6), 13, 0.13, 0.05, 1e-10
    print(f"\n[case] update hops over many blocks L={L4} nrhs={nrhs}", flush=True)
    U, b = gauge_field(L4, "exp", eps=0.4, seed=91), gaussian_spinor(L4, seed=92, nrhs=nrhs)
    b[5] = 0.0
    for k in range(0, nrhs, 3):  # a point source
        b[k] = 0.0
        b[k].reshape(-1)[k] = 1.0
    lat = fields.Lattice(L4, THETA)
    o = lqcd.op(kappa, mu, 64, 18)
    p = lqcd.solve_params(nrhs=nrhs, tol=tol, maxiter=500, eo=1, inner_prec=32, inner_recon=12, delta_reliable=0.02)
    xd = lat.zeros(lqcd.FIELD_SPINOR_FULL, 64, nrhs=nrhs)
    rc, info = lqcd.cg_solve(lat.g, o, lat.gauge(U), lat.spinor(b), xd, p, lat.workspace(o, p))
    assert rc == 0, info
    x = lat.unpack(xd, 64, nrhs=nrhs).reshape(nrhs, lat.V, 4, 3)
    assert not x[5].any()
    for k in (0, 4, 12):
        tr = W.true_residual(U, x[k], b[k], L4, THETA, kappa, mu)
        assert tr <= tol and abs(tr - info[k]["true_resid"]) <= 1e-3 * tol, (k, tr, info[k])
    assert all(i["true_resid"] <= tol for i in info)
