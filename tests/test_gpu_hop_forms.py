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
