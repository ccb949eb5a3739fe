"""The force kernel's block order where the 64-site segments of an xy plane
group unevenly: a ragged last segment, a prime count above and below the group,
several groups; with and without accumulation."""

import math

import numpy as np
import pytest

from gpu_util import site_rel_err
from lattice_inputs import gauge_field, gaussian_spinor
from oracle import force as F
from oracle import wilson as W

pytestmark = pytest.mark.gpu

KAPPA, MU = 0.13, 0.2


@pytest.fixture(scope="module")
def mods():
    import torch
    from paper_1411_5219_amd import fields, lqcd
    assert torch.cuda.is_available()
    return torch, fields, lqcd


@pytest.mark.parametrize("L4", [(2, 2, 4, 2), (14, 10, 4, 2), (22, 12, 2, 4), (16, 28, 2, 2), (24, 32, 2, 2)])
@pytest.mark.parametrize("recon", [18, 12])
def test_groups(mods, L4, recon):
    torch, fields, lqcd = mods
    theta = (0.3, -0.7, 1.1, math.pi)
    print(f"\n[case] force blocks L={L4} recon={recon}", flush=True)
    U = gauge_field(L4, "haar", seed=81)
    X, Z = gaussian_spinor(L4, seed=82), gaussian_spinor(L4, seed=83)
    lat = fields.Lattice(L4, theta)
    _, g5 = W.gammas()
    Wf = np.einsum("st,...tc->...sc", g5, Z)
    ref = F.force(U, X, Z, L4, theta, KAPPA)
    rng = np.random.default_rng(84)
    F0 = rng.normal(size=(4, lat.V, 3, 3)) + 1j * rng.normal(size=(4, lat.V, 3, 3))
    o = lqcd.op(KAPPA, MU, 64, recon)
    Ud, Xd, Wd = lat.gauge(U, 64, recon), lat.spinor(X), lat.spinor(Wf)
    out = torch.full((4, lat.V, 3, 3), float("nan"), dtype=torch.complex128, device=lat.device)
    lqcd.tm_force(lat.g, o, Ud, Xd, Wd, out, scale=1.0, accumulate=0)
    acc = torch.as_tensor(F0).to(lat.device).contiguous()
    lqcd.tm_force(lat.g, o, Ud, Xd, Wd, acc, scale=-0.5, accumulate=1)
    got, ga = out.cpu().numpy(), acc.cpu().numpy()
    # the bounds of test_gpu_force.py, and the rounding of one addition to entries below 8
    tol = 1e-13 if recon == 18 else 1e-12
    assert site_rel_err(got, ref, ncomp=9) <= tol
    assert np.abs(ga.reshape(F0.shape) - (F0 - 0.5 * ref.reshape(F0.shape))).max() <= tol * np.abs(ref).max() + 4e-15
