"""Norm of complex128 3D meshes over many steps.  A step's cosines come back through the
phase table; an error of their product would scale every site alike at every step.  What
may remain are the roundings of the entries (different at every site, the same at every
step) and of the arithmetic (different at both): over 2^14 sites of equal weight they
move the norm by less than 2^-53 * 2 / 128 a step each, so a quarter of an ulp of
each step is an ample bound; the last odd x factor and the sum add a few ulps."""
import numpy as np
import pytest
import torch

import paper_1208_2407_amd as tsq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("angle", [0.025, 0.1, 0.2, 0.3, 0.4, 0.5, 0.8, 0.95])  # rad per step and axis
def test_norm_does_not_drift(angle):
    nx, ny, nz, dt, steps = 64, 16, 16, 0.1, 800
    dx = np.sqrt(dt / (2 * angle))
    rng = np.random.default_rng(2)
    psi0 = np.exp(2j * np.pi * rng.random((nz, ny, nx)))
    psi = torch.from_numpy(psi0).cuda()
    plan = tsq.Plan(nx, ny, dt, "c128", nz=nz, dx=dx, dy=dx, dz=dx)
    plan.set_potential(torch.from_numpy(rng.uniform(-5, 5, (nz, ny, nx))).cuda())
    plan.evolve(psi, steps)
    got = torch.view_as_real(psi).cpu().numpy().astype(np.longdouble)
    want = psi0.view(np.float64).astype(np.longdouble)
    drift = float((got ** 2).sum() / (want ** 2).sum() - 1)
    assert abs(drift) <= (steps / 4 + 8) * 2.0 ** -53
