"""3D meshes over the range of complex64: scaling the state by a power of two scales the
result by it, to the bit, as long as nothing leaves the type's range.  Sizes of the
slab march's one and two stages and, from 6M sites, two row pairs per wavefront."""
import pytest
import torch

import paper_1208_2407_amd as tsq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [0.1, 2.7])  # tangent form, delta form
@pytest.mark.parametrize("n3", [(34, 18, 12), (130, 98, 120), (194, 250, 126)])
def test_large_amplitudes_stay_in_range(n3, dt):
    nx, ny, nz = n3
    gen = torch.Generator(device="cuda").manual_seed(3)
    psi0 = torch.randn(nz, ny, nx, dtype=torch.complex64, device="cuda", generator=gen)
    V = torch.rand(nz, ny, nx, dtype=torch.float64, device="cuda", generator=gen)
    plan = tsq.Plan(nx, ny, dt, "c64", nz=nz)
    plan.set_potential(V)
    for steps in (1, 4, 5):
        want, big = psi0.clone(), psi0 * 2.0 ** 110  # parts up to 8e33
        plan.evolve(want, steps)
        plan.evolve(big, steps)
        assert torch.isfinite(torch.view_as_real(want)).all()
        assert torch.equal(big * 2.0 ** -110, want), steps
