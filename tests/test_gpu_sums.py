"""GPU test of how the norm and energy sums are cut: bands of rows that end inside
a walk of four, one block to more items than blocks, and last-stage sums of one
partial up to thousands (3D: one a row).  Bounds as in the other tests of the
sums: 1e-13 for the norm, 1e-12 for the energy, relative; the same bits twice."""
import numpy as np
import pytest
import torch

import oracle
import paper_1208_2407_amd as tsq
from paper_1208_2407_amd import workloads as wl
from tests.gpu_helpers import TORCH_DT, as_input

pytestmark = pytest.mark.gpu


def setup_module(_):
    oracle.build(force=False)
    tsq.load_library()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape,bc", [((4, 1023), "closed"), ((2, 1030), "periodic"), ((4, 8202), "periodic"),
                                      ((514, 3074), "periodic"), ((257, 4101), "closed"),
                                      ((526338, 2), "periodic"), ((262403, 3), "closed")])
def test_sums_of_uneven_bands(shape, bc, dtype):
    nx, ny = shape
    psi0 = as_input(wl.random_state(nx, ny, 8) * 1.3, dtype)
    V = wl.random_potential(nx, ny, 9)
    psi, Vd = torch.from_numpy(psi0).to(TORCH_DT[dtype]).cuda(), torch.from_numpy(V).cuda()
    n, e = tsq.observables(psi, Vd, bc=bc)
    n0, e0 = oracle.observables(psi0, V, bc=bc)
    assert abs(n - n0) <= 1e-13 * abs(n0) and abs(e - e0) <= 1e-12 * max(1.0, abs(e0))
    assert tsq.observables(psi, Vd, bc=bc) == (n, e)


@pytest.mark.parametrize("shape", [(2, 2, 2), (2, 64, 64), (6, 66, 64), (4, 130, 66)])
def test_3d_sums_of_many_rows(shape):
    rng = np.random.default_rng(6)
    psi0 = rng.standard_normal(shape[::-1]) + 1j * rng.standard_normal(shape[::-1])
    V = rng.standard_normal(shape[::-1])
    psi, Vd = torch.from_numpy(psi0).cuda(), torch.from_numpy(V).cuda()
    n, e = tsq.observables(psi, Vd)
    n0, e0 = oracle.observables3(psi0, V)
    assert abs(n - n0) <= 1e-13 * n0 and abs(e - e0) <= 1e-12 * max(1.0, abs(e0))
    assert tsq.observables(psi, Vd) == (n, e)
