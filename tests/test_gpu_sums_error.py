"""Rounding of the norm and energy sums.  u = 2^-53.

A state of one real value r on a mesh of 2^k sites: every site adds q = fl(r r), and the
mesh's norm 2^k q is a double.  A thread's rows must not round one behind the other (the
same error in every thread): one rounding for a thread's sum, at most two in the tree
of the bands where they leave a remainder, so 4 u.

Random states: the additions of a tree round by up to half an ulp of their result (0 to u
of it, 0.43 u rms); the errors of a level of n equal parts come to 1/sqrt(n) of that, so all
levels together to 0.43 sqrt(1 + 1/2 + 1/4 + ...) = 0.61 u rms.  32 draws estimate that to
an eighth; 0.9 u allows for it four times and fails one behind the other sums of 16
parts (0.43 sqrt(16 / 3) = 1.0 u and more)."""
import numpy as np
import pytest
import torch

import paper_1208_2407_amd as tsq

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.mark.parametrize("bc", ["periodic", "closed"])
@pytest.mark.parametrize("shape", [(2048, 16384), (512, 8192), (16384, 2048)])
def test_norm_of_a_flat_state(shape, bc):
    nx, ny = shape
    V = torch.zeros(ny, nx, dtype=torch.float64, device="cuda")
    for r in (1 / 3, 0.1, 0.7, np.pi / 4, np.e / 3, 0.123456789):
        psi = torch.full((ny, nx), complex(r, 0.0), dtype=torch.complex128, device="cuda")
        n, _ = tsq.observables(psi, V, bc=bc)
        assert abs(n / (nx * ny * (r * r)) - 1) <= 4 * U, r


@pytest.mark.parametrize("bc", ["periodic", "closed"])
def test_norm_of_random_states(bc):
    nx, ny = 512, 2048
    V = torch.zeros(ny, nx, dtype=torch.float64, device="cuda")
    rng = np.random.default_rng(4)
    err = []
    for _ in range(32):
        x = rng.standard_normal((ny, nx, 2))
        n, _ = tsq.observables(torch.view_as_complex(torch.from_numpy(x)).cuda(), V, bc=bc)
        exact = (x.astype(np.longdouble) ** 2).sum()
        err.append(float((n - exact) / exact) / U)
    assert np.sqrt(np.mean(np.square(err))) <= 0.9


@pytest.mark.parametrize("bc", ["periodic", "closed"])
def test_infinite_and_missing_values_stay_so(bc):
    V = torch.zeros(64, 64, dtype=torch.float64, device="cuda")
    for big, want in ((1e200, np.inf), (np.nan, np.nan)):
        psi = torch.ones(64, 64, dtype=torch.complex128, device="cuda")
        psi[7, 9] = big
        n, _ = tsq.observables(psi, V, bc=bc)
        assert np.array_equal(n, want, equal_nan=True)
