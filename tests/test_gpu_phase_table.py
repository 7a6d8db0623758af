"""GPU test of the phase table: angles on both sides of the complex64 table's own
reduction (|phi| < 2^30), quadrant borders, site counts on both sides of the
four-sites-a-thread grid, and the closed meshes' odd last column and row.  One
step with each against the oracle, at the dtype's tolerance."""
import numpy as np
import pytest

import oracle
import paper_1208_2407_amd as tsq
from paper_1208_2407_amd import workloads as wl
from tests.gpu_helpers import TOL, as_input, gpu_evolve, rel_l2
from tests.test_gpu_parity import oracle_evolve

pytestmark = pytest.mark.gpu


def setup_module(_):
    oracle.build(force=False)
    tsq.load_library()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("shape", [(2, 2), (1030, 614), (77, 45)])  # (77, 45): closed
@pytest.mark.parametrize("angle", [0.0, 1e-9, 1.0, 1e4, 1e9, 3e9])
def test_one_step_at_angles_of_every_size(dtype, shape, angle):
    nx, ny = shape
    dt = 0.05
    psi0 = as_input(wl.random_state(nx, ny, 3), dtype)
    # even and odd multiples of pi/4 among the angles, as near as doubles come
    quarter = np.pi / 4 * np.random.default_rng(4).integers(-9, 10, (ny, nx))
    V = (angle * np.random.default_rng(5).uniform(-1, 1, (ny, nx)) + quarter) / dt
    more = {"bc": "closed"} if nx & 1 else {}
    want = oracle_evolve(psi0, V, dt, 1, dtype, **more)
    # the angle itself carries an ulp (2^-53 of it); 3e9 keeps that under 4e-7
    tol = max(TOL[dtype], 2.0 ** -51 * angle)
    assert rel_l2(gpu_evolve(psi0, V, dt, 1, dtype, **more), want) <= tol
