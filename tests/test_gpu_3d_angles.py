"""3D meshes over the angles of the tangent form, up to 1 rad a step and axis, and the delta
form just beyond, against the oracle: one stage, two stages with one and (complex64) two
row pairs per wavefront.  complex128 <= 1e-12.  complex64 <= 1e-5: a rounded tangent
turns a pair by up to 2^-26 rad too far, nine factors a step, so 40 steps come to 5.4e-6
at most, and their rounding to about 3e-6."""
import numpy as np
import pytest

import oracle
import paper_1208_2407_amd as tsq
from tests.gpu_helpers import TOL, as_input, rel_l2
from tests.test_gpu_3d import gpu_evolve3, rand3

pytestmark = pytest.mark.gpu


def setup_module(_):
    oracle.build(force=False)
    tsq.load_library()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("angle", [0.3, 0.5, 0.8, 0.95, 0.999, 1.001])  # rad per step along x
@pytest.mark.parametrize("n3,steps", [((34, 18, 12), (1, 40)), ((130, 98, 120), (7, 8)), ((194, 250, 126), (3, 4))])
def test_3d_angles_match_the_oracle(n3, steps, angle, dtype):
    dt = 0.1
    dx = float(np.sqrt(dt / (2 * angle)))
    spacing = dict(dx=dx, dy=1.1 * dx, dz=1.05 * dx)
    psi0, V = rand3(n3, 71, scale=2.0)
    psi0 = as_input(psi0, dtype)
    want, done = psi0, 0
    for n in steps:
        want, done = oracle.evolve3(want, V, dt, n - done, **spacing), n
        assert rel_l2(gpu_evolve3(psi0, V, dt, n, dtype, **spacing), want) <= TOL[dtype], n
