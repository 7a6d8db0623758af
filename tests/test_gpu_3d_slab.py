"""The slab march of 3D meshes at the sizes its forms start from (one stage below 1.5M
sites, two stages above, complex64 with two row pairs per wavefront from 6M), at sides
that leave remainders of strip, slab and segment, against the oracle; odd counts end
with the closing factors in their last pass or by themselves, so 1 to 6 steps take
every ending.  Steps beyond the tangent form's angles keep the delta form.
Tolerances as in the other 3D tests: complex128 <= 1e-12, complex64 <= 1e-5."""
import numpy as np
import pytest
import torch

import oracle
import paper_1208_2407_amd as tsq
from tests.gpu_helpers import TOL, as_input, rel_l2
from tests.test_gpu_3d import ANISO3, gpu_evolve3, rand3

pytestmark = pytest.mark.gpu


def setup_module(_):
    oracle.build(force=False)
    tsq.load_library()


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n3", [(130, 98, 120), (122, 26, 476), (194, 250, 126)])
def test_slab_two_stages_match_the_oracle(n3, dtype):
    assert np.prod(n3) >= 1500000
    psi0, V = rand3(n3, 61, scale=0.5)
    psi0 = as_input(psi0, dtype)
    want = psi0
    for steps in range(1, 7):
        want = oracle.evolve3(want, V, 0.11, 1, **ANISO3)
        got = gpu_evolve3(psi0, V, 0.11, steps, dtype, **ANISO3)
        assert rel_l2(got, want) <= TOL[dtype], (n3, steps)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n3", [(130, 98, 120), (194, 250, 126)])
def test_slab_segments_do_not_change_a_bit(n3, dtype):
    psi0, V = rand3(n3, 62)
    for steps in (5, 6, 7):
        ref = gpu_evolve3(psi0, V, 0.09, steps, dtype, segment_planes=n3[2])
        for seg in (2, 6, 34, 0):
            assert np.array_equal(gpu_evolve3(psi0, V, 0.09, steps, dtype, segment_planes=seg), ref), (steps, seg)


@pytest.mark.parametrize("dtype", ["c128", "c64"])
def test_large_angles_keep_the_delta_form(dtype):
    psi0, V = rand3((66, 34, 12), 63, scale=0.1)
    psi0 = as_input(psi0, dtype)
    for steps in (1, 4):
        want = oracle.evolve3(psi0, V, 2.7, steps)
        assert rel_l2(gpu_evolve3(psi0, V, 2.7, steps, dtype), want) <= TOL[dtype], steps
