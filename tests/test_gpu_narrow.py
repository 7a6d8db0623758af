"""GPU test of the segment heights the library picks for meshes of one to four strips
(a block's empty wavefronts), from shorter than a segment to many segments: the bits
of two explicit heights."""
import numpy as np
import pytest

import paper_1208_2407_amd as tsq
from paper_1208_2407_amd import workloads as wl
from tests.gpu_helpers import as_input, gpu_evolve

pytestmark = pytest.mark.gpu


def setup_module(_):
    tsq.load_library()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("bc", ["periodic", "closed"])
@pytest.mark.parametrize("S,store", [(2, 1), (5, 1), (7, 2)])
@pytest.mark.parametrize("shape", [(42, 6218), (118, 400), (120, 3000), (330, 1030), (470, 34)])
def test_narrow_meshes(shape, S, store, bc, dtype):
    nx, ny = shape
    psi0, V = as_input(wl.random_state(nx, ny, 3), dtype), wl.random_potential(nx, ny, 4, scale=0.5)
    for steps in (2, 9):
        got = [gpu_evolve(psi0, V, 0.1, steps, dtype, steps_per_pass=S, segment_rows=rows, phase_store=store, bc=bc)
               for rows in (0, 16, 100)]
        assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
