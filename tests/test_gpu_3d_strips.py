"""GPU test of the slab march's left-over strip, whose lanes serve several slabs of
a block: widths that leave one pair (many groups), a half wavefront and more (one
group), none, or less than a strip in all, with slab counts that fill the groups'
last block or not.  One stage (small meshes) and two, against the oracle;
tolerances as in the other 3D tests."""
import pytest

import oracle
import paper_1208_2407_amd as tsq
from tests.gpu_helpers import TOL, as_input, rel_l2
from tests.test_gpu_3d import ANISO3, gpu_evolve3, rand3

pytestmark = pytest.mark.gpu


def setup_module(_):
    oracle.build(force=False)
    tsq.load_library()


ONE = [(2, 2, 2), (2, 66, 4), (12, 94, 6), (58, 26, 8), (126, 14, 10), (128, 38, 6), (188, 14, 4), (254, 102, 4)]
TWO = [(2, 970, 780), (12, 302, 420), (56, 122, 222), (124, 50, 244), (126, 98, 124), (188, 90, 90),
       (250, 146, 42), (372, 26, 160), (126, 302, 160), (256, 198, 120)]


@pytest.mark.parametrize("dtype", ["c128", "c64"])
@pytest.mark.parametrize("n3", ONE + TWO)
def test_left_over_strips(n3, dtype):
    psi0, V = rand3(n3, 71, scale=0.5)
    psi0 = as_input(psi0, dtype)
    steps = 5 if n3 in ONE else 3
    want = oracle.evolve3(psi0, V, 0.11, steps, **ANISO3)
    assert rel_l2(gpu_evolve3(psi0, V, 0.11, steps, dtype, **ANISO3), want) <= TOL[dtype]
