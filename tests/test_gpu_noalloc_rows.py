"""GPU test of the workspace-free batched call where the work lists of the library's
tile heights outgrow its fixed array: it falls back on taller tiles with shorter
lists, and the results are tsq_batch_evolve's to the bit."""
import numpy as np
import pytest
import torch

import paper_1208_2407_amd as tsq
from tests.test_zz_no_alloc import both

pytestmark = pytest.mark.gpu

ARRAY = 16 << 20


def setup_module(_):
    tsq.load_library()


def test_noalloc_falls_back_on_taller_tiles():
    rng = np.random.default_rng(5)
    plans, psis = [], []
    for _ in range(512):
        nx, ny = 2 * rng.integers(32, 257, 2)
        plan = tsq.Plan(int(nx), int(ny), 0.05, "c64")
        plan.set_potential(torch.rand(ny, nx, dtype=torch.float64, device="cuda"))
        plans.append(plan)
        psis.append(torch.randn(ny, nx, dtype=torch.complex64, device="cuda"))
    sc = (5, 0, 1, 1)
    args = [p.handle for p in plans], [x.data_ptr() for x in psis], [p.workspace().data_ptr() for p in plans]
    # step counts all over 1 .. 5 m passes: every pass has another set of problems, so
    # another tile list; the first m whose lists are too long for the array
    for m in range(40, 400, 2):
        steps = [5 * (1 + i * m // 512) for i in range(512)]
        if tsq.tsq_batch_evolve_workspace_size(*args, steps, tsq.tsq_schedule(*sc)) > ARRAY:
            break
    else:
        pytest.fail("no batch with lists beyond the array")
    a, b, need = both(plans, psis, steps, sc)
    assert need > ARRAY
    assert all(torch.equal(x, y) for x, y in zip(a, b))
