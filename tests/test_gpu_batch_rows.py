"""GPU test of the tile heights the library picks for a batch: whatever the
height (one round of low tiles, several rounds, problems lower than a tile),
every problem is bit for bit the one evolved alone, also after a second launch.
"""
import pytest
import torch

import paper_1208_2407_amd as tsq
from paper_1208_2407_amd import workloads as wl
from tests.gpu_helpers import TORCH_DT, as_input
from tests.test_gpu_batch import build_batch

pytestmark = pytest.mark.gpu


def setup_module(_):
    tsq.load_library()


# sides of the problems: one tile; a few low tiles; uneven heights; more strips
# than wavefronts resident in either dtype, so that every height takes several rounds
@pytest.mark.parametrize("sides", [[(2, 2)], [(66, 40), (130, 258), (6, 300)],
                                   [(512, 2), (40, 1024), (300, 130), (130, 66)] * 3,
                                   [(258, 80), (300, 40)] * 400])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("steps_per_pass", [0, 6])
def test_library_tile_heights(dtype, sides, steps_per_pass):
    steps = 13
    kinds = {s: (as_input(wl.random_state(*s, 5 + s[0]), dtype), wl.random_potential(*s, 9 + s[1], scale=0.5),
                 0.05, steps) for s in set(sides)}
    batch, plans, psis, _ = build_batch([kinds[s] for s in sides], dtype, (steps_per_pass, 0, 0, 0))
    batch.launch()
    batch.launch()
    torch.cuda.synchronize()
    alone = {}
    for s, (psi0, V, dt, _) in kinds.items():
        psi = torch.from_numpy(psi0).to(TORCH_DT[dtype]).cuda()
        plan = tsq.Plan(*s, dt, dtype, device=psi.device)
        plan.set_schedule(5, 20, 1, 1)
        plan.set_potential(torch.from_numpy(V).cuda())
        plan.evolve(psi, steps)
        plan.evolve(psi, steps)
        alone[s] = psi
    torch.cuda.synchronize()
    assert all(torch.equal(psi, alone[s]) for psi, s in zip(psis, sides))
