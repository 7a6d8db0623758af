"""The tile kernels of small 2D meshes: which calls they take (host logic), and on the
GPU the march's own bits at the edges of their tiles (the march itself is held to
the oracle in the other tests)."""
import numpy as np
import pytest
import torch

import paper_1208_2407_amd as tsq
from paper_1208_2407_amd import workloads as wl
from tests.gpu_helpers import TORCH_DT, as_input

MARCH = (5, 0, 1, 1)   # the defaults, set explicitly: the march


def test_tile_kernels_take_small_meshes_under_the_default_schedule_only():
    for n, steps in ((64, 100), (256, 100), (1030, 200)):
        plan = tsq.Plan(n, n, 0.05, "c64")
        own = plan.passes(steps)
        assert own[0] != steps // 5 and own[0] % 2 == 0 and own[1] is False
        assert plan.passes(1) == (1, True) and plan.passes(2) == (2, False)
        assert plan.passes(0) == (0, False)
        plan.set_schedule(*MARCH)
        assert plan.passes(steps) == (steps // 5, False) and plan.schedule() == MARCH
        plan.set_schedule(0, 0, 0, 0)
        assert plan.passes(steps) == own and plan.schedule() == MARCH
        plan.set_schedule(0, 64, 0, 0)
        assert plan.passes(steps) == (steps // 5, False)
    assert tsq.Plan(4096, 4096, 0.05, "c64").passes(100) == (20, False)
    assert tsq.Plan(64, 64, 0.05, "c64", order=4).passes(7) == (7, True)


def run(nx, ny, dtype, bc, kind, steps, schedule):
    """psi after `steps` steps of a random problem; the passes made."""
    psi = torch.from_numpy(as_input(wl.random_state(nx, ny, 90 + nx), dtype)).to(TORCH_DT[dtype]).cuda()
    V = torch.from_numpy(wl.random_potential(nx, ny, 91 + ny)).cuda()
    plan = tsq.Plan(nx, ny, 0.11, dtype, dx=1.3, dy=0.8, mass=1.7, hbar=0.9, bc=bc,
                    order=4 if kind == "order4" else 2)
    plan.set_schedule(*schedule)
    if kind == "td":
        plan.set_potential_td(V, torch.from_numpy(wl.random_potential(nx, ny, 92)).cuda())
        plan.evolve_td(psi, np.random.default_rng(93).uniform(-1, 1, steps))
    else:
        plan.set_potential(V)
        plan.evolve(psi, steps)
    return psi.cpu(), plan.passes(steps)


# sides at the edges of a tile: fewer rows than a block holds, one strip, strips and
# segments with a remainder; the largest take two blocks per compute unit
SHAPES = [(2, 2), (6, 50), (64, 64), (102, 34), (130, 66), (300, 258), (770, 514), (1030, 614)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("bc,kind", [("periodic", "static"), ("periodic", "td"), ("periodic", "order4"),
                                     ("closed", "static"), ("closed", "td")])
@pytest.mark.parametrize("shape", SHAPES)
def test_tile_kernels_give_the_marchs_bits(shape, bc, kind, dtype):
    nx, ny = shape
    if bc == "closed":
        nx, ny = nx + 1, ny - 1 if ny > 2 else ny + 1
    for steps in (1, 2, 6, 7, 13, 40) if kind != "order4" else (1, 2, 5):
        want, march = run(nx, ny, dtype, bc, kind, steps, MARCH)
        got, own = run(nx, ny, dtype, bc, kind, steps, (0, 0, 0, 0))
        assert torch.equal(got, want), (steps, own, march)
