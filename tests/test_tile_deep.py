"""The deep passes of the tile kernels, up to 15 stages of 32 row pairs (2 of them stored, 34
of 64 lanes kept, the tightest remainder): the march's own bits.  `stages` is the deepest
pass of each evolution, the steps and the closing factors dealt evenly over its passes."""
import pytest
import torch

import paper_1208_2407_amd as tsq
from tests.test_tile import MARCH, run

CASES = [  # nx, ny, dtype, bc, {steps: stages}
    (64, 64, "c64", "periodic", {13: 7, 17: 5, 28: 15, 29: 15, 46: 6}),
    (65, 63, "c64", "closed", {13: 7, 28: 15, 29: 15}),
    (102, 34, "c64", "periodic", {28: 15, 29: 15}),
    (256, 256, "c128", "periodic", {16: 9, 17: 9, 28: 15, 29: 15, 46: 6}),
    (301, 257, "c128", "closed", {16: 9, 17: 9}),
    (770, 514, "c64", "periodic", {15: 8, 17: 9, 100: 9}),
    (1030, 614, "c64", "periodic", {14: 8, 15: 8, 28: 8, 46: 8}),
    (1031, 613, "c64", "closed", {14: 8, 15: 8, 29: 8}),
]


@pytest.mark.parametrize("nx,ny,dtype,bc,stages", CASES)
def test_the_deep_split_is_taken(nx, ny, dtype, bc, stages):
    plan = tsq.Plan(nx, ny, 0.05, dtype, bc=bc)
    for steps, deepest in stages.items():
        passes, copy = plan.passes(steps)
        assert -(-(steps + 1) // passes) == deepest and not copy, steps


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["static", "td"])
@pytest.mark.parametrize("nx,ny,dtype,bc,stages", CASES)
def test_deep_passes_give_the_marchs_bits(nx, ny, dtype, bc, stages, kind):
    for steps in stages:
        want, march = run(nx, ny, dtype, bc, kind, steps, MARCH)
        got, own = run(nx, ny, dtype, bc, kind, steps, (0, 0, 0, 0))
        assert torch.equal(got, want), (steps, own, march)
