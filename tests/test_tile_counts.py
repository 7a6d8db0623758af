"""Pass counts of the tile kernels up to the largest step counts the type holds."""
import pytest

import paper_1208_2407_amd as tsq


@pytest.mark.parametrize("n", [64, 300])
def test_pass_counts_of_huge_evolutions(n):
    plan = tsq.Plan(n, n, 0.05, "c64")
    for steps in (10 ** 12, 2 ** 62, 2 ** 63 - 20, 2 ** 63 - 8, 2 ** 63 - 2, 2 ** 63 - 1):
        passes, copy_back = plan.passes(steps)
        assert passes % 2 == 0 and not copy_back
        assert steps / 15 <= passes <= steps / 2
