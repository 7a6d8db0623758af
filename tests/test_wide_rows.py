"""Rows of more than 4 GiB: one instance of the complex64 march addresses a lane's site by a
32-bit byte offset within its row, so meshes wider than 2^29 sites (only 2 rows of them
make a legal plan) must not take it.  Which passes do is host logic; on the GPU such a
mesh holds two packets, one across column 2^29 and one across the wrap, each of which
must evolve as on a small mesh, to the bit, with exact zeros elsewhere."""
import ctypes
import itertools

import pytest
import torch

import paper_1208_2407_amd as tsq

EDGE = 1 << 29


def test_rows_beyond_the_lane_offsets_keep_lane_addresses():
    # tsq::march_phase_lds(dtype, nx, steps, last, pairs_per_lane, phase_lds)
    rule = ctypes.CDLL(tsq.library_path())._ZN3tsq15march_phase_ldsEiiibib
    rule.argtypes = [ctypes.c_int] * 3 + [ctypes.c_bool, ctypes.c_int, ctypes.c_bool]
    rule.restype = ctypes.c_bool
    for nx in (2, 4096, EDGE - 2, EDGE, EDGE + 2, 2 * EDGE - 2):
        wide = (nx - 2) * 8 >= 1 << 32
        assert wide == (nx > EDGE)
        for dtype, S, last, ppl, lds in itertools.product((0, 1), range(1, 9), (False, True), (1, 2), (False, True)):
            scalar_rows = dtype == 0 and S == 6 and last and ppl == 1 and not lds
            assert rule(dtype, nx, S, last, ppl, lds) == (lds or (wide and scalar_rows))
    # the longest legal row: two of them make 2^31 - 4 sites
    tsq.Plan(2 * EDGE - 2, 2, 0.05, "c64")


@pytest.mark.gpu
def test_wide_mesh_evolves_as_small_ones():
    nx, ny, W, steps = EDGE + 4096, 2, 1024, 12  # light cone: 2 * 12 + 1 columns per side
    gen = torch.Generator().manual_seed(7)
    psi0 = torch.zeros(ny, W, dtype=torch.complex64)
    psi0[:, 64:-64] = torch.randn(ny, W - 128, dtype=torch.complex64, generator=gen)
    V0 = torch.rand(ny, W, dtype=torch.float64, generator=gen)
    starts = (EDGE - W // 2, nx - W // 2)  # the second wraps

    def window(x, x0):
        return torch.cat([x[:, x0:x0 + W], x[:, :max(0, x0 + W - nx)]], 1)

    psi = torch.zeros(ny, nx, dtype=torch.complex64, device="cuda")
    V = torch.zeros(ny, nx, dtype=torch.float64, device="cuda")
    plan = tsq.Plan(nx, ny, 0.11, "c64", dx=1.3, dy=0.8)
    small = tsq.Plan(W, ny, 0.11, "c64", dx=1.3, dy=0.8)
    small.set_potential(V0.cuda())
    for x0 in starts:
        n = min(W, nx - x0)
        V[:, x0:x0 + n], V[:, :W - n] = V0[:, :n].cuda(), V0[:, n:].cuda() if n < W else 0.0
    plan.set_potential(V)
    for schedule in ((0, 0, 0, 0), (6, 0, 1, 1), (8, 0, 1, 2), (3, 0, 2, 1), (1, 0, 1, 1)):
        psi.zero_()
        for x0 in starts:
            n = min(W, nx - x0)
            psi[:, x0:x0 + n] = psi0[:, :n].cuda()
            if n < W:
                psi[:, :W - n] = psi0[:, n:].cuda()
        want = psi0.cuda()
        for p, x in ((plan, psi), (small, want)):
            p.set_schedule(*schedule)
            p.evolve(x, steps)
        for x0 in starts:
            assert torch.equal(window(psi, x0), want), (schedule, x0)
            n = min(W, nx - x0)
            psi[:, x0:x0 + n] = 0
            if n < W:
                psi[:, :W - n] = 0
        assert not torch.view_as_real(psi).any(), schedule  # nothing outside the windows
