"""tsq_evolve_passes is host only: counting the passes of a small mesh, which may be the
tile kernels', opens no device (in a process of its own, before anything else does)."""
import os
import subprocess
import sys

import pytest

import paper_1208_2407_amd as tsq

CODE = """
import ctypes, os, sys
lib = ctypes.CDLL(sys.argv[1])

class Problem(ctypes.Structure):
    _fields_ = ([(n, ctypes.c_int32) for n in ("nx", "ny")]
                + [(n, ctypes.c_double) for n in ("dx", "dy", "mass", "hbar", "dt")]
                + [(n, ctypes.c_int32) for n in ("bc", "dtype", "order", "nz")] + [("dz", ctypes.c_double)])

def devices():
    links = []
    for fd in os.listdir("/proc/self/fd"):
        try:
            links.append(os.readlink("/proc/self/fd/" + fd))
        except OSError:
            pass
    return [x for x in links if x.startswith("/dev/kfd") or x.startswith("/dev/dri")]

for nx in (64, 256, 1030, 4096):
    for dtype in (0, 1):
        for bc, order, nz in ((0, 2, 0), (1, 2, 0), (0, 4, 0), (0, 2, 64)):
            if nz and nx > 256:
                continue
            plan, passes, copy = ctypes.c_void_p(), ctypes.c_int64(), ctypes.c_int32()
            p = Problem(nx, nx, 1.0, 1.0, 1.0, 1.0, 0.05, bc, dtype, order, nz, 1.0)
            assert lib.tsq_plan_create(ctypes.byref(p), ctypes.byref(plan)) == 0
            assert lib.tsq_evolve_passes(plan, ctypes.c_int64(100), ctypes.byref(passes), ctypes.byref(copy)) == 0
            print(nx, dtype, bc, order, nz, passes.value)
print("open:", devices())
"""


def run():
    out = subprocess.run([sys.executable, "-c", CODE, tsq.library_path()], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr
    return out.stdout


def test_counts_are_the_plans():
    for line in run().splitlines()[:-1]:
        nx, dtype, bc, order, nz, passes = map(int, line.split())
        plan = tsq.Plan(nx, nx, 0.05, ("c64", "c128")[dtype], bc=("periodic", "closed")[bc], order=order, nz=nz)
        assert plan.passes(100)[0] == passes, line


@pytest.mark.gpu
def test_counting_passes_opens_no_device():
    assert os.path.exists("/dev/kfd")
    assert run().splitlines()[-1] == "open: []"
