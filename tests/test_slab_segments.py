"""Plane pairs per tile of the 3D slab march: the least cost over all segment counts, found
without trying each (host logic; long thin meshes have up to 2^28 counts)."""
import ctypes
import time

import numpy as np
import pytest

import paper_1208_2407_amd as tsq


@pytest.fixture(scope="module")
def rule():
    # tsq::slab_segment_pairs(columns, pairs, stages, cus)
    f = ctypes.CDLL(tsq.library_path())._ZN3tsq18slab_segment_pairsExxix
    f.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong]
    f.restype = ctypes.c_longlong
    return f


def least(columns, pairs, stages, cus):
    segs = np.arange(1, pairs + 1, dtype=np.int64)
    q = (pairs + segs - 1) // segs
    tiles = columns * ((pairs + q - 1) // q)
    cost = ((tiles + cus - 1) // cus) * (q + 2 * stages - 1) + (tiles * (q + 2 * stages)) / cus
    return int(q[np.argmin(cost)])


def test_the_least_cost_of_all_counts(rule):
    rng = np.random.default_rng(5)
    for _ in range(3000):
        columns, pairs = (int(np.exp(rng.uniform(0, np.log(most)))) for most in (3000, 20000))
        stages, cus = int(rng.integers(1, 3)), int(rng.choice([32, 256, 304]))
        assert rule(columns, pairs, stages, cus) == least(columns, pairs, stages, cus), (columns, pairs, stages, cus)


def test_long_meshes_take_no_time(rule):
    t0 = time.perf_counter()
    for pairs in (1 << 15, 500000, 5 * 10 ** 7, 1 << 28):
        for stages in (1, 2):
            assert 1 <= rule(1, pairs, stages, 256) <= pairs
    assert time.perf_counter() - t0 < 0.1  # each of the counts in turn takes seconds
