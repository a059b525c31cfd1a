"""Which draft blocks run launches whose workgroups wait for each other (no GPU).

Such a launch finishes only if all of its workgroups are resident, and each of them fills
a compute unit: two that do not fit on the device together can keep each other's
workgroups out until their waits give up and the blocks are invalid.  Small batches, of
which an engine runs several side by side, must not take one.
"""
import ctypes

import pytest

from paper_2607_05147_amd import dspark

CUS = 256
VOCABS = [4, 128, 1000, 4000, 8192, 12416, 16384, 32000, 32768, 50000, 65536, 100000, 129280, 131072, 131076, 262144]


@pytest.fixture(scope="module")
def grid():
    f = dspark.lib()._ZN6dspark16markov_coop_gridEii
    f.argtypes = [ctypes.c_int, ctypes.c_int]
    return f


def test_small_batches_wait_for_no_workgroup(grid):
    for V in VOCABS:
        for R in range(1, 65):
            assert grid(R, V) == 0, (R, V)


def test_large_batches_fit_on_the_device(grid):
    taken = set()
    for V in VOCABS:
        for R in (65, 76, 77, 78, 100, 127, 128, 129, 300, 8192):
            G = grid(R, V)
            assert G in (0, -(-V // 512)) and G <= CUS
            # as many logits as a launch of up to 128 requests needs, a vocabulary that its statistics hold
            assert (G > 0) == (min(R, 128) * V >= 10_000_000 and V <= 131072), (R, V)
            taken.add(G)
    assert len(taken) > 2
