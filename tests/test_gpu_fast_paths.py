"""Edges of the kernels' shortcuts and tilings, each against the plain form of the same result: remainders,
the smallest and the largest of a range, data that defeats the shortcut."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import GpuProblem, dev
from paper_1611_05402_amd import synth, zipml

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.mark.parametrize("M,bits", [(1, 1), (7, 3), (64, 2), (65, 4), (511, 3), (512, 5), (513, 3), (1023, 2), (1024, 4),
                                    (1500, 3)])
def test_pruned_level_search_equals_the_full_one(M, bits, knobs):
    """The device's dynamic program tries only the candidates that can be the best one; the host's tries all.
    Values are multiples of 2^-10 on [0, 1], so the bin moments are exact and both see the same numbers.
    Columns: even, skewed, mostly zero, constant, two values, a hole in the middle, integers of one bin apart."""
    say("pruned level search", M, bits)
    rng = np.random.default_rng(M)
    n = 700
    u = rng.integers(0, 1025, n)
    cols = [u, (u * u) // 1024, np.where(rng.random(n) < 0.95, 0, u), np.full(n, 512), np.where(u < 300, 100, 900),
            np.where((u > 200) & (u < 800), 1024 - u // 8, u), (u // 64) * 64]
    A = (np.stack(cols, 1) / 1024.0).astype(np.float32)
    d = A.shape[1]
    res = []
    for host in (0, 1):
        knobs(zipml.KNOB_HOST_DP, host)
        p = GpuProblem(A, np.zeros(n, np.float32), bits, 32, n_candidates=M)
        mv = p.make_levels(zipml.OPTIMAL, 0, lo=np.zeros(d), hi=np.ones(d), n_candidates=M, want_mv=True)
        res.append((p.grid.cpu().numpy().copy(), p.levels.cpu().numpy().copy(), mv))
    assert np.array_equal(res[0][0], res[1][0])
    assert np.array_equal(res[0][1], res[1][1])
    assert res[0][2] == res[1][2]
