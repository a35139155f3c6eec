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


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("n,d", [(1, 1), (63, 31), (130, 32), (129, 33), (700, 65), (40000, 96), (2051, 1030)])
def test_loss_on_packed_copies_of_every_width(n, d, bits):
    """Both copies, levels evenly spaced (matrix cores on copy 2) and not (tables in LDS, several chunks of
    features at 1,030): ragged tiles of samples, odd numbers of feature groups, fewer and more samples than
    blocks.  A dot product is off by at most (d + 4) 2^-24 times the sum of
    the magnitudes, for evenly spaced levels those of the two terms lo_j x_j and (hi_j - lo_j) x_j."""
    rng = np.random.default_rng(bits * 1000 + n + d)
    K = 1 << bits
    b = rng.standard_normal(n).astype(np.float32)
    x = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    lo, hi = rng.uniform(-2, -1, d).astype(np.float32), rng.uniform(1, 2, d).astype(np.float32)
    even = oracle.levels_uniform(lo, hi, bits)
    uneven = np.sort(rng.uniform(-1, 1, (d, K)), axis=1).astype(np.float32)
    for L in (even, uneven):
        p = GpuProblem(A, b, bits, 32)
        p.set_levels(L)
        p.quantize(3, 0)
        for copy in (1, 2):
            say("packed loss", n, d, bits, copy, L is even)
            v = np.take_along_axis(L, p.codes(copy).astype(np.int64).T, axis=1).T.astype(np.float64)
            ref = float(np.sum((v @ x.astype(np.float64) - b) ** 2) / (2 * n))
            # the loss moves by the mean of |r| times the error of a dot product
            mag = float((np.abs(L[:, 0]) + np.abs(L[:, -1] - L[:, 0])).astype(np.float64) @ np.abs(x))
            band = float(np.mean(np.abs(v @ x - b))) * mag * (d + 4) * 2.0 ** -24
            got = p.loss(dev(x), packed_copy=copy)
            assert abs(got - ref) <= band + 1e-7 * ref + 1e-14, (got, ref, band)
