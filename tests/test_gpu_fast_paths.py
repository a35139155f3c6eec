"""Edges of the kernels' shortcuts and tilings, each against the plain form of the same result: remainders,
the smallest and the largest of a range, data that defeats the shortcut."""
import numpy as np
import pytest
import torch

import oracle
from gpu_harness import GpuProblem, dev, e2e_step_check
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


def _searches(A, bits, M, knobs):
    """Grid, levels and objective of the device's search and of the host's."""
    n, d = A.shape
    res = []
    for host in (0, 1):
        knobs(zipml.KNOB_HOST_DP, host)
        p = GpuProblem(A, np.zeros(n, np.float32), bits, 32, n_candidates=M)
        mv = p.make_levels(zipml.OPTIMAL, 0, lo=np.zeros(d), hi=np.ones(d), n_candidates=M, want_mv=True)
        res.append((p.grid.cpu().numpy().copy(), p.levels.cpu().numpy().copy(), mv))
    return res


@pytest.mark.parametrize("M,bits", [(3148, 1), (3149, 1), (2558, 3), (2559, 3), (2046, 4), (2047, 4), (929, 6), (291, 8),
                                    (292, 8)])
def test_level_search_at_the_last_size_that_fits_on_the_chip(M, bits, knobs):
    """Tables that end just below the limit of a workgroup's memory, and the first that do not fit."""
    say("level search at the limit", M, bits)
    u = np.random.default_rng(M).integers(0, 1025, (400, 3))
    u[:, 1] = u[:, 1] ** 2 // 1024
    dev_, host = _searches((u / 1024.0).astype(np.float32), bits, M, knobs)
    assert np.array_equal(dev_[0], host[0]) and np.array_equal(dev_[1], host[1]) and dev_[2] == host[2]


@pytest.mark.parametrize("M,bits", [(2728, 1), (2729, 1), (2273, 3), (2274, 3), (1363, 5), (1364, 5)])
def test_level_search_with_and_without_room_for_pairs(M, bits, knobs):
    """The last size whose tables hold both coefficients of a candidate, and the first that computes one of them."""
    say("level search, room for pairs", M, bits)
    u = np.random.default_rng(M).integers(0, 1025, (400, 3))
    u[:, 1] = u[:, 1] ** 2 // 1024
    u[:, 2] = np.where(u[:, 2] < 600, u[:, 2] // 128 * 128, 1000)
    dev_, host = _searches((u / 1024.0).astype(np.float32), bits, M, knobs)
    assert np.array_equal(dev_[0], host[0]) and np.array_equal(dev_[1], host[1]) and dev_[2] == host[2]


@pytest.mark.parametrize("M,bits", [(929, 4), (930, 4), (1022, 4), (1023, 4), (1135, 3), (1136, 3), (1278, 3), (1279, 3)])
def test_level_search_where_pairs_cost_a_workgroup(M, bits, knobs):
    """The last and the first size at which two workgroups of a compute unit hold both coefficients of a candidate, and
    at which they hold one of them."""
    say("level search, pairs or a second workgroup", M, bits)
    u = np.random.default_rng(M).integers(0, 1025, (400, 3))
    u[:, 1] = u[:, 1] ** 2 // 1024
    u[:, 2] = np.where(u[:, 2] < 600, u[:, 2] // 128 * 128, 1000)
    dev_, host = _searches((u / 1024.0).astype(np.float32), bits, M, knobs)
    assert np.array_equal(dev_[0], host[0]) and np.array_equal(dev_[1], host[1]) and dev_[2] == host[2]


@pytest.mark.parametrize("M,bits", [(100, 2), (513, 3), (1024, 4), (2000, 3)])
def test_pruned_level_search_with_sums_that_round(M, bits, knobs):
    """At most two values to a bin, anywhere inside it: the bin moments do not depend on the order of their sums,
    but everything that the search makes of them is rounded, which is what its margin is for.  Columns: two values
    to every bin, to every third, values crowded at one end, two clusters, almost no variance."""
    say("pruned level search, inexact sums", M, bits)
    rng = np.random.default_rng(M + bits)
    n = 2 * M
    two = np.repeat(np.arange(M), 2)
    def at(bins):
        return (bins + rng.uniform(0.01, 0.99, n)) / M
    cols = [at(two), at(np.where(two % 3 == 0, two, two // 3 * 3)), at(two) ** 6, np.where(at(two) < 0.5, at(two) * 0.01, 1 - at(two) * 0.01),
            0.5 + 1e-7 * at(two)]
    A = np.stack(cols, 1).astype(np.float32)
    # (no more than two to a bin where a column was bent: the others move to the bottom, whose sum is exact)
    for j in range(A.shape[1]):
        t = A[:, j].astype(np.float64)
        m = np.minimum((t * M).astype(int), M - 1)
        for b in np.unique(m):
            rows = np.nonzero(m == b)[0]
            A[rows[2:], j] = 0.0
    dev_, host = _searches(A, bits, M, knobs)
    assert np.array_equal(dev_[0], host[0]) and np.array_equal(dev_[1], host[1]) and dev_[2] == host[2]


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


@pytest.mark.parametrize("n", [16384, 16385])
@pytest.mark.parametrize("d", [479, 480, 481, 512, 513, 961])
def test_loss_through_tables_of_both_chunk_sizes(n, d):
    """3 bits, uneven levels: at 256 compute units chunks of 512 features up to 16,384 samples and of 480 beyond, whole and
    ragged.  The band is that of the test above."""
    rng = np.random.default_rng(n + d)
    say("packed loss, chunks of features", n, d)
    b = rng.standard_normal(n).astype(np.float32)
    x = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    L = np.sort(rng.uniform(-1, 1, (d, 8)), axis=1).astype(np.float32)
    p = GpuProblem(rng.uniform(-1, 1, (n, d)).astype(np.float32), b, 3, 32)
    p.set_levels(L)
    p.quantize(3, 0)
    v = np.take_along_axis(L, p.codes(2).astype(np.int64).T, axis=1).T.astype(np.float64)
    r = v @ x.astype(np.float64) - b
    ref = float(np.sum(r ** 2) / (2 * n))
    mag = float((np.abs(L[:, 0]) + np.abs(L[:, -1] - L[:, 0])).astype(np.float64) @ np.abs(x))
    band = float(np.mean(np.abs(r))) * mag * (d + 4) * 2.0 ** -24
    got = p.loss(dev(x), packed_copy=2)
    assert abs(got - ref) <= band + 1e-7 * ref + 1e-14, (got, ref, band)


@pytest.mark.parametrize("d", [9152, 9153])
def test_loss_through_tables_where_a_second_block_just_fits(d):
    """3 bits, uneven levels, more tiles than compute units: chunks of 480 features as long as the digits of even levels
    leave room for a second block, of 512 beyond.  The band is that of the test above."""
    n = 16385
    rng = np.random.default_rng(d)
    say("packed loss, second block", n, d)
    b = rng.standard_normal(n).astype(np.float32)
    x = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    L = np.sort(rng.uniform(-1, 1, (d, 8)), axis=1).astype(np.float32)
    p = GpuProblem(rng.random((n, d), dtype=np.float32) * np.float32(2) - np.float32(1), b, 3, 32)
    p.set_levels(L)
    p.quantize(3, 0)
    codes = torch.zeros(n, d, dtype=torch.uint8, device="cuda:0")
    zipml.unpack_codes(p.p2, 2, n, d, 3, codes)
    Ld, xd = dev(L).double(), dev(x).double()
    z = torch.zeros(n, dtype=torch.float64, device="cuda:0")
    for j0 in range(0, d, 1024):
        c = codes[:, j0:j0 + 1024].T.long()
        z += xd[j0:j0 + 1024] @ torch.gather(Ld[j0:j0 + 1024], 1, c)
    r = z.cpu().numpy() - b
    ref = float(np.sum(r ** 2) / (2 * n))
    mag = float((np.abs(L[:, 0]) + np.abs(L[:, -1] - L[:, 0])).astype(np.float64) @ np.abs(x))
    band = float(np.mean(np.abs(r))) * mag * (d + 4) * 2.0 ** -24
    got = p.loss(dev(x), packed_copy=2)
    assert abs(got - ref) <= band + 1e-7 * ref + 1e-14, (got, ref, band)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("d", [19904, 19905, 39808, 39809, 39872, 39873])
def test_loss_where_the_digits_of_the_model_just_fit_on_the_chip(d, bits):
    """The widths around which the digits of the model stop fitting in a workgroup's memory: every one has a result.
    Levels on [0, 1] and a model of one sign: no cancellation, the sums are off by (d + 4) 2^-24 at most."""
    say("packed loss of a wide problem", d, bits)
    rng = np.random.default_rng(d + bits)
    n = 70
    A = rng.uniform(0, 1, (n, d)).astype(np.float32)
    x = (rng.uniform(0.5, 1, d) / d).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    p = GpuProblem(A, b, bits, 32)
    p.make_levels(zipml.UNIFORM, 0, lo=np.zeros(d), hi=np.ones(d))
    p.quantize(3, 0)
    ref = oracle.loss_codes(p.codes(2), p.levels.cpu().numpy(), bits, b, x)
    got = p.loss(dev(x), packed_copy=2)
    r = float(np.mean(np.abs(b))) + 1.0
    assert abs(got - ref) <= r * (d + 4) * 2.0 ** -24, (got, ref)


@pytest.mark.parametrize("bits", range(1, 9))
def test_loss_of_small_models_and_of_no_numbers(bits):
    """Model and labels far below one: the loss scales with their square.  An infinite or NaN element ends in a loss
    that is not finite."""
    rng = np.random.default_rng(bits)
    n, d = 200, 512
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    x1, b1 = rng.standard_normal(d) / np.sqrt(d), rng.standard_normal(n)
    L = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    for scale in (1.0, 1e-12, 1e-16, 1e-24, 1e-32):
        say("loss of a small model", bits, scale)
        x, b = (x1 * scale).astype(np.float32), (b1 * scale).astype(np.float32)
        p = GpuProblem(A, b, bits, 32)
        p.set_levels(L)
        p.quantize(3, 0)
        for copy in (1, 2):
            v = np.take_along_axis(L, p.codes(copy).astype(np.int64).T, axis=1).T.astype(np.float64)
            r = v @ x.astype(np.float64) - b
            ref = float(np.sum(r * r) / (2 * n))
            band = float(np.mean(np.abs(r)) * 3.0 * np.abs(x.astype(np.float64)).sum()) * (d + 4) * 2.0 ** -24
            got = p.loss(dev(x), packed_copy=copy)
            assert abs(got - ref) <= band + 1e-7 * ref, (got, ref, band)
    for bad in (np.inf, -np.inf, np.nan):
        x = x1.astype(np.float32)
        x[77] = bad
        say("loss of", bad)
        for copy in (1, 2):
            assert not np.isfinite(p.loss(dev(x), packed_copy=copy))


@pytest.mark.parametrize("large", [1e6, 1e15])
@pytest.mark.parametrize("bits,even", [(b, e) for b in range(1, 9) for e in (True, False) if b > 1 or e])
def test_loss_of_small_products_beside_a_large_one(bits, even, large):
    """One element of the model is 10^6 times the others and meets only the level zero: the dot products are those of
    the others, each to (d + 4) 2^-24 of the sum of its magnitudes.  The labels are the exact dot products, so the
    loss is the mean square of their errors.  Also 10^15 times: more than the digits of the matrix cores span."""
    rng = np.random.default_rng(bits)
    n, d, K = 100, 256, 1 << bits
    x = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    x[100] = large
    A = rng.uniform(0, 1, (n, d)).astype(np.float32)
    A[:, 100] = 0.0
    L = oracle.levels_uniform(np.zeros(d, np.float32), np.ones(d, np.float32), bits)
    if not even:
        L[:, 1:-1] = np.sort(rng.uniform(0, 1, (d, K - 2)), axis=1)
    p = GpuProblem(A, np.zeros(n, np.float32), bits, 32)
    p.set_levels(L)
    p.quantize(3, 0)
    for copy in (1, 2):
        say("small products beside a large one", bits, even, large, copy)
        codes = p.codes(copy)
        assert not codes[:, 100].any()
        v = np.take_along_axis(L, codes.astype(np.int64).T, axis=1).T.astype(np.float64)
        b = (v @ x.astype(np.float64)).astype(np.float32)
        p.b.copy_(dev(b))
        mag = np.abs(v) @ np.abs(x.astype(np.float64))
        got = p.loss(dev(x), packed_copy=copy)
        assert got <= 0.5 * float(np.mean((mag * (d + 4) * 2.0 ** -24) ** 2)), got


@pytest.mark.parametrize("bits", [3, 6, 8])
def test_error_of_long_dot_products_on_copy_1(bits):
    """Root mean square error of the dot products over 16,384 features, against that of 256 fp32 chains of 64 terms
    whose ends are added pairwise: (256 * 64 * 65 / 2 + 6 * 16384 + 9 * 4096) / 16384 = 40.7 squared roundings of an
    rms term each, a rounding at most 2^-24 / sqrt(3) in rms.  The labels are the exact dot products."""
    say("long dot products", bits)
    rng = np.random.default_rng(bits)
    n, d = 512, 16384
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    x = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    p = GpuProblem(A, np.zeros(n, np.float32), bits, 32)
    p.make_levels(zipml.UNIFORM, 0, lo=-np.ones(d), hi=np.ones(d))
    p.quantize(3, 0)
    L = p.levels.cpu().numpy()
    z = np.take_along_axis(L, p.codes(1).astype(np.int64).T, axis=1).T.astype(np.float64) @ x.astype(np.float64)
    p.b.copy_(dev(z.astype(np.float32)))
    own = np.mean((z - z.astype(np.float32)) ** 2)                # the rounding of the labels
    err = np.sqrt(max(0.0, 2.0 * p.loss(dev(x), packed_copy=1) - own)) / np.sqrt(np.mean(z * z))
    assert err <= np.sqrt(40.7 / 3) * 2.0 ** -24, err


def test_loss_on_a_stream_that_is_being_captured_is_refused():
    """Before anything is enqueued: the recording goes on, and holds nothing of the call."""
    say("loss under capture")
    rng = np.random.default_rng(0)
    n, d, bits = 300, 40, 3
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b, xh = rng.standard_normal(n).astype(np.float32), rng.standard_normal(d).astype(np.float32)
    p = GpuProblem(A, b, bits, 32)
    p.make_levels(zipml.UNIFORM, 0, lo=-np.ones(d), hi=np.ones(d))
    p.quantize(3, 0)
    x, t = dev(xh), torch.zeros(64, device="cuda:0")
    ref = [p.loss(x), p.loss(x, 1), p.loss(x, 2)]
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        t.add_(1.0)
        for copy in (0, 1, 2):
            with pytest.raises(zipml.ZipmlError) as e:
                p.loss(x, copy)
            assert e.value.code == zipml.ELAUNCH
    for k in range(3):
        g.replay()
        assert [p.loss(x), p.loss(x, 1), p.loss(x, 2)] == ref
        torch.cuda.synchronize()
        assert bool((t == k + 1).all())


SOLO = [(n, d, B) for n, d, B in [(64, 1, 4), (96, 8, 8), (128, 33, 16), (192, 64, 64), (256, 65, 32), (192, 100, 96), (640, 130, 64),
                                 (640, 255, 160), (512, 256, 256), (1024, 64, 512), (2048, 31, 1024)]]


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("n,d,B", SOLO)
def test_single_workgroup_epochs_of_every_width(n, d, B, bits):
    """Problems of one workgroup: every width, evenly spaced and other levels, batches below a sample group,
    of one block of samples and of several (the last one half full), features of one tile to sixteen; two
    epochs, plain, with the l2 term and with the l1 step."""
    rng = np.random.default_rng(bits * 7919 + n + d + B)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    x0 = (rng.standard_normal(d) / np.sqrt(d)).astype(np.float32)
    b = (A @ x0 + 0.1 * rng.standard_normal(n)).astype(np.float32)
    lo, hi = rng.uniform(-1.5, -1, d).astype(np.float32), rng.uniform(1, 1.5, d).astype(np.float32)
    uneven = np.sort(rng.uniform(-1, 1, (d, 1 << bits)), axis=1).astype(np.float32)
    lr = 0.3 / d
    for L in (oracle.levels_uniform(lo, hi, bits), uneven):
        p = GpuProblem(A, b, bits, B)
        p.set_levels(L)
        p.quantize(5, 0)
        c1, c2 = p.codes(1), p.codes(2)
        args = (p.p1, p.p2, p.levels, p.b, n, d, bits)
        for form in ("plain", "l2", "l1"):
            say("one workgroup", n, d, B, bits, form, L is uneven)
            x, ref = dev(np.zeros(d, np.float32)), np.zeros(d, np.float32)
            for _ in range(2):
                if form == "plain":
                    zipml.sgd_epoch(*args, x, B, lr, p.ws)
                    ref = oracle.sgd_epoch(c1, c2, L, b, bits, ref, B, lr)
                elif form == "l2":
                    zipml.sgd_epoch_l2(*args, x, B, lr, 0.05, p.ws)
                    ref = oracle.sgd_epoch(c1, c2, L, b, bits, ref, B, lr, l2=0.05)
                else:
                    zipml.sgd_epoch_prox(*args, x, B, lr, zipml.PROX_L1, 0.01, p.ws)
                    ref = oracle.sgd_epoch(c1, c2, L, b, bits, ref, B, lr, prox_kind=oracle.PROX_L1, prox_coef=0.01)
            assert zipml.sgd_status(p.ws) == 0
            got = x.cpu().numpy().astype(np.float64)
            # 1e-5: the library's bound for an fp32 model after an epoch
            assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref) + 1e-12
            assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max() + 1e-12


@pytest.mark.parametrize("even", [True, False])
@pytest.mark.parametrize("bits", range(1, 9))
def test_single_workgroup_steps_coordinate_by_coordinate(bits, even):
    """One step from a given model, every coordinate of the gradient on its own: within (d + B + 8) 2^-24 of the sum
    of the magnitudes that reach it.  Some residuals are 10^6 or 10^9 times the others, and half of the features have the
    level zero in those samples; one element of the model is as much larger than the others and meets only zeros."""
    rng = np.random.default_rng(bits + 100 * even)
    K = 1 << bits
    if bits == 1 and not even:
        return                                         # (two levels are evenly spaced)
    for d, B in ((64, 16), (60, 64), (100, 8), (120, 64), (64, 256), (90, 160), (96, 256), (40, 128)):
        for large in (1.0, 1e6, 1e9):
            say("single step", bits, even, d, B, large)
            A = rng.uniform(0, 1, (B, d)).astype(np.float32)
            b = rng.standard_normal(B).astype(np.float32)
            x0 = (rng.standard_normal(d) * 0.1).astype(np.float32)
            rows = np.arange(B) % 16 == 3
            b[rows] *= np.float32(large)
            A[np.ix_(rows, np.arange(d) % 2 == 0)] = 0.0
            A[:, 5] = 0.0
            x0[5] = 0.1 * large
            L = oracle.levels_uniform(np.zeros(d, np.float32), np.ones(d, np.float32), bits)
            if not even:
                L[:, 1:-1] = np.sort(rng.uniform(0, 1, (d, K - 2)), axis=1)
            p = GpuProblem(A, b, bits, B)
            p.set_levels(L)
            p.quantize(3, 0)
            v1, v2 = (np.take_along_axis(L, p.codes(c).astype(np.int64).T, axis=1).T.astype(np.float64) for c in (1, 2))
            x64 = x0.astype(np.float64)
            r = v2 @ x64 - b
            ref = x64 - v1.T @ r / B
            mag = np.abs(x64) + v1.T @ (v2 @ np.abs(x64) + np.abs(b)) / B
            x = dev(x0)
            zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, B, d, bits, x, B, 1.0, p.ws)
            err = np.abs(x.cpu().numpy().astype(np.float64) - ref) / mag
            assert err.max() <= (d + B + 8) * 2.0 ** -24, (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("bits", range(1, 9))
def test_single_workgroup_epochs_of_small_numbers(bits):
    """Labels and model far below one: the epoch is linear in them."""
    rng = np.random.default_rng(bits)
    for d, B, even in ((40, 128, True), (40, 128, False), (64, 16, True), (100, 32, True), (60, 64, False)):
        n = 4 * B
        A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
        b1 = rng.standard_normal(n)
        L = oracle.levels_uniform(np.full(d, -1, np.float32), np.ones(d, np.float32), bits)
        if not even:
            L[:, 1:-1] = np.sort(rng.uniform(-1, 1, (d, (1 << bits) - 2)), axis=1)
        for scale in (1e-22, 1e-26, 1e-30):
            say("small numbers", bits, d, B, even, scale)
            b = (b1 * scale).astype(np.float32)
            p = GpuProblem(A, b, bits, B)
            p.set_levels(L)
            p.quantize(5, 0)
            x = dev(np.zeros(d, np.float32))
            zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, n, d, bits, x, B, 0.1 / d, p.ws)
            got = x.cpu().numpy().astype(np.float64) / scale
            ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, 0.1 / d) / scale
            assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
def test_single_workgroup_epochs_at_the_ends_of_the_number_range(bits):
    """Tiny and huge labels keep their digits, levels whose spacing rounds in fp64 are decoded, and an
    infinite label ends in a model without a finite element (as it does in plain fp32 arithmetic)."""
    n, d, B = 256, 40, 128
    rng = np.random.default_rng(bits)
    L = np.sort(rng.uniform(-1, 1, (d, 1 << bits)), axis=1).astype(np.float32)
    L[:, 0], L[:, -1] = -1.0, 1e-30
    L[:, 1:-1] = np.minimum(L[:, 1:-1], 0.0)
    A = rng.uniform(-1, 0, (n, d)).astype(np.float32)
    for scale in (1e-20, 1.0, 1e30, np.inf):
        say("range", bits, scale)
        b = rng.standard_normal(n).astype(np.float32)
        b = b * np.float32(scale) if np.isfinite(scale) else b
        if not np.isfinite(scale):
            b[7] = np.inf
        p = GpuProblem(A, b, bits, B)
        p.set_levels(np.sort(L, axis=1))
        p.quantize(5, 0)
        x = dev(np.zeros(d, np.float32))
        zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, n, d, bits, x, B, 0.01, p.ws)
        got = x.cpu().numpy().astype(np.float64)
        if not np.isfinite(scale):
            assert not np.isfinite(got).any()
            continue
        ref = oracle.sgd_epoch(p.codes(1), p.codes(2), np.sort(L, axis=1), b, bits, np.zeros(d, np.float32), B, 0.01)
        assert np.linalg.norm(got / scale - ref / scale) <= 1e-5 * np.linalg.norm(ref / scale)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("d,B", [(300, 32), (290, 1024), (1100, 96), (1100, 480), (4000, 96), (4000, 224)])
def test_end_to_end_steps_on_the_matrix_cores(d, B, bits):
    """One, two and four feature groups per workgroup, whole and half blocks of samples, the largest batch;
    uneven levels; labels that spread the residuals over sixty powers of two."""
    say("end-to-end on the matrix cores", d, B, bits)
    rng = np.random.default_rng(bits * 31 + d + B)
    M, n = 200, 2 * B
    G = np.stack([np.sort(rng.choice(M - 1, (1 << bits) - 2, replace=False) + 1) if bits > 1 else np.zeros(0, int)
                  for _ in range(d)])
    G = np.concatenate([np.zeros((d, 1)), G.reshape(d, -1), np.full((d, 1), M)], axis=1).astype(np.uint16)
    L = (G / np.float64(M)).astype(np.float32)
    A = rng.uniform(0, 1, (n, d)).astype(np.float32)
    b = (rng.standard_normal(n) * 2.0 ** rng.uniform(-40, 20, n)).astype(np.float32)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L, G)
    p.quantize(4, 0)
    c1, c2 = p.codes(1), p.codes(2)
    for scale in (0.0, 0.1):
        x0 = (rng.standard_normal(d) * scale).astype(np.float32)
        for step in (0, 1):
            e2e_step_check(p, oracle, c1, c2, L, G, np.float32(0), np.float32(1.0 / M), M, b, x0, 0.3, 8, 8, 4, 0, step,
                           zipml.SGD_PRODUCTION)


@pytest.mark.parametrize("bits", [1, 2, 3, 4])
@pytest.mark.parametrize("d,B", [(300, 32), (290, 256), (4000, 224)])
def test_end_to_end_gradient_is_the_exact_mean(d, B, bits):
    """Levels and residuals of very different size: one level 2^-30 of the largest (all that a feature's codes take in
    half of the columns), residuals over 2^35.  The gradient before its quantisation is the exact mean rounded to
    fp32, element by element (the levels need not lie on the grid that the dot products use)."""
    say("exact mean gradient", d, B, bits)
    rng = np.random.default_rng(bits * 31 + d + B)
    K, M = 1 << bits, 200
    G = np.tile(np.linspace(0, M, K).round().astype(np.uint16), (d, 1))
    L = np.sort(rng.uniform(0.25, 1, (d, K)), axis=1).astype(np.float32)
    L[:, 0] = (rng.uniform(0.5, 1, d) * 2.0 ** -30).astype(np.float32)
    A = rng.uniform(0.3, 1, (B, d)).astype(np.float32)
    A[:, : d // 2] = L[: d // 2, 0]                        # only the smallest level
    b = (rng.standard_normal(B) * 2.0 ** rng.uniform(-35, 0, B)).astype(np.float32)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L, G)
    p.quantize(4, 0)
    c1, c2 = p.codes(1), p.codes(2)
    assert not c1[:, : d // 2].any()
    e2e_step_check(p, oracle, c1, c2, L, G, np.float32(0), np.float32(1.0 / M), M, b, np.zeros(d, np.float32), 0.3, 8, 8,
                   4, 0, 0, zipml.SGD_PRODUCTION)


@pytest.mark.parametrize("bits,d", [(8, 100), (8, 170), (7, 161)])
def test_level_tables_in_memory_are_not_read_past_their_end(bits, d, knobs):
    """Tables too large for LDS, a last feature group with padding features: the rows behind the table (NaN
    here) have no part in the result."""
    say("level table in memory", bits, d)
    n, B = 128, 32
    rng = np.random.default_rng(d)
    L = np.sort(rng.uniform(-1, 1, (d, 1 << bits)), axis=1).astype(np.float32)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L)
    p.quantize(5, 0)
    room = torch.full((d + 64, 1 << bits), float("nan"), device="cuda:0")
    room[:d] = p.levels
    knobs(zipml.KNOB_NO_MATRIX_CORES, 1)
    x = dev(np.zeros(d, np.float32))
    zipml.sgd_epoch(p.p1, p.p2, room[:d], p.b, n, d, bits, x, B, 0.1 / d, p.ws)
    ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, 0.1 / d)
    got = x.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("groups", [2, 9, 64, 65, 70])
@pytest.mark.parametrize("B,bits", [(4, 3), (8, 4), (32, 6), (96, 2), (64, 8), (576, 4)])
def test_epochs_over_exchange_words_of_every_spacing(B, bits, groups, knobs):
    """Both spacings of the exchange words (up to 64 workgroups, and more), sums that end inside and at the end of a
    run of eight words, more steps than exchange buffers; even levels in the loop in which waves own samples (64 features to
    a workgroup, whatever the knob) and in the loops that follow it, uneven levels.  The model of the oracle (fp64 inside
    a step) to 1e-5, the bound of every epoch test."""
    say("spread exchange words", B, bits, groups)
    # (so few groups as two would be one workgroup's: sixteen then, on two workgroups, on eight at 576 samples)
    knobs(zipml.KNOB_TARGET_WORKGROUPS, 2 if groups == 2 else 128)
    d, steps = (16 if groups == 2 else groups) * 32 - 5, 9
    n, K = B * steps, 1 << bits
    rng = np.random.default_rng(B * 100 + groups)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    even = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    uneven = np.sort(rng.uniform(-1, 1, (d, K)), axis=1).astype(np.float32)
    for L in (even, uneven):
        p = GpuProblem(A, b, bits, B)
        p.set_levels(L)
        p.quantize(5, 0)
        lr = 0.25 / d
        ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, lr)
        for xmin in (-1, 1 << 40) if L is even else (-1,):
            knobs(zipml.KNOB_STORE_EXCHANGE_MIN, xmin)
            x = dev(np.zeros(d, np.float32))
            p.epoch(x, lr)
            err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
            assert err <= 1e-5, err


@pytest.mark.parametrize("groups", [33, 64, 65, 128, 129, 257])
@pytest.mark.parametrize("B,bits", [(128, 3), (160, 3), (256, 8), (320, 4)])
def test_epochs_on_both_sides_of_the_numbers_of_workgroups(B, bits, groups):
    """The workgroups that sizes give: either side of 32, 64 and 128 of them and of the units from which more are taken;
    even and uneven levels.  The model of the oracle (fp64 inside a step) to 1e-5, the bound of every epoch test."""
    say("number of workgroups", B, bits, groups)
    d, steps = groups * 32 - 3, 3
    n, K = B * steps, 1 << bits
    rng = np.random.default_rng(B * 100 + groups)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    even = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    uneven = np.sort(rng.uniform(-1, 1, (d, K)), axis=1).astype(np.float32)
    for L in (even, uneven):
        p = GpuProblem(A, b, bits, B)
        p.set_levels(L)
        p.quantize(5, 0)
        x = dev(np.zeros(d, np.float32))
        lr = 0.25 / d
        p.epoch(x, lr)
        ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, lr)
        err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
        assert err <= 1e-5, err


def _averaged(B, d, bits, steps, lr, seed=5):
    """An epoch of the symmetrised estimator on random data and even levels, and the oracle's."""
    n = B * steps
    rng = np.random.default_rng(B * 100 + d)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    L = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L)
    p.quantize(seed, 0)
    p1s, p2s = torch.zeros_like(p.p1), torch.zeros_like(p.p2)
    zipml.quantize_swapped(p.A, n, d, d, 0, n, p.levels, bits, seed, 0, p1s, p2s)
    x = dev(np.zeros(d, np.float32))
    zipml.sgd_epoch_avg(p.p1, p.p2, p1s, p2s, p.levels, p.b, n, d, bits, x, B, lr, p.ws)
    assert zipml.sgd_status(p.ws) == 0
    ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, lr, symmetric=True)
    return x.cpu().numpy().astype(np.float64), ref


@pytest.mark.parametrize("B,d,bits,chunk,steps", [
    (2048, 4100, 8, 0, 3),       # replicas, four feature groups, two units a thread
    (2048, 600, 8, 0, 6),        # replicas, one group, two units
    (512, 4090, 4, 128, 6),      # replicas, four groups, one unit
    (512, 600, 2, 128, 6),       # replicas, one group, one unit
    (512, 2040, 2, 0, 6),        # no replicas: 64 workgroups, one unit
    (1024, 2100, 4, 0, 4),       # 66 workgroups: the wider spacing of the exchange words, two units
    (256, 4100, 4, 0, 5),        # four groups, two units
    (1024, 4100, 2, 0, 3),       # exchange through tagged stores, one group
    (256, 16400, 2, 0, 3),       # the same, four groups
])
def test_symmetrised_epochs_of_every_kernel(B, d, bits, chunk, steps, knobs):
    """The kernels of two code pairs, each by itself.  The model of the oracle (fp64 inside a step) to 1e-5, the bound
    of every epoch test."""
    say("two code pairs", B, d, bits, chunk)
    if chunk:
        knobs(zipml.KNOB_CHUNK_SAMPLES, chunk)
    got, ref = _averaged(B, d, bits, steps, 0.25 / d)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err <= 1e-5, err


@pytest.mark.parametrize("B,d,bits", [(4096, 600, 8), (4096, 1030, 8), (2048, 600, 4), (2048, 4100, 2), (1024, 4100, 4)])
def test_large_epochs_of_one_pair(B, d, bits):
    """Four units a thread, and replicas: one place a lane for its units, or a pointer each.  The bound as above."""
    say("large minibatches", B, d, bits)
    steps = 3
    n = B * steps
    rng = np.random.default_rng(B + d)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    L = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L)
    p.quantize(5, 0)
    x = dev(np.zeros(d, np.float32))
    p.epoch(x, 0.25 / d)
    assert zipml.sgd_status(p.ws) == 0
    ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, 0.25 / d)
    err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    assert err <= 1e-5, err


@pytest.mark.parametrize("B", [64, 128])
@pytest.mark.parametrize("d", [4096, 4097, 8192, 8193, 16390])
def test_symmetrised_epochs_of_small_minibatches_on_wide_problems(B, d):
    """More than 32 workgroups of four feature groups, which eight groups could replace but for the matrix cores."""
    say("two code pairs, wide", B, d)
    got, ref = _averaged(B, d, 4, 5, 0.25 / d)
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err <= 1e-5, err


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("B,d", [(64, 2047), (192, 4100), (256, 290), (256, 2049), (320, 290), (512, 600)])
def test_epochs_on_both_sides_of_the_small_steps(B, d, bits):
    """Up to 256 samples and 64 features a workgroup, and beyond; even and uneven levels.  The bound as above."""
    say("small steps", B, d, bits)
    steps = 6
    n, K = B * steps, 1 << bits
    rng = np.random.default_rng(B + d + bits)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    even = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    for L in (even, np.sort(rng.uniform(-1, 1, (d, K)), axis=1).astype(np.float32)):
        p = GpuProblem(A, b, bits, B)
        p.set_levels(L)
        p.quantize(5, 0)
        x = dev(np.zeros(d, np.float32))
        p.epoch(x, 0.25 / d)
        assert zipml.sgd_status(p.ws) == 0
        ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, 0.25 / d)
        err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
        assert err <= 1e-5, err


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("B,d,steps", [
    (4, 290, 21), (8, 600, 5), (16, 1000, 3), (32, 257, 20), (64, 320, 1), (64, 2100, 35), (96, 1030, 2), (160, 4100, 3),
    (256, 2060, 17), (320, 8200, 2), (512, 300, 2), (512, 4130, 2), (544, 700, 3), (992, 1100, 2), (1024, 2080, 2)])
def test_epochs_with_samples_owned_by_waves(B, d, steps, bits):
    """Minibatches inside a group of 32 samples, of odd numbers of groups, of one wave, of all eight and of two blocks a wave;
    a last workgroup with one group of features; one, two and four exchange words a sample; steps before, at and after the
    refresh of the bounds; copy 1 requested at either place.  The model of the oracle (fp64 inside a step) to 1e-5, the
    bound of every epoch test; the preparation's flags say that the levels count as even, so that the loop runs (two levels
    whose difference is not a fp32 number among them)."""
    say("waves own samples", B, d, steps, bits)
    n = B * steps
    rng = np.random.default_rng(B + d + bits)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    x0 = (rng.standard_normal(d) / d ** 0.5).astype(np.float32)
    L = oracle.levels_uniform(-rng.uniform(0.5, 1, d).astype(np.float32), rng.uniform(0.5, 1, d).astype(np.float32), bits)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L)
    p.quantize(5, 0)
    lr = 0.25 / d
    for form in ("plain", "l2", "prox"):
        x, ref = dev(x0), x0.copy()
        args = (p.p1, p.p2, p.levels, p.b, n, d, bits)
        if form == "plain":
            zipml.sgd_epoch(*args, x, B, lr, p.ws)
            ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, ref, B, lr)
            assert p.ws[5120:5120 + 4 * 64].view(torch.int32).all()      # Workspace::kEven, kEvenBlocks
        elif form == "l2":
            zipml.sgd_epoch_l2(*args, x, B, lr, 0.05, p.ws)
            ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, ref, B, lr, l2=0.05)
        else:
            zipml.sgd_epoch_prox(*args, x, B, lr, zipml.PROX_L1, 0.01, p.ws)
            ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, ref, B, lr, prox_kind=oracle.PROX_L1, prox_coef=0.01)
        assert zipml.sgd_status(p.ws) == 0
        got = x.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - ref) <= 1e-5 * np.linalg.norm(ref)
        if d * n > 1 << 21:
            break                                      # (the oracle's time)


@pytest.mark.parametrize("bits", range(1, 9))
def test_steps_with_samples_owned_by_waves_coordinate_by_coordinate(bits):
    """One step from a given model at the widths and sizes that the vector loop computed in fp32 (2, 4 and 8 bits: minibatches
    that are not whole blocks of 64 samples), every coordinate of the
    gradient on its own: within (d + B + 8) 2^-24 of the sum of the magnitudes that reach it.  Some residuals are 10^6 or
    10^9 times the others, and half of the features have the level zero in those samples; one element of the model is 10^6
    times the others and meets only zeros (2^-42 of it is what the exchange resolves)."""
    rng = np.random.default_rng(bits)
    sizes = ((290, 64), (1000, 16), (520, 96), (300, 256), (300, 576)) if bits in (1, 3, 5, 6, 7) else ((1000, 16), (290, 32), (520, 96), (300, 288), (300, 608))
    for d, B in sizes:
        for large in (1.0, 1e6, 1e9):
            say("single step of waves", bits, d, B, large)
            A = rng.uniform(0, 1, (B, d)).astype(np.float32)
            b = rng.standard_normal(B).astype(np.float32)
            x0 = (rng.standard_normal(d) * 0.1).astype(np.float32)
            rows = np.arange(B) % 16 == 3
            b[rows] *= np.float32(large)
            A[np.ix_(rows, np.arange(d) % 2 == 0)] = 0.0
            A[:, 5] = 0.0
            x0[5] = 0.1 * min(large, 1e6)
            L = oracle.levels_uniform(np.zeros(d, np.float32), np.ones(d, np.float32), bits)
            p = GpuProblem(A, b, bits, B)
            p.set_levels(L)
            p.quantize(3, 0)
            v1, v2 = (np.take_along_axis(L, p.codes(c).astype(np.int64).T, axis=1).T.astype(np.float64) for c in (1, 2))
            x64 = x0.astype(np.float64)
            ref = x64 - v1.T @ (v2 @ x64 - b) / B
            mag = np.abs(x64) + v1.T @ (v2 @ np.abs(x64) + np.abs(b)) / B
            x = dev(x0)
            zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, B, d, bits, x, B, 1.0, p.ws)
            err = np.abs(x.cpu().numpy().astype(np.float64) - ref) / mag
            assert err.max() <= (d + B + 8) * 2.0 ** -24, (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("d", [16384, 16385, 20000])
@pytest.mark.parametrize("B,bits", [(64, 8), (96, 4), (256, 2), (512, 4), (512, 8)])
def test_epochs_on_both_sides_of_the_widest_problems(d, B, bits):
    """Up to 256 workgroups of 64 features waves own samples; on more features the matrix-core loop runs, with the reducers
    and the workgroups that read ahead that the library chooses from 128 workgroups x 256 samples on, and the vector loop on
    minibatches that are not whole blocks of 64.  Even and uneven levels; the model of the oracle (fp64 inside a step) to
    1e-5, the bound of every epoch test."""
    say("widest problems", d, B, bits)
    n, K = 3 * B, 1 << bits
    rng = np.random.default_rng(d + B + bits)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    for even in (True, False):
        L = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
        if not even:
            L[d - 1] = np.sort(rng.uniform(-1, 1, K)).astype(np.float32)
        p = GpuProblem(A, b, bits, B)
        p.set_levels(L)
        p.quantize(5, 0)
        x = dev(np.zeros(d, np.float32))
        p.epoch(x, 0.25 / d)
        ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, 0.25 / d)
        err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
        assert err <= 1e-5, err


@pytest.mark.parametrize("n", [58_719_744, 58_720_256])
def test_step_at_the_end_of_the_largest_copies(n):
    """Offsets of codes at the last multiple of a minibatch for which two groups of a copy lie within 7 * 2^29 bytes, and
    beyond, where the matrix-core loop runs.  Only the last 1,024 samples are written; the last step's residuals and
    gradient against fp64, to 1e-5 like every production step."""
    say("largest copies", n)
    d, bits, B, rows = 290, 8, 512, 1024
    groups = (d + 31) // 32
    rng = np.random.default_rng(n)
    A = rng.uniform(-1, 1, (rows, d)).astype(np.float32)
    b = rng.standard_normal(rows).astype(np.float32)
    x0 = (rng.standard_normal(d) / d ** 0.5).astype(np.float32)
    L = oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits)
    p1, p2 = (torch.empty(zipml.packed_bytes(n, d, bits), dtype=torch.uint8, device="cuda:0") for _ in (1, 2))
    labels = torch.empty(n, dtype=torch.float32, device="cuda:0")
    labels[n - rows:] = dev(b)
    levels = dev(L)
    ws = torch.zeros(zipml.workspace_bytes(n, d, bits, B), dtype=torch.uint8, device="cuda:0")
    zipml.quantize(dev(A), rows, d, d, n - rows, n, levels, bits, 3, 0, p1, p2)
    # (copy 2: samples x 32 features in a group; copy 1: groups of 32 samples, 32 features x 32 samples in each)
    c2 = p2.view(groups, n, 32)[:, n - B:].permute(1, 0, 2).reshape(B, groups * 32)[:, :d].cpu().numpy()
    c1 = p1.view(groups, n // 32, 32, 32)[:, (n - B) // 32:].permute(1, 3, 0, 2).reshape(B, groups * 32)[:, :d].cpu().numpy()
    v1, v2 = (np.take_along_axis(L.T, c.astype(np.int64), axis=0).astype(np.float64) for c in (c1, c2))
    r_ref = v2 @ x0.astype(np.float64) - b[rows - B:]
    g_ref = v1.T @ r_ref / B
    x = dev(x0)
    r, g = torch.zeros(B, device="cuda:0"), torch.zeros(d, device="cuda:0")
    zipml.debug_step(p1, p2, levels, labels, n, d, bits, x, B, 0.05, n // B - 1, ws, r=r, g=g, flags=zipml.SGD_PRODUCTION)
    assert zipml.sgd_status(ws) == 0
    for got, want in ((r, r_ref), (g, g_ref), (x, x0 - np.float32(0.05) * g_ref)):
        assert np.linalg.norm(got.cpu().numpy().astype(np.float64) - want) <= 1e-5 * np.linalg.norm(want)


@pytest.mark.parametrize("d,B,bits", [(8192, 64, 2), (8192, 256, 4), (16384, 128, 2), (16384, 512, 4)])
def test_digits_of_the_model_behind_a_refresh_of_the_bounds(d, B, bits):
    """The refreshed bound of y is the sum of the maxima of W workgroups of 64 features, and half as many of 128 features
    would have half the sum: y is to be resolved as finely as there, to 2^-30 of the power of two above that sum.  All
    elements of the model are 1.25 and that unit, which half the resolution would round the same way in every product.  17
    minibatches of zeros leave the model as it is and refresh the bounds; the next step's model, relative to itself in L2:
    fp32 roundings of z, the gradient and the model, at most 2^-24 each and of either sign, below 2^-23 in all, against
    2^-21 / 1.25 (16,384 features) and 2^-22 / 1.25 with half the resolution."""
    say("digits of y", d, B, bits)
    K, W = 1 << bits, d // 64
    unit = 2.0 ** (int(np.ceil(np.log2(W * 1.25 * 1.001))) - 30)
    rng = np.random.default_rng(d + B + bits)
    A = np.zeros((18 * B, d), np.float32)
    A[17 * B:] = rng.uniform(0, K - 1, (B, d))
    x0 = np.full(d, 1.25 + unit, np.float32)
    L = oracle.levels_uniform(np.zeros(d, np.float32), np.full(d, K - 1, np.float32), bits)
    p = GpuProblem(A, np.zeros(18 * B, np.float32), bits, B)
    p.set_levels(L)
    p.quantize(3, 0)
    c1, c2 = (p.codes(c)[17 * B:].astype(np.float64) for c in (1, 2))
    ref = x0.astype(np.float64) - c1.T @ (c2 @ x0.astype(np.float64)) / B
    x = dev(x0)
    zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, 18 * B, d, bits, x, B, 1.0, p.ws)
    assert zipml.sgd_status(p.ws) == 0
    err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    say("error", err)
    assert err <= 2.0 ** -23, err


@pytest.mark.parametrize("bits", range(1, 9))
def test_epochs_with_samples_owned_by_waves_at_the_ends_of_the_number_range(bits):
    """Tiny and huge labels keep their digits; an infinite label, and one that is no number, end in a model without a
    finite element."""
    n, d, B = 288, 300, 96
    rng = np.random.default_rng(bits)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    L = oracle.levels_uniform(np.full(d, -1, np.float32), np.ones(d, np.float32), bits)
    for scale in (1e-30, 1e-20, 1.0, 1e30, np.inf, np.nan):
        say("range of waves", bits, scale)
        b = rng.standard_normal(n).astype(np.float32)
        if np.isfinite(scale):
            b *= np.float32(scale)
        else:
            b[7] = scale
        p = GpuProblem(A, b, bits, B)
        p.set_levels(L)
        p.quantize(5, 0)
        x = dev(np.zeros(d, np.float32))
        zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, n, d, bits, x, B, 0.1 / d, p.ws)
        assert zipml.sgd_status(p.ws) == 0
        got = x.cpu().numpy().astype(np.float64)
        if not np.isfinite(scale):
            assert not np.isfinite(got).any()
            continue
        ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, np.zeros(d, np.float32), B, 0.1 / d)
        assert np.linalg.norm(got / scale - ref / scale) <= 1e-5 * np.linalg.norm(ref / scale)


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("d,B", [(60, 16), (100, 256), (300, 96), (300, 64), (2100, 256)])
def test_epochs_on_levels_that_descend(d, B, bits):
    """Evenly spaced levels from the highest to the lowest, on one workgroup and on several: the bounds of y are of
    magnitudes, at the launch and from step to step (one workgroup begins at a model of zeros).  The model of the oracle (fp64
    inside a step) to 1e-5, the bound of every epoch test."""
    say("descending levels", d, B, bits)
    n = 3 * B
    rng = np.random.default_rng(d + B + bits)
    A = rng.uniform(-1, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    x0 = (rng.standard_normal(d) / d ** 0.5).astype(np.float32) if d > 256 else np.zeros(d, np.float32)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(oracle.levels_uniform(np.full(d, -1, np.float32), np.full(d, 1, np.float32), bits))
    p.quantize(5, 0)
    L = oracle.levels_uniform(np.full(d, 1, np.float32), np.full(d, -1, np.float32), bits)
    p.set_levels(L)
    x = dev(x0)
    zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, n, d, bits, x, B, 0.25 / d, p.ws)
    assert zipml.sgd_status(p.ws) == 0
    ref = oracle.sgd_epoch(p.codes(1), p.codes(2), L, b, bits, x0.copy(), B, 0.25 / d)
    err = np.linalg.norm(x.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    assert err <= 1e-5, err


@pytest.mark.parametrize("d,B,bits", [(2111, 512, 3), (4030, 512, 2), (4095, 32, 1), (4100, 480, 3), (2111, 96, 3), (8190, 96, 3)])
def test_end_to_end_epochs_with_the_dot_pass_on_the_matrix_cores(d, B, bits):
    """Grid indices from a lowest one that is not zero up to thousands, an odd last group of features, whole and half blocks of
    samples, one and two exchange words a sample.  The integers of a step are the oracle's, and an epoch of more steps than
    exchange buffers is that of its steps launched one by one, bit for bit."""
    say("end-to-end dot pass", d, B, bits)
    rng = np.random.default_rng(d + B + bits)
    K, M, n = 1 << bits, 1900, 9 * B
    G = np.sort(np.stack([rng.choice(M, K, replace=False) + 1 for _ in range(d)]), axis=1).astype(np.uint16)
    L = (G / np.float64(M)).astype(np.float32)
    A = rng.uniform(0, 1, (n, d)).astype(np.float32)
    b = rng.standard_normal(n).astype(np.float32)
    x0 = (rng.standard_normal(d) * 0.1).astype(np.float32)
    p = GpuProblem(A, b, bits, B)
    p.set_levels(L, G)
    p.quantize(4, 0)
    e2e_step_check(p, oracle, p.codes(1)[:2 * B], p.codes(2)[:2 * B], L, G, np.float32(0), np.float32(1.0 / M), M, b, x0, 0.3, 8, 8,
                   4, 0, 1, zipml.SGD_PRODUCTION)
    kw = dict(grid_idx=p.grid, grid_lo=0.0, grid_step=1.0 / M, grid_max=M, grad_bits=8, model_bits=8, seed=4, epoch=0)
    x, y = dev(x0), dev(x0)
    zipml.sgd_epoch(p.p1, p.p2, p.levels, p.b, n, d, bits, x, B, 0.01, p.ws, **kw)
    assert zipml.sgd_status(p.ws) == 0
    r = torch.zeros(B, dtype=torch.float32, device=y.device)
    for step in range(9):
        zipml.debug_step(p.p1, p.p2, p.levels, p.b, n, d, bits, y, B, 0.01, step, p.ws, flags=zipml.SGD_PRODUCTION, r=r, **kw)
    assert torch.equal(x, y)


@pytest.mark.parametrize("d,B,bits", [(2999, 128, 4), (2999, 128, 3), (2999, 128, 2), (4523, 160, 5), (2047, 512, 4), (300, 96, 4), (4097, 96, 4)])
def test_end_to_end_epochs_by_the_forms_of_the_norm_exchange(d, B, bits):
    """One and two waves that own features, levels beyond the matrix cores, one and two exchange words a sample: likewise."""
    test_end_to_end_epochs_with_the_dot_pass_on_the_matrix_cores(d, B, bits)
