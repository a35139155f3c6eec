"""The workloads by which this library's speed is judged, through its public entry points.

A case is one call sequence of a user's program on one problem shape:

  epoch     zipml.sgd_epoch (or its l2 / proximal / symmetrised form): one pass of double-sampled
            minibatch SGD over the resident packed copies; the model goes on from pass to pass
  levels    zipml.levels: variance-optimal or greedy levels of a fp32 matrix, its column ranges included
  quantize  zipml.levels (column ranges, uniform levels) and zipml.quantize: a fp32 matrix becomes
            the two packed copies
  loss      zipml.loss on the fp32 rows or on a packed copy, as a training loop calls it after an epoch

``listed()`` names the fixed cases, ``draw()`` gives further ones from the ranges they stand for.
"""
from __future__ import annotations

import math

import torch

from paper_1611_05402_amd import zipml


def _epoch(name, n, d, bits, batch, data="uniform", levels="fixed", lr=0.0, form="plain", model_bits=0, candidates=0):
    c = {"op": "epoch", "n": n, "d": d, "bits": bits, "batch": batch, "data": data, "levels": levels, "lr": lr,
         "form": form, "model_bits": model_bits, "candidates": candidates}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest training job: 256 steps of 16 samples, everything fits one compute unit
        _epoch("epoch_tiny_4bit_b16", 4096, 64, 4, 16, lr=0.01),
        # ordinary dense least squares at the batch size the paper recommends
        _epoch("epoch_dense_8bit_b256", 65536, 2048, 8, 256, data="gauss", lr=1e-3),
        # many samples, few features, lowest precision, columns of different range
        _epoch("epoch_lowbit_2bit_b1024", 1048576, 512, 2, 1024, data="columns", levels="columns", lr=0.2),
        # the largest problem: tomography-shaped rows, 4 GiB of codes an epoch
        _epoch("epoch_tomo_4bit_b512", 262144, 16384, 4, 512, data="sparse", levels="unit", lr=1.0),
        # end to end in low precision: variance-optimal levels, model and gradient in 8 bits
        _epoch("epoch_end_to_end_3bit", 524288, 4096, 3, 512, data="lognormal", levels="optimal", lr=0.5, model_bits=8,
               candidates=1024),
        # gradient descent: one step over all samples, 2 GiB of codes
        _epoch("epoch_full_batch_8bit", 524288, 2048, 8, 524288, data="gauss", lr=0.05),
        # a narrow regression set (90 columns) with data-only quantisation on variance-optimal levels
        _epoch("epoch_narrow_optimal_3bit", 131072, 90, 3, 256, data="lognormal", levels="optimal", candidates=256),
        # two-class least-squares SVM on 1,000 columns (a ragged width) at one of the widths the paper finds sufficient
        _epoch("epoch_svm_6bit_b64", 65536, 1000, 6, 64, data="gauss", form="l2"),
        # the level search that comes before training on optimal levels
        {"name": "levels_optimal_3bit", "op": "levels", "n": 65536, "d": 2048, "bits": 3, "mode": "optimal",
         "candidates": 1024, "data": "lognormal"},
        # a data set prepared for training: ranges, levels, both copies
        {"name": "quantize_8bit", "op": "quantize", "n": 65536, "d": 2048, "bits": 8, "data": "gauss"},
        # the smallest call: the loss of the tiny job after an epoch
        {"name": "loss_rows_tiny", "op": "loss", "n": 4096, "d": 64, "bits": 4, "on": "rows", "data": "uniform",
         "levels": "fixed", "candidates": 0},
        # the loss on the data as it is stored for training when the fp32 rows are gone
        {"name": "loss_packed_optimal_3bit", "op": "loss", "n": 131072, "d": 4096, "bits": 3, "on": "copy 2",
         "data": "lognormal", "levels": "optimal", "candidates": 1024},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(["epoch", "full", "end_to_end", "levels", "quantize", "loss"], [6, 1, 1, 1, 1.5, 1.5])[0]
    bits = rng.choice([1, 2, 2, 3, 4, 4, 5, 6, 7, 8, 8])
    if op == "epoch":
        d = _log(rng, 8, 16384)
        batch = rng.choice([4, 8, 16]) if rng.random() < 0.15 else 32 * _log(rng, 1, 32)
        steps = _log(rng, 32, 512)
        while steps * batch * d * bits > 1 << 32:          # at most 1 GiB of codes
            steps //= 2
        data, levels = rng.choice([("uniform", "fixed"), ("gauss", "fixed"), ("gauss", "columns"), ("columns", "columns"),
                                   ("sparse", "unit"), ("lognormal", "optimal")])
        if levels == "optimal" and bits > 5:               # (so many levels are not worth a search)
            bits = 3
        form = rng.choice(["plain", "plain", "plain", "l2", "prox", "average"])
        if form == "average" and (levels == "optimal" or bits not in (2, 4, 8) or batch % 64 or d <= 256):
            form = "plain"                                 # (the symmetrised form is built for these)
        cand = max(64, 1 << (bits + 2)) if levels == "optimal" else 0
        return _epoch(None, max(1, steps) * batch, d, bits, batch, data, levels, form=form, candidates=cand)
    if op == "full":                                       # minibatches of thousands to hundreds of thousands of samples
        bits = rng.choice([2, 4, 8])
        d = _log(rng, 300, 8192)
        batch = 64 * _log(rng, 512, 4096)
        while batch * d * bits > 1 << 33:
            batch = batch // 128 * 64
        if batch < 32768 or rng.random() < 0.2:
            batch = rng.choice([2048, 4096, 8192, 16384])
        return _epoch(None, batch * rng.choice([1, 2, 4] if batch < 32768 else [1, 1, 2]), d, bits, batch, "gauss", rng.choice(["fixed", "columns"]))
    if op == "end_to_end":
        bits = rng.choice([2, 3, 3, 4, 5])
        d = _log(rng, 64, 8192)
        batch = 32 * _log(rng, 1, 16)
        steps = _log(rng, 32, 512)
        while steps * batch * d * bits > 1 << 32:
            steps //= 2
        return _epoch(None, max(1, steps) * batch, d, bits, batch, "lognormal", "optimal", model_bits=8,
                      candidates=rng.choice([128, 256, 512]))
    d = _log(rng, 16, 4096)
    n = max(100, min(_log(rng, 1000, 300000), (1 << 27) // d))
    if op == "levels":
        bits = rng.choice([2, 3, 3, 4])
        return {"op": "levels", "n": n, "d": d, "bits": bits, "mode": rng.choice(["optimal", "optimal", "greedy"]),
                "candidates": rng.choice([128, 256, 512, 1000, 1024]), "data": rng.choice(["lognormal", "gauss", "uniform"])}
    if op == "quantize":
        return {"op": "quantize", "n": n, "d": d, "bits": bits, "data": rng.choice(["gauss", "uniform", "columns"])}
    opt = bits <= 5 and rng.random() < 0.5
    return {"op": "loss", "n": n, "d": d, "bits": bits, "on": rng.choice(["rows", "copy 2", "copy 1"]),
            "data": "lognormal" if opt else "gauss", "levels": "optimal" if opt else rng.choice(["fixed", "columns"]),
            "candidates": max(64, 1 << (bits + 2)) if opt else 0}


# ------------------------------------------------------------------------------------------------
# inputs, made on the device
# ------------------------------------------------------------------------------------------------
DEV = "cuda:0"


class State:
    """What a program holds before the call: buffers, sizes, hyper-parameters."""


def _rows(case, g, rows, scale):
    """`rows` fp32 rows of the case's distribution."""
    d, kind = case["d"], case["data"]
    if kind == "gauss":                                    # clipped normal values on [-1, 1]
        return torch.randn(rows, d, generator=g, device=DEV).clamp_(-3.0, 3.0).div_(3.0)
    if kind == "lognormal":                                # skewed, nonnegative, on [0, 1]
        return torch.randn(rows, d, generator=g, device=DEV).exp_().div_(64.0).clamp_(0.0, 1.0)
    A = torch.rand(rows, d, generator=g, device=DEV)
    if kind == "sparse":                                   # line integrals: one pixel in 128 is crossed, with a weight of its own
        return A.sub_(1.0 - 1.0 / 128.0).clamp_(min=0.0).mul_(128.0)
    A.mul_(2.0).sub_(1.0)
    return A.mul_(scale) if kind == "columns" else A       # columns: a fifth of them 20 times smaller


def _chunk(case):
    return max(32, (1 << 26) // case["d"] // 32 * 32)      # 256 MiB of fp32 rows at a time


def _generators(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (1 << 62) + 17)
    d = case["d"]
    scale = torch.where(torch.rand(d, generator=g, device=DEV) < 0.2, 0.05, 1.0)
    xs = torch.randn(d, generator=g, device=DEV) / math.sqrt(d)
    return g, scale, xs


def _labels(case, A, xs, g):
    b = A @ xs
    b += 0.1 * torch.randn(b.shape[0], generator=g, device=DEV)
    return torch.where(b >= 0, 1.0, -1.0) if case.get("form") == "l2" else b


def _make_levels(s, case, A, n):
    """Levels as the case asks for; A: fp32 rows the ranges or the search are taken from (None for fixed ranges)."""
    d, bits, kind = case["d"], case["bits"], case["levels"]
    if kind in ("fixed", "unit"):
        s.lo.fill_(-1.0 if kind == "fixed" else 0.0)
        s.hi.fill_(1.0)
        zipml.levels(None, n, d, d, bits, zipml.UNIFORM, zipml.RANGE_GIVEN, 0, s.lo, s.hi, s.levels, s.grid, s.ws)
    elif kind == "columns":
        zipml.levels(A, n, d, d, bits, zipml.UNIFORM, zipml.SYMMETRIC, 0, s.lo, s.hi, s.levels, s.grid, s.ws)
    else:
        s.lo.zero_()
        s.hi.fill_(1.0)
        zipml.levels(A, n, d, d, bits, zipml.OPTIMAL, zipml.RANGE_GIVEN, case["candidates"], s.lo, s.hi, s.levels,
                     s.grid, s.ws)


def prepare(case, seed):
    n, d, bits, op = case["n"], case["d"], case["bits"], case["op"]
    K = 1 << bits
    s = State()
    s.case, s.seed = case, int(seed) & 0x7FFFFFFF
    batch = case.get("batch", 32)
    s.ws = torch.zeros(zipml.workspace_bytes(n, d, bits, batch, case.get("candidates", 0)), dtype=torch.uint8, device=DEV)
    s.lo, s.hi = torch.zeros(d, device=DEV), torch.zeros(d, device=DEV)
    s.levels = torch.zeros(d, K, device=DEV)
    s.grid = torch.zeros(d, K, dtype=torch.int16, device=DEV)
    g, scale, xs = _generators(case, seed)
    packs = op in ("epoch", "quantize") or case.get("on") != "rows" and op == "loss"
    if packs:
        s.p1 = torch.zeros(zipml.packed_bytes(n, d, bits), dtype=torch.uint8, device=DEV)
        s.p2 = torch.zeros_like(s.p1)
    if case.get("form") == "average":
        s.p1s, s.p2s = torch.zeros_like(s.p1), torch.zeros_like(s.p1)
    s.b = torch.zeros(n, device=DEV)
    keep = op in ("levels", "quantize") or case.get("levels") in ("columns", "optimal") or case.get("on") == "rows"
    A_all = torch.empty(n, d, device=DEV) if keep else None
    if op in ("epoch", "loss") and case["levels"] in ("fixed", "unit"):
        _make_levels(s, case, None, n)
    step, ms = _chunk(case), 0.0
    for r0 in range(0, n, step):
        rows = min(step, n - r0)
        A = _rows(case, g, rows, scale)
        s.b[r0:r0 + rows] = _labels(case, A, xs, g)
        if r0 == 0:
            ms = float(A.square().mean()) if op == "epoch" and not case["lr"] else 0.0
        if keep:
            A_all[r0:r0 + rows] = A
        else:
            _pack(s, A, rows, r0)
        del A
    if op in ("levels", "quantize") or case.get("on") == "rows":
        s.A = A_all
    if keep and op in ("epoch", "loss"):
        _make_levels(s, case, A_all, n)
        if packs:
            _pack(s, A_all, n, 0)
    if op == "loss":
        s.x = torch.randn(d, generator=g, device=DEV) / math.sqrt(d)
    if op == "epoch":
        # a step size that every batch size bears (a quarter of one over the mean squared norm of a sample)
        # where the workload has none of its own
        s.lr = case["lr"] or 0.25 / (d * max(ms, 1e-6))
        s.x = torch.zeros(d, device=DEV)
        s.epoch = 0
    return s


def _pack(s, A, rows, r0):
    c = s.case
    zipml.quantize(A, rows, c["d"], c["d"], r0, c["n"], s.levels, c["bits"], s.seed, 0, s.p1, s.p2)
    if c.get("form") == "average":
        zipml.quantize_swapped(A, rows, c["d"], c["d"], r0, c["n"], s.levels, c["bits"], s.seed, 0, s.p1s, s.p2s)


def run(s):
    c = s.case
    n, d, bits, op = c["n"], c["d"], c["bits"], c["op"]
    if op == "epoch":
        B, form = c["batch"], c["form"]
        if form == "l2":
            zipml.sgd_epoch_l2(s.p1, s.p2, s.levels, s.b, n, d, bits, s.x, B, s.lr, 0.05, s.ws)
        elif form == "prox":
            zipml.sgd_epoch_prox(s.p1, s.p2, s.levels, s.b, n, d, bits, s.x, B, s.lr, zipml.PROX_L1, 1e-4, s.ws)
        elif form == "average":
            zipml.sgd_epoch_avg(s.p1, s.p2, s.p1s, s.p2s, s.levels, s.b, n, d, bits, s.x, B, s.lr, s.ws)
        elif c["model_bits"]:
            M = c["candidates"]
            zipml.sgd_epoch(s.p1, s.p2, s.levels, s.b, n, d, bits, s.x, B, s.lr, s.ws, grid_idx=s.grid, grid_lo=0.0,
                            grid_step=1.0 / M, grid_max=M, grad_bits=8, model_bits=c["model_bits"], seed=s.seed,
                            epoch=s.epoch)
            s.epoch += 1
        else:
            zipml.sgd_epoch(s.p1, s.p2, s.levels, s.b, n, d, bits, s.x, B, s.lr, s.ws)
        return s.x
    if op == "levels":
        mode = zipml.OPTIMAL if c["mode"] == "optimal" else zipml.GREEDY
        zipml.levels(s.A, n, d, d, bits, mode, 0, c["candidates"], s.lo, s.hi, s.levels, s.grid, s.ws)
        return {"lo": s.lo, "hi": s.hi, "levels": s.levels, "grid": s.grid}
    if op == "quantize":
        zipml.levels(s.A, n, d, d, bits, zipml.UNIFORM, zipml.SYMMETRIC, 0, s.lo, s.hi, s.levels, s.grid, s.ws)
        zipml.quantize(s.A, n, d, d, 0, n, s.levels, bits, s.seed, 0, s.p1, s.p2)
        return {"lo": s.lo, "hi": s.hi, "levels": s.levels, "copy 1": s.p1, "copy 2": s.p2}
    if c["on"] == "rows":
        return zipml.loss(s.b, s.x, n, d, s.ws, A=s.A, lda=d)
    copy = 1 if c["on"] == "copy 1" else 2
    return zipml.loss(s.b, s.x, n, d, s.ws, packed=s.p1 if copy == 1 else s.p2, copy=copy, levels_t=s.levels, bits=bits)


def work(case):
    n, d, bits, op = case["n"], case["d"], case["bits"], case["op"]
    K = 1 << bits
    codes = n * d * bits / 8
    if op == "epoch":
        pairs = 2 if case["form"] == "average" else 1      # the labels, both copies (twice for the symmetrised form)
        return {"bytes": pairs * 2 * codes + 4 * n + 8 * d + 4 * d * K, "flops": pairs * 4 * n * d}
    if op == "levels":
        return {"bytes": 4 * n * d + 6 * d * K + 8 * d, "flops": 8 * n * d}
    if op == "quantize":
        return {"bytes": 4 * n * d + 2 * codes + 4 * d * K + 8 * d, "flops": 8 * n * d}
    rows = 4 * n * d if case["on"] == "rows" else codes + 4 * d * K
    return {"bytes": rows + 4 * n + 4 * d, "flops": 2 * n * d}


def tolerance(case):
    if case["op"] == "quantize":
        return "exact"                                     # draws and decisions are fixed by the seed
    if case["op"] == "levels":
        # the bin moments are fp64 sums in no fixed order: where two level sets cost the same to the last
        # bits, either may be chosen, and a level then moves by one bin
        return {"rel": 1e-4, "max": 2e-2, "differ": 1e-3}
    if case["op"] == "epoch" and case["model_bits"]:
        # fp32 sums decide integer codes of the gradient: an element on a rounding boundary moves one
        # coordinate by a step of its 8-bit grid
        return {"rel": 1e-3, "max": 2e-1}
    return {"rel": 1e-5, "max": 4e-4}                      # sums of 32-bit numbers
