"""Rounding errors of FP32 half-length lines against the doubled lines that took the lengths before.

DOUBLED holds the relative L2 error, root mean square over 24 seeds, that the doubled lines (generic kernel)
had on the sources of `source`, measured with this file's code.  A sum of that many roundings scatters by a few per
cent from seed to seed, so each length may have 6 % more and their mean no more.
"""
import math
import sys

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SEEDS = 24
# (axis, length): error of the doubled lines
DOUBLED = {
    (1, 50): 8.165e-08, (1, 100): 8.231e-08, (1, 125): 9.433e-08, (1, 150): 8.765e-08, (1, 200): 8.503e-08, (1,
    250): 9.337e-08, (1, 300): 8.848e-08,
    (2, 50): 8.073e-08, (2, 100): 8.268e-08, (2, 125): 1.01e-07, (2, 150): 8.853e-08, (2, 200): 8.279e-08, (2, 250):
    9.636e-08, (2, 300): 9.016e-08,
}


def source(axis, length, seed):
    """Blob and slab along one axis of a mesh of 2 x 2 lines, FP32 values."""
    rng = np.random.default_rng(1000 * length + seed)
    q = (np.arange(length) + 0.5) / length
    r = rng.random(4)
    s = np.exp(-0.5 * ((q - 0.3 - 0.4 * r[0]) / (0.05 + 0.1 * r[1])) ** 2)
    s = s + 4.0 * np.pi * (np.abs(q - 0.4 - 0.2 * r[2]) < 0.1 + 0.1 * r[3])
    shape = [2, 2, 2]
    shape[2 - axis] = length
    line = [1, 1, 1]
    line[2 - axis] = length
    other = [2, 2, 2]
    other[2 - axis] = 1
    return (s.reshape(line) * (1.0 + 0.3 * rng.random(other))).reshape(shape).astype(np.float32)


def error(axis, length):
    from paper_1106_0557_amd import Plan

    n = [2, 2, 2]
    n[axis] = length
    h = (1.0 / length,) * 3
    plan = Plan(*n, h=h, dtype=torch.float32)
    e = 0.0
    for seed in range(SEEDS):
        S = source(axis, length, seed)
        ref = oracle.solve_fft(S.astype(np.float64), h)
        got = plan.solve(torch.from_numpy(S).cuda()).double().cpu().numpy()
        e += np.sum((got - ref) ** 2) / np.sum(ref ** 2)
    plan.close()
    return math.sqrt(e / SEEDS)


def test_errors_of_lines_with_a_factor_of_five():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ratios = []
    for (axis, length), want in DOUBLED.items():
        got = error(axis, length)
        print("[rounding]", "xyz"[axis], length, got, want, file=sys.stderr, flush=True)
        ratios.append(got / want)
        assert got <= 1.06 * want, (axis, length, got, want)
    assert math.exp(sum(map(math.log, ratios)) / len(ratios)) <= 1.0
