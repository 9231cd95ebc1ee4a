"""Meshes whose planes are too large for the 32-bit addresses of half-length z lines: their z passes stay with the
radix families (wavefront-owned z lines of 576 and 1152 cells, column lines of the others).

The source is a few hundred unit cells, so that the discrete convolution (Sec. 2.1, Hockney's method) is a sum
of as many terms at any cell, taken in FP64.  Bar: 1e-5 of the largest potential, as for the other large FP32 meshes.
"""
import math
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

FP32_TOL = 1e-5


@pytest.mark.parametrize("n", [(2048, 2048, 576), (2048, 1536, 1152), (4096, 1024, 512)])
def test_fp32_planes_of_huge_meshes(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1106_0557_amd import Plan

    torch.cuda.empty_cache()  # (what earlier tests' tensors left with the allocator)
    nx, ny, nz = n
    h = np.array((0.011, 0.009, 0.013))
    rng = np.random.default_rng(sum(n))
    src = np.unique(rng.integers(0, nx * ny * nz, size=300))
    targets = np.unique(np.concatenate([rng.integers(0, nx * ny * nz, size=3000), src,
                                        [0, nx * ny * nz - 1]]))
    val = rng.uniform(0.5, 1.5, size=src.size).astype(np.float32)

    def cell(i):
        return np.stack([i % nx, i // nx % ny, i // (nx * ny)], axis=1)

    d = (cell(targets)[:, None, :] - cell(src)[None, :, :]) * h
    r = np.sqrt((d * d).sum(axis=2))
    r[r == 0.0] = h.min()  # the discrete Green's function at its own cell
    want = (-np.prod(h) / (4.0 * math.pi) * val.astype(np.float64) / r).sum(axis=1)

    S = torch.zeros((nz, ny, nx), dtype=torch.float32, device="cuda")
    S.view(-1)[torch.from_numpy(src).cuda()] = torch.from_numpy(val).cuda()
    plan = Plan(*n, h=tuple(h), dtype=torch.float32)
    print("[huge]", n, plan.workspace_bytes, plan.ztile, file=sys.stderr, flush=True)
    plan.solve(S, out=S)
    got = S.view(-1)[torch.from_numpy(targets).cuda()].double().cpu().numpy()
    plan.close()
    del S
    torch.cuda.empty_cache()
    assert np.abs(got - want).max() <= FP32_TOL * np.abs(want).max()
