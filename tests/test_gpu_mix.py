"""Half-length lines with mixed radices (mix_lines.h): every length of their table on
each axis, odd and even, two and three stages, partial tiles, several tiles per
workgroup, tiled workspaces and the blocked spectrum (Sec. 2.1 defines the result).

Bars as elsewhere: FP64 <= 1e-12 relative L2 and max against the FP64 oracle, FP32
<= 1e-5 relative L2.
"""
import os
import re
import sys

import numpy as np
import pytest
import torch

import oracle
from oracle import norms
from paper_1106_0557_amd import sources

pytestmark = pytest.mark.gpu

FP64_TOL = 1e-12
FP32_TOL = 1e-5

_CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1106_0557_amd", "csrc")


def _lengths(header, fields):
    with open(os.path.join(_CSRC, header)) as f:
        return sorted({int(m) for m in re.findall(r"\bX\((\d+)(?:, \d+){%d}\)" % fields, f.read())})


LENGTHS = _lengths("mix_lines.h", 5)
PLANES = _lengths("mix_plane.h", 4)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    yield


def check(n, dtypes=(torch.float64, torch.float32)):
    from paper_1106_0557_amd import Plan

    print("[mix]", n, file=sys.stderr, flush=True)
    h = (0.021, 0.017, 0.013)
    S = sources.random_field(n, seed=sum(n))
    ref = oracle.solve_fft(S.numpy(), h)
    for dt in dtypes:
        plan = Plan(*n, h=h, dtype=dt)
        got = plan.solve(S.to("cuda", dt)).double().cpu().numpy()
        plan.close()
        r = norms.report(got, ref)
        assert r["rel_l2"] <= (FP64_TOL if dt == torch.float64 else FP32_TOL), (n, dt, r)
        assert dt == torch.float32 or r["rel_max"] <= FP64_TOL, (n, dt, r)


@pytest.mark.parametrize("n", LENGTHS)
def test_every_length_on_each_axis(n):
    for mesh in ((n, 3, 2), (2, n, 3), (3, 2, n)):
        check(mesh)


# x and y transforms of a plane in one kernel, odd and even n, against the five-pass plan too
@pytest.mark.parametrize("n", PLANES)
def test_planes(n):
    from paper_1106_0557_amd import Plan

    check((n, n, 5))
    S = sources.random_field((n, n, 5), seed=n).to("cuda")
    for dt, tol in ((torch.float64, FP64_TOL), (torch.float32, FP32_TOL)):
        out = []
        for five in (False, True):
            plan = Plan(n, n, 5, h=0.1, dtype=dt, five_pass=five)
            assert not (five and plan.fused)
            out.append(plan.solve(S.to(dt)).double().cpu().numpy())
            plan.close()
        assert norms.rel_l2(out[0], out[1]) <= tol


# several tiles per launch with a partial last one, three mixed axes, odd rows, and z lines
# whose persistent workgroups take several tiles
@pytest.mark.parametrize("n", [(45, 100, 27), (100, 27, 45), (27, 45, 100), (75, 50, 120), (20, 18, 1080),
                               (100, 18, 480), (16, 540, 30)])
def test_meshes_of_several_tiles(n):
    check(n)


@pytest.mark.parametrize("n,ztile", [((24, 20, 480), "16"), ((30, 16, 600), "4"), ((20, 12, 240), "2")])
def test_tiled_workspaces(n, ztile, monkeypatch):
    """Workspaces in tiles of z planes (PSPFFT_ZTILE), which large meshes get by themselves."""
    from paper_1106_0557_amd import Plan

    monkeypatch.setenv("PSPFFT_ZTILE", ztile)
    plan = Plan(*n, h=0.1, dtype=torch.float32)
    assert 1 < plan.ztile <= int(ztile) and n[2] % plan.ztile == 0
    plan.close()
    check(n)


# whole and partial last slabs, odd rows, partial tiles, and z tiles within slabs
@pytest.mark.parametrize("n", [(96, 25, 27), (45, 100, 150), (80, 27, 160), (125, 30, 80), (243, 25, 192)])
def test_slabs(n, monkeypatch):
    """Workspaces in slabs of kx (PSPFFT_SLABS), which large meshes get by themselves."""
    from paper_1106_0557_amd import Plan, _lib

    for v, want in (("0", n[0]), ("1", 32)):
        monkeypatch.setenv("PSPFFT_SLABS", v)
        plan = Plan(*n, h=0.1, dtype=torch.float32)
        assert _lib.load().pspfft_workspace_slab(plan._handle) == want
        plan.close()
    check(n)


# 32 problems of 563 row tiles (8 rows): workgroups take four tiles each, over problem boundaries
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_several_row_tiles_per_workgroup(dtype):
    import paper_1106_0557_amd as ps

    n = (270, 75, 60)
    check(n, (dtype,))
    plan = ps.Plan(*n, h=0.1, dtype=dtype)
    ws = [plan.workspace() for _ in range(32)]
    S = [sources.random_field(n, seed=i).to("cuda", dtype) for i in range(32)]
    out = [torch.empty_like(s) for s in S]
    ps.solve_batched(ws, S, out)
    alone = [plan.solve(s) for s in S]
    assert all(torch.equal(a, b) for a, b in zip(out, alone))
    for w in ws:
        w.close()
    plan.close()


@pytest.mark.parametrize("n", [(25, 18, 60), (16, 10, 135), (40, 12, 960)])
def test_blocked_spectrum_exports_the_octant(n):
    from paper_1106_0557_amd import Plan

    h = (0.05, 0.04, 0.03)
    want, _, abs_max = oracle.green_hat_octant(n, h)
    for dtype, tol in ((torch.float64, FP64_TOL), (torch.float32, 1e-7)):
        plan = Plan(*n, h=h, dtype=dtype)
        assert plan.spectrum_kz_fastest
        err = np.abs(plan.green().double().cpu().numpy() - want).max() / abs_max
        plan.close()
        assert err <= tol, (n, dtype, err)
