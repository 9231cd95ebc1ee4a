"""Which lengths half-length lines take (include/pspfft.h, Supported sizes), by the messages of plan creation
(Sec. 3.2, VerbosityOption).  Runs without a GPU: they are emitted before any device work.
"""
import ctypes

import pytest

import paper_1106_0557_amd as ps
from paper_1106_0557_amd import _lib

AXES = "xyz"


def smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


def family(axis, n, prec):
    """A radix family has the length: x lines of n points, y and z lines of 2n."""
    length = n if axis == 0 else 2 * n
    odd = length
    while odd % 2 == 0:
        odd //= 2
    count = {1: 16, 3: 24, 5: 20, 9: 36}.get(odd)
    return count is not None and length % count == 0 and n <= (2048, 1152)[prec] * (2 if axis == 0 else 1)


@pytest.fixture()
def messages():
    lib = _lib.load()
    before = lib.pspfft_get_verbosity()
    out = []
    ps.set_log_callback(lambda level, text: out.append((level, text)))
    ps.set_verbosity(ps.CONSOLE_INFO_2)
    yield out
    ps.set_log_callback(None)
    ps.set_verbosity(before)


def create(n, prec, flags=0):
    lib = _lib.load()
    handle = ctypes.c_void_p()
    if lib.pspfft_plan_create_ex(*n, (ctypes.c_double * 3)(0.1, 0.1, 0.1), prec, flags, ctypes.byref(handle)) == 0:
        assert lib.pspfft_destroy(handle.value) == 0  # on a GPU the plan exists


@pytest.mark.parametrize("axis", range(3))
@pytest.mark.parametrize("prec", range(2))
def test_lengths_of_half_length_lines(axis, prec, messages):
    for n in (n for n in range(1, 1300) if smooth(n)):
        mesh = [2, 4, 3]
        mesh[axis] = n
        messages.clear()
        create(mesh, prec)
        half = any(f"axis {AXES[axis]}: taken by half-length lines instead" in t for _, t in messages)
        generic = any(f"axis {AXES[axis]} (n = {n}) runs on the generic line kernel" in t for _, t in messages)
        if family(axis, n, prec):
            want = n in (80, 96) or 144 <= n <= 1152 or (n == 128 and prec == 1 and axis != 2)
            assert not generic, (mesh, prec)
        else:
            want = 25 <= n <= 1152 and not (n == 625 and prec == 1)
            assert generic == (not want), (mesh, prec)
        assert half == want, (mesh, prec)


def test_plane_lengths(messages):
    """Square planes of half-length lines: lengths up to 64, and others than a family's up to 120 (FP64 81)."""
    for prec in range(2):
        for n in (16, 18, 24, 25, 32, 45, 64, 72, 75, 81, 90, 120, 125):
            messages.clear()
            create((n, n, 5), prec)
            half = any("axis x: taken by half-length lines instead" in t for _, t in messages)
            assert half == (n != 72), (n, prec)  # (the others above 64 have rows of their own)
