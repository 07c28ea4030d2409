"""The window of fine bins that the exact threshold's one pass lays around its bracket (csrc/qa_exact_window.h, compiled
for the CPU): it has to hold the whole bracket, or the proof fails and the levels read the gradient again."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def window(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("window") / "exact_window.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2208_05631_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "exact_window.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def bits(x):
    return int(np.float32(x).view(np.uint32))


def holds(below, above, near0, near, far, spare):
    return (near0 << far) + spare < below and above + spare < (near0 + near) << far


@pytest.mark.parametrize("half", [1e-4, 1e-3, 0.005, 0.01, 0.015, 0.02, 0.03, 0.05, 0.1, 0.12])
def test_window_holds_the_bracket_with_the_finest_bins(window, half):
    """Thresholds all over the accepted range 1e-25 .. 1e30, half-widths up to the widest that is accepted, moved by
    the probe's step."""
    shape = (C.c_uint32 * 4)()
    window.near_window_shape(shape)
    far, finest, widest, bins = shape
    rng = np.random.default_rng(int(half * 1e4))
    near0, shift = C.c_uint32(), C.c_uint32()
    for _ in range(4000):
        t = 10.0 ** rng.uniform(-25, 30)
        mid = t * (1 + rng.uniform(-0.05, 0.05))
        below, above = bits(mid - half * t), bits(mid + half * t)
        window.near_window(below, bits(mid), above, C.byref(near0), C.byref(shift))
        assert finest <= shift.value <= widest, (t, mid, half)
        assert holds(below, above, near0.value, bins >> (far - shift.value), far, 4 << shift.value), (t, mid, half, shift.value)
        for finer in range(finest, shift.value):         # centred on mid to half a bin of 2^far
            near = bins >> (far - finer)
            n0 = (bits(mid) - ((near - 1) << (far - 1))) >> far
            assert not holds(below, above, n0, near, far, 4 << finer), (t, mid, half, finer)
