"""The monotone repair's wave pass, run on the host lane by lane from the
template that the kernels instantiate: runs of values that merge one after the
other, shorter and longer than the windows that take them ahead, ending inside
the input, at its end, or in a merge into a pool that was stored before."""
import ctypes
import os
import subprocess
import tempfile

import numpy as np
import pytest

from oracle import iterate as OI

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
RUNS = [1, 2, 3, 4, 5, 6, 8, 9, 12, 13, 16, 24, 63, 64, 65, 130, 400]


@pytest.fixture(scope="module")
def pv():
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    so = os.path.join(tempfile.mkdtemp(), "pvl.so")
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                           "-I", os.path.join(ROOT, "paper_1912_09240_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                           os.path.join(HERE, "pava_lanes.hip"), "-o", so], stderr=subprocess.DEVNULL)
    L = ctypes.CDLL(so)
    L.pv_pava_windows.argtypes = [ctypes.c_void_p, ctypes.c_int]
    L.pv_pava_windows.restype = ctypes.c_int
    return L


def _check(pv, v):
    ref = np.asarray(OI.pava(v.copy()))
    got = np.ascontiguousarray(v.copy())
    windows = pv.pv_pava_windows(got.ctypes.data_as(ctypes.c_void_p), len(got))
    assert np.array_equal(got, ref), np.abs(got - ref).max()
    return windows


@pytest.mark.parametrize("run", RUNS)
@pytest.mark.parametrize("end", ["inside", "end", "stored", "two_stored", "first"])
def test_runs_of_merges(pv, run, end):
    rng = np.random.default_rng(run)
    rise = np.linspace(0.0, 1.0, 20)
    fall = 3.0 - 0.5 * np.arange(run + 1) / (run + 1) - 1e-3 * rng.random(run + 1)  # stays above what is before it
    stored = np.array([2.0, 1.5, 1.6, 2.2, 1.9, 2.0])  # pools of two values, the last ones kept when the run starts
    deep = 3.0 - 4.0 * np.arange(run + 1) / (run + 1) ** 0.5
    v = {"inside": np.concatenate([rise, fall, 4.0 + rise]),
         "end": np.concatenate([rise, fall]),
         "stored": np.concatenate([rise, stored, fall, [-1.0 * (run + 2), 5.0]]),
         "two_stored": np.concatenate([rise, stored, 0.4 + stored, deep, 6.0 + rise]),
         "first": np.concatenate([fall, 4.0 + rise])}[end]
    windows = _check(pv, v)
    if end in ("inside", "end", "first"):  # one run: a window as soon as the pool has taken a few values
        assert (windows > 0) == (run > 5) or run in (4, 5), (run, windows)


def test_random_runs(pv):
    rng = np.random.default_rng(77)
    windows = 0
    for t in range(400):
        parts = []
        level = 0.0
        for _ in range(int(rng.integers(1, 12))):
            k = int(rng.choice(RUNS[:14]))
            down = -np.abs(rng.normal(0.0, 0.3, k)) if rng.random() < 0.6 else np.abs(rng.normal(0.0, 0.5, k))
            parts.append(level + np.cumsum(down))
            level = parts[-1][-1] + rng.normal(1.0, 1.0)
        v = np.concatenate(parts)
        if t % 3 == 0:
            v = np.round(v * 4.0) / 4.0
        windows += _check(pv, v)
    assert windows > 100


def test_windows_follow_the_last_run(pv):
    """Runs of twelve merges one after the other: the first is recognised after
    four single steps and leaves one window of eight, the following ones are
    taken ahead from their second merge on, in a window of eight and one for
    the last three.  Runs of three merges never pay for a window."""
    runs = 40
    v = np.concatenate([3.0 * r + 2.0 - 0.2 * np.arange(13) for r in range(runs)])
    assert _check(pv, v) >= 2 * (runs - 2)
    v = np.concatenate([3.0 * r + 2.0 - 0.2 * np.arange(4) for r in range(runs)])
    assert _check(pv, v) == 0
