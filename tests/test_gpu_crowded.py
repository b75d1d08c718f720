"""Buckets of the splitter sort whose value sub-buckets are crowded, which are
ordered by digits: values of many magnitudes, ties, outliers, and FP64 keys
that agree in their highest 32 differing bits in short and in long runs; one
bucket and several, few ensembles (one kernel) and many (the rest in a second
one).  And the time such values take against smooth ones."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import restrict as OR
from tests.test_gpu_splitter import _check

pytestmark = pytest.mark.gpu

SIZES = [2, 65, 1025, 2049, 7168, 7169, 14_336, 14_337, 30_000]


def _crowded(case, k, n, rng):
    z = rng.normal(0.0, 1.0, (k, n))
    if case == "magnitudes":  # both signs, subnormal numbers and zeros of both signs
        x = np.sign(z) * 10.0 ** rng.uniform(-44, 30, (k, n))
        x[:, ::9] = np.where(z[:, ::9] < 0, -0.0, 0.0)
    elif case == "values":
        x = np.round(z * 20.0) / 7.0
    elif case == "outliers":
        x = 1.5 + 1e-3 * z
        x[:, n // 2], x[:, n // 3] = 1e30, -1e25
    else:
        # an outlier moves the highest differing bit to the sign; the others
        # differ below the 32 bits from there on
        per = 3 if case == "short_runs" else 1000
        base = 1.0 + (np.arange(n) // per) * 2.0 ** -20
        x = base[None, :] + rng.integers(0, 2 ** 20, (k, n)) * 2.0 ** -52
        x = np.take_along_axis(x, rng.random((k, n)).argsort(axis=1), axis=1)
        x[:, n // 2] = -1e30
    return np.ascontiguousarray(x)


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("case", ["magnitudes", "values", "outliers", "short_runs", "long_runs"])
def test_crowded_buckets(case, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(21)
    for n, k in [(n, 2) for n in SIZES] + [(500, 300), (7168, 257)]:
        print(f"crowded {case} precision={prec} n={n} k={k}", flush=True)
        with np.errstate(under="ignore"):
            xs = _crowded(case, k, n, rng).astype(np.float64 if prec == pr.PR_F64 else np.float32)
        _check(torch, xs, prec, 7)


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("n,k", [(10_000, 10), (14_336, 100)])
def test_time_of_crowded_values(n, k, prec):
    """The digits take at most one pass per byte of 32 bits and the second
    half only for long runs: no values take more than five times as long as
    smooth ones (the shortest of several passes; counted pairwise or sorted in
    global memory they took 7 to 14 times as long)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(22)
    ws = torch.empty(pr.pr_restrict_workspace_size(n, k, prec), dtype=torch.uint8, device="cuda")
    q = torch.empty((k, 101), dtype=torch.float64, device="cuda")
    rank = torch.empty((k, n), dtype=torch.int32, device="cuda")
    smooth = rng.normal(0.0, 1.0, (k, n))
    outlier = smooth.copy()
    outlier[:, n // 3] = 1e6
    ties = np.floor(rng.random((k, n)) * 64.0)
    us = []
    for name, v in (("smooth", smooth), ("outlier", outlier), ("ties", ties), ("cauchy", rng.standard_cauchy((k, n)))):
        print(f"crowded time {name} n={n} k={k} precision={prec}", flush=True)
        x = torch.from_numpy(v.astype(np.float64 if prec == pr.PR_F64 else np.float32)).cuda()
        best = np.inf
        for _ in range(20):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            pr.pr_restrict_quantiles(x, prec, n, k, 100, q, ws, rank=rank)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) * 1e3)
        us.append(best)
    assert max(us) < 5.0 * us[0], us
