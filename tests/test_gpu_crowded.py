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


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
def test_time_of_one_value(prec):
    """A bucket of copies of one value leaves with the scatter: equal values do
    not take longer than smooth ones (by more than a quarter, the shortest of
    several passes; one block that read and wrote them all took 2.9 to 3.9 times
    as long)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 2 ** 20 + 2 ** 16
    ws = torch.empty(pr.pr_restrict_workspace_size(n, 1, prec), dtype=torch.uint8, device="cuda")
    q = torch.empty((1, 101), dtype=torch.float64, device="cuda")
    rank = torch.empty((1, n), dtype=torch.int32, device="cuda")
    smooth = np.random.default_rng(23).normal(0.0, 1.0, n)
    us = []
    for name, v in (("smooth", smooth), ("equal", np.full(n, 0.3)), ("half", np.where(smooth > 0, smooth, 0.0))):
        print(f"one value time {name} precision={prec}", flush=True)
        x = torch.from_numpy(v.astype(np.float64 if prec == pr.PR_F64 else np.float32)).cuda()
        best = np.inf
        for _ in range(20):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            pr.pr_restrict_quantiles(x, prec, n, 1, 100, q, ws, rank=rank)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) * 1e3)
        us.append(best)
    assert max(us) < 1.25 * us[0], us


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("n", [14_337, 20_000, 70_001])
def test_buckets_of_one_value(n, prec):
    """Values with buckets of their own beside others: the smallest, the
    largest and one between, and all values equal."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"one value n={n} precision={prec}", flush=True)
    rng = np.random.default_rng(24)
    x = rng.normal(0.0, 1.0, (5, n))
    part = rng.random((5, n)) < 0.6
    for row, v in enumerate((-9.0, 9.0, 0.125, -0.0)):
        x[row, part[row]] = v
    x[3, ::3] = 0.0
    x[4] = 2.5
    _check(torch, np.ascontiguousarray(x.astype(np.float64 if prec == pr.PR_F64 else np.float32)), prec, 7)


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("case", ["values", "zeros", "mixed", "outliers", "short_runs"])
def test_crowded_buckets_without_ranks(case, prec):
    """Knots and sorted values alone, where a crowded sub-bucket of one value is
    left as it was counted: ties, zeros of both signs (one sub-bucket, two keys),
    crowded sub-buckets of several values beside ones of one."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(23)
    dt = np.float64 if prec == pr.PR_F64 else np.float32
    for n, k in [(n, 3) for n in SIZES] + [(500, 300), (7168, 257), (14_337, 20), (200_000, 2)]:
        print(f"crowded without ranks {case} precision={prec} n={n} k={k}", flush=True)
        if case == "zeros":
            xs = np.where(rng.random((k, n)) < 0.5, -0.0, 0.0)
            xs[:, ::7] = np.round(rng.normal(0.0, 1.0, (k, len(range(0, n, 7)))) * 4.0) / 4.0
        elif case == "mixed":  # 64 values, those of the upper half with a few ulp around them
            xs = 1.0 + np.floor(rng.random((k, n)) * 64.0) / 64.0
            xs += np.where(xs > 1.5, rng.integers(0, 5, (k, n)) * np.spacing(dt(1.0)), 0.0)
        else:
            xs = _crowded(case, k, n, rng)
        xs = np.ascontiguousarray(xs.astype(dt))
        x = torch.from_numpy(xs).cuda()
        ws = torch.empty(pr.pr_restrict_workspace_size(n, k, prec), dtype=torch.uint8, device="cuda")
        q = torch.zeros((k, 101), dtype=torch.float64, device="cuda")
        srt = torch.zeros((k, n), dtype=torch.float64, device="cuda")
        pr.pr_restrict_quantiles(x, prec, n, k, 100, q, ws, x_sorted=srt)
        torch.cuda.synchronize()
        for s in range(0, k, max(1, k // 5)):
            v = OR.sort_ranks(xs[s].astype(np.float64))[2]
            assert np.array_equal(srt[s].cpu().numpy().view(np.uint64), v.view(np.uint64)), (n, s)
            assert np.array_equal(q[s].cpu().numpy(), OR.hazen_knots(v, 100)), (n, s)
