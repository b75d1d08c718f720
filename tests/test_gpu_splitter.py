"""The splitter sort at the edges of its ranges against the oracle's stable
sort, bit for bit: ensembles of one bucket (up to 7168 and 14336 keys) and just above,
of one sampled run and of several, the longest it takes and one key more;
values that leave buckets too large for a block or for the value
sub-buckets (ties, a far outlier, infinities), a gap between two wells, and
a particle order whose period meets a fixed sampling stride."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import restrict as OR

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 1025, 4096, 4097, 7168, 7169, 8192, 8193, 14_336, 14_337, 16_385, 65_537]
LONGEST = 2 ** 20 + 2 ** 16


def _values(case, k, n, rng):
    x = rng.normal(0.0, 1.0, (k, n))
    if case == "equal":
        x[:] = -0.375
    elif case == "outlier":
        x[:, n // 2] = 1e30
    elif case == "few":
        x = np.round(x * 2.0) / 2.0
    elif case == "many":
        x = np.round(x * 300.0) / 300.0
    elif case == "half":
        x[:, ::2] = 0.25
    elif case == "inf":
        x[:, ::5] = np.inf
        x[:, 1::7] = -np.inf
        x[:, 2::3] = -0.0
    elif case == "gap":
        x = 0.02 * x + np.where(rng.random((k, n)) < 0.4, -1.0, 1.0)
    elif case == "period":
        x = 1e-3 * x + (np.arange(n) % 64)
    return np.ascontiguousarray(x)


def _check(torch, xs, prec, nq, want_perm=True):
    k, n = xs.shape
    x = torch.from_numpy(xs).cuda()
    ws = torch.empty(pr.pr_restrict_workspace_size(n, k, prec), dtype=torch.uint8, device="cuda")
    q = torch.zeros((k, nq + 1), dtype=torch.float64, device="cuda")
    rank, perm = (torch.zeros((k, n), dtype=torch.int32, device="cuda") for _ in range(2))
    srt = torch.zeros((k, n), dtype=torch.float64, device="cuda")
    only = torch.zeros_like(rank)
    q2, q3 = torch.zeros_like(q), torch.zeros_like(q)
    pr.pr_restrict_quantiles(x, prec, n, k, nq, q, ws, rank=rank, perm=perm, x_sorted=srt)
    pr.pr_restrict_quantiles(x, prec, n, k, nq, q2, ws, rank=only)
    pr.pr_restrict_quantiles(x, prec, n, k, nq, q3, ws)
    torch.cuda.synchronize()
    assert torch.equal(rank, only) and torch.equal(q, q2) and torch.equal(q, q3)
    for s in range(k):
        p, r, v = OR.sort_ranks(xs[s].astype(np.float64))
        assert np.array_equal(rank[s].cpu().numpy().view(np.uint32), r), s
        assert np.array_equal(perm[s].cpu().numpy().view(np.uint32), p), s
        assert np.array_equal(srt[s].cpu().numpy().view(np.uint64), v.view(np.uint64)), s
        if np.isfinite(v).all():
            assert np.array_equal(q[s].cpu().numpy(), OR.hazen_knots(v, nq)), s


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("case", ["smooth", "equal", "outlier", "few", "many", "half", "inf", "gap", "period"])
def test_splitter_sort_edges(case, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(11)
    for n in SIZES:
        print(f"splitter {case} precision={prec} n={n}", flush=True)
        xs = _values(case, 3, n, rng).astype(np.float64 if prec == pr.PR_F64 else np.float32)
        _check(torch, xs, prec, 7)


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("n", [LONGEST, LONGEST + 1])
@pytest.mark.parametrize("case", ["smooth", "half", "gap", "period"])
def test_splitter_sort_longest(case, n, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"splitter {case} precision={prec} n={n}", flush=True)
    xs = _values(case, 1, n, np.random.default_rng(12)).astype(np.float64 if prec == pr.PR_F64 else np.float32)
    _check(torch, xs, prec, 100)
