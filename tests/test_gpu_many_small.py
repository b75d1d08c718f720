"""Ensembles of one bucket each, as many as fit the chip at one block per CU and
one more: hard ones (ties, outliers, infinities) among smooth ones."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import restrict as OR

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("k,n", [(256, 700), (257, 700), (256, 7169), (257, 7169), (300, 1)])
def test_many_small_ensembles(k, n, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"many small k={k} n={n} precision={prec}", flush=True)
    x = np.random.default_rng(k).normal(0.0, 1.0, (k, n))
    x[0::5] = 0.5
    x[1::5, n // 2] = 1e30
    x[2::5, ::3] = np.inf
    x[3::5] = np.round(x[3::5])
    xs = np.ascontiguousarray(x.astype(np.float64 if prec == pr.PR_F64 else np.float32))
    xd = torch.from_numpy(xs).cuda()
    ws = torch.empty(pr.pr_restrict_workspace_size(n, k, prec), dtype=torch.uint8, device="cuda")
    q = torch.zeros((k, 11), dtype=torch.float64, device="cuda")
    rank, perm = (torch.zeros((k, n), dtype=torch.int32, device="cuda") for _ in range(2))
    pr.pr_restrict_quantiles(xd, prec, n, k, 10, q, ws, rank=rank, perm=perm)
    torch.cuda.synchronize()
    for s in range(k):
        p, r, v = OR.sort_ranks(xs[s].astype(np.float64))
        assert np.array_equal(rank[s].cpu().numpy().view(np.uint32), r), s
        assert np.array_equal(perm[s].cpu().numpy().view(np.uint32), p), s
        if np.isfinite(v).all():
            assert np.array_equal(q[s].cpu().numpy(), OR.hazen_knots(v, 10)), s
