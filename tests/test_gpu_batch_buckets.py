"""Batched instances whose ensembles lie at the edges of the sort's buckets
(one block's 7168 keys, tiles of 4096, 14336) against single-instance handles:
knots and states agree bit for bit."""
import pytest

import paper_1912_09240_amd as pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(7168, 500), (7169, 8192, 8193), (14336, 14337, 64, 12289)])
def test_unequal_ensembles_at_bucket_edges(sizes):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"batch buckets sizes={sizes}", flush=True)
    sde, sched, grid = pr.Sde(lam=1.1, eps=0.1), pr.Schedule(40, 4, 0.002), pr.Grid(n_cells=50, n_q=40)
    ids = list(range(3, 3 + len(sizes)))

    def states(get, n):
        out = []
        for t in range(5):
            x = torch.empty(n, dtype=torch.float64, device="cuda")
            y = torch.empty(n, dtype=torch.float64, device="cuda")
            q = torch.empty(41, dtype=torch.float64, device="cuda")
            get(t, x, y, q)
            out += [x, y, q]
        torch.cuda.synchronize()
        return out

    h = pr.pr_parareal_batch_create([sde] * len(sizes), [sched] * len(sizes), list(sizes), grid, 7, instances=ids)
    try:
        pr.pr_parareal_batch_iterate(h, 2)
        got = [states(lambda t, x, y, q, i=i: pr.pr_parareal_batch_state(h, i, t, x=x, y=y, q=q), n)
               for i, n in enumerate(sizes)]
    finally:
        pr.pr_parareal_batch_destroy(h)
    for i, n in enumerate(sizes):
        hs = pr.pr_parareal_create(sde, sched, grid, 7, ids[i], n)
        try:
            pr.pr_parareal_iterate(hs, 2)
            ref = states(lambda t, x, y, q: pr.pr_parareal_state(hs, t, x=x, y=y, q=q), n)
        finally:
            pr.pr_parareal_destroy(hs)
        assert all(torch.equal(a, b) for a, b in zip(got[i], ref)), n
