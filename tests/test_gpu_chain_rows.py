"""The serial coarse chain of one block (rows of E streamed in pairs, groups of
64 rows) against the coarse propagator slice by slice: the same bits at row
counts around the groups, odd and even, and beyond the streamed sizes, with
slices of two lengths."""
import pytest

import paper_1912_09240_amd as pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [3, 4, 31, 32, 33, 63, 64, 65, 127, 128, 129, 199, 200, 255, 256, 257])
def test_chain_is_slice_by_slice(cells):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"chain cells={cells}", flush=True)
    K, nq, n = 5, 40, 600
    sde, sched, grid = pr.Sde(eps=0.1), pr.Schedule(5 * 30 + 2, K, 2e-3), pr.Grid(n_cells=cells, n_q=nq)
    new = lambda m: torch.empty(m, dtype=torch.float64, device="cuda")
    h = pr.pr_parareal_create(sde, sched, grid, 3, 0, n)
    hb = pr.pr_parareal_batch_create([sde], [sched], [n], grid, 3, instances=[0])
    hc = pr.pr_coarse_create(sde, sched, grid)
    try:
        # the zeroth states are the initial ensemble matched to the chain's knots
        x0, x, xb, matched, q, qn = new(n), new(n), new(n), new(n), new(nq + 1), new(nq + 1)
        rank = torch.empty(n, dtype=torch.int32, device="cuda")
        ws = torch.empty(pr.pr_restrict_workspace_size(n, 1), dtype=torch.uint8, device="cuda")
        pr.pr_parareal_state(h, 0, x=x0)
        pr.pr_restrict_quantiles(x0, pr.PR_F64, n, 1, nq, q, ws, rank=rank)
        q0 = q.clone()
        for t in range(K):
            pr.pr_coarse_fp_step(hc, t, 1, q, qn)
            q, qn = qn, q
            pr.pr_match_quantiles(q, q0, rank, n, 1, nq, x0, matched)
            pr.pr_parareal_state(h, t + 1, x=x)
            pr.pr_parareal_batch_state(hb, 0, t + 1, x=xb)
            torch.cuda.synchronize()
            assert torch.isfinite(matched).all() and not torch.equal(matched, x0)
            assert torch.equal(matched, x), t
            assert torch.equal(matched, xb), t
    finally:
        pr.pr_coarse_destroy(hc)
        pr.pr_parareal_batch_destroy(hb)
        pr.pr_parareal_destroy(h)
