"""Few particles (normals generated ahead by other waves of the block) against
many (every thread its own): the first particles of a large ensemble must
have the bits of the small one, at step counts around the rounds of 14, with
ragged slices, particle counts around the blocks of 64 and at both edges of
the rule (16384 particles; 49152 with slices of 48 steps)."""
import pytest

import paper_1912_09240_amd as pr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,steps", [(1, 1, 1), (63, 2, 27), (64, 1, 13), (65, 3, 14 * 3 + 1), (1000, 2, 15 * 2),
                                       (129, 7, 200), (16_384, 1, 29), (16_385, 1, 47), (16_385, 1, 48),
                                       (12_288, 4, 4 * 48), (12_289, 4, 4 * 48), (500, 1, 1000)])
def test_small_launch_has_the_large_launchs_bits(n, k, steps):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"fine split n={n} k={k} steps={steps}", flush=True)
    sde, sched = pr.Sde(eps=0.05), pr.Schedule(steps, k, 1e-3)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    N = 60_000  # above the rule for any k
    x = torch.randn((k, N), generator=g, device="cuda", dtype=torch.float64)
    y = torch.randn((k, N), generator=g, device="cuda", dtype=torch.float64)
    xs, ys = x[:, :n].contiguous(), y[:, :n].contiguous()
    pr.pr_fine_propagate(sde, sched, 3, 1, N, 0, k, x, y)
    pr.pr_fine_propagate(sde, sched, 3, 1, n, 0, k, xs, ys)
    torch.cuda.synchronize()
    assert torch.equal(x[:, :n], xs) and torch.equal(y[:, :n], ys)
    assert not torch.isnan(x).any()
