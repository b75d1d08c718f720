"""Observables and their seeds around the blocks of 256 particles, and the sum
of the reverse sweep's block sums over few and many blocks."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import restrict as OR

pytestmark = pytest.mark.gpu


def _torch():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 10_001])
@pytest.mark.parametrize("alphas", [(), (0.5,), (0.0, 1.0, 0.37), (0.5, 0.5, 0.5)])
def test_observable_seeds(n, alphas):
    torch = _torch()
    print(f"observables n={n} alphas={alphas}", flush=True)
    x = np.random.default_rng(n).standard_normal(n)
    xd = torch.tensor(x, device="cuda")
    k = 1 + len(alphas)
    obs = torch.full((k,), np.nan, dtype=torch.float64, device="cuda")
    seeds = torch.full((k, n), np.nan, dtype=torch.float64, device="cuda")
    ws = torch.empty(pr.pr_observables_workspace_size(n), dtype=torch.uint8, device="cuda")
    pr.pr_observables(xd, n, alphas, obs, ws, seed_x=seeds)
    got, sd = obs.cpu().numpy(), seeds.cpu().numpy()
    perm = np.argsort(x, kind="stable")
    assert np.array_equal(sd[0], 2.0 * x / n)
    for a, al in enumerate(alphas):
        # the quantile is the seed's own combination of the particles
        assert abs(got[1 + a] - OR.hazen_at(x[perm], al)[0]) < 1e-14
        ref = np.zeros(n)
        t = al * n - 0.5
        if t <= 0:
            ref[perm[0]] = 1.0
        elif t >= n - 1:
            ref[perm[n - 1]] = 1.0
        else:
            r = int(np.floor(t))
            ref[perm[r]], ref[perm[r + 1]] = 1.0 - (t - r), t - r
        assert np.array_equal(sd[1 + a], ref)
    obs2 = torch.full((k,), np.nan, dtype=torch.float64, device="cuda")
    pr.pr_observables(xd, n, alphas, obs2, ws)  # no seeds asked for
    assert torch.equal(obs, obs2)


@pytest.mark.parametrize("n", [1, 257, 256 * 256 + 3, 256 * 2048 + 1])
def test_one_step_gradient_sums_every_particle(n):
    torch = _torch()
    print(f"one step n={n}", flush=True)
    dt = 1e-2
    sde, sched = pr.Sde(), pr.Schedule(1, 1, dt)
    x = torch.empty(n, dtype=torch.float64, device="cuda")
    y = torch.empty(n, dtype=torch.float64, device="cuda")
    pr.pr_init_ensemble(sde, 0, 0, n, x, y)
    x0, y0 = x.clone(), y.clone()
    ck = torch.empty((1, 2, n), dtype=torch.float64, device="cuda")
    pr.pr_fine_checkpoint(sde, sched, 0, 0, n, x, y, ck, 8)
    w = torch.rand(n, dtype=torch.float64, device="cuda")
    grad = torch.empty((1, 4), dtype=torch.float64, device="cuda")
    ws = torch.empty(pr.pr_adjoint_workspace_size(n, 8, 1), dtype=torch.uint8, device="cuda")
    pr.pr_fine_adjoint(sde, sched, 0, 0, n, ck, 8, w, 1, grad, ws, from_initial=0)
    for col, term in ((0, -dt * w * (x0 - y0)), (3, -dt * w * x0 ** 3)):
        # n additions, a few roundings per term
        assert abs(grad[0, col].item() - term.sum().item()) <= 1e-15 * (64 + n ** 0.5) * term.abs().sum().item()
