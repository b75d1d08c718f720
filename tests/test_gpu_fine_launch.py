"""Launch shapes of the fine propagator: the time of short slices, where a block's
start weighs more than its steps."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr

pytestmark = pytest.mark.gpu


def _best(torch, fn):
    best = np.inf
    for _ in range(20):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1e3)
    return best


def _propagate(torch, n, k, steps, prec):
    dt = torch.float64 if prec == pr.PR_F64 else torch.float32
    x, y = (torch.zeros((k, n), dtype=dt, device="cuda") for _ in range(2))
    sde = pr.Sde(eps=0.1, precision=prec)
    return lambda: pr.pr_fine_propagate(sde, pr.Schedule(steps * k, k, 1e-3), 1, 0, n, 0, k, x, y)


def test_time_of_short_ensembles_in_many_slices():
    """One particle in each of 16384 slices, one step: FP64 takes no more than
    1.6 times the FP32 launch, which has the same blocks (2.2 times with 512
    threads per slice that generate normals ahead)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("fine launch n=1 k=16384", flush=True)
    f64 = _best(torch, _propagate(torch, 1, 16_384, 1, pr.PR_F64))
    f32 = _best(torch, _propagate(torch, 1, 16_384, 1, pr.PR_F32))
    assert f64 < 1.6 * f32, (f64, f32)


def test_time_of_short_slices():
    """One step of 8 x 2^20 particles is little more than reading and writing
    them: no more than 1.8 times a copy of the states (2.4 times with the
    tables filled for every 256 particles)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("fine launch n=2^20 k=8", flush=True)
    a = torch.zeros((2, 8, 2 ** 20), dtype=torch.float64, device="cuda")
    b = torch.empty_like(a)
    step = _best(torch, _propagate(torch, 2 ** 20, 8, 1, pr.PR_F64))
    copy = _best(torch, lambda: b.copy_(a))
    assert step < 1.8 * copy, (step, copy)


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
@pytest.mark.parametrize("n,k,steps", [(262_144, 2, 2), (262_145, 4, 3), (700_001, 3, 20), (769, 1200, 1), (257, 2100, 7)])
def test_groups_of_a_block_have_the_bits_of_their_own(n, k, steps, prec):
    """Short slices whose blocks take several groups of 256 particles, ragged
    at the end, against the same slices one launch each (one group per block)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"fine groups n={n} k={k} steps={steps} precision={prec}", flush=True)
    dt = torch.float64 if prec == pr.PR_F64 else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn((k, n), generator=g, device="cuda", dtype=dt)
    y = torch.randn((k, n), generator=g, device="cuda", dtype=dt)
    sde, sched = pr.Sde(eps=0.05, precision=prec), pr.Schedule(steps * k, k, 1e-3)
    xs, ys = x.clone(), y.clone()
    pr.pr_fine_propagate(sde, sched, 3, 1, n, 0, k, x, y)
    for s in list(range(0, k, max(1, k // 5))) + [k - 1]:
        xa, ya = xs[s].clone(), ys[s].clone()
        m = min(n, 200_000)  # few enough blocks for one group each
        pr.pr_fine_propagate(sde, sched, 3, 1, m, s, 1, xa, ya)
        torch.cuda.synchronize()
        assert torch.equal(x[s, :m], xa[:m]) and torch.equal(y[s, :m], ya[:m]), s
    assert not torch.isnan(x).any()
    # the last particles, in a launch of fewer groups
    xa, ya = xs[0].clone(), ys[0].clone()
    pr.pr_fine_propagate(sde, sched, 3, 1, n, 0, 1, xa, ya)
    torch.cuda.synchronize()
    assert torch.equal(x[0], xa) and torch.equal(y[0], ya)


@pytest.mark.parametrize("n,steps", [(262_145, 3), (700_001, 9), (262_145, 15)])
def test_groups_of_the_chemical_and_checkpointed_steps(n, steps):
    """The same for the chemical system and the forward pass with
    checkpoints: the first particles alone (one group per block) have the bits
    of the whole ensemble's."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"fine groups, chemical and checkpoints n={n} steps={steps}", flush=True)
    k, m = 2, 100_000
    g = torch.Generator(device="cuda")
    g.manual_seed(steps)
    x = 100.0 + torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
    y = 100.0 + torch.randn((k, n), generator=g, device="cuda", dtype=torch.float64)
    xs, ys = x[:, :m].contiguous(), y[:, :m].contiguous()
    sched = pr.Schedule(steps * k, k, 1e-3)
    pr.pr_chem_fine_propagate(pr.Chem(), sched, 3, 1, n, 0, k, x, y)
    for s in range(k):
        pr.pr_chem_fine_propagate(pr.Chem(), sched, 3, 1, m, s, 1, xs[s], ys[s])
    torch.cuda.synchronize()
    assert torch.equal(x[:, :m], xs) and torch.equal(y[:, :m], ys)
    sde, sched, every = pr.Sde(eps=0.1), pr.Schedule(steps, 1, 1e-3), 4
    count = (steps + every - 1) // every
    x, y = (torch.randn(n, generator=g, device="cuda", dtype=torch.float64) for _ in range(2))
    xs, ys = x[:m].clone(), y[:m].clone()
    ck = torch.zeros((count, 2, n), device="cuda", dtype=torch.float64)
    cks = torch.zeros((count, 2, m), device="cuda", dtype=torch.float64)
    pr.pr_fine_checkpoint(sde, sched, 3, 1, n, x, y, ck, every)
    pr.pr_fine_checkpoint(sde, sched, 3, 1, m, xs, ys, cks, every)
    torch.cuda.synchronize()
    assert torch.equal(x[:m], xs) and torch.equal(y[:m], ys) and torch.equal(ck[:, :, :m], cks)
    assert not torch.isnan(x).any() and (ck[:, :, -1] != 0).all()


@pytest.mark.parametrize("prec", [pr.PR_F64, pr.PR_F32])
def test_time_of_waves_without_particles(prec):
    """Slices of fewer particles than a block has threads: a wave without a
    particle takes no steps (5000 slices of 64 particles, d = 32: one wave of
    each block's four; with all four stepping, the time of 256 particles)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"fine waves without particles precision={prec}", flush=True)
    k, d, dt = 5000, 32, torch.float64 if prec == pr.PR_F64 else torch.float32
    sde, sched = pr.Sde(eps=0.05, precision=prec, d=d), pr.Schedule(4 * k, k, 1e-3)
    us = {}
    for n in (64, 256):
        x = torch.zeros((k, n), device="cuda", dtype=dt)
        y = torch.zeros((k, d, n), device="cuda", dtype=dt)
        best = float("inf")
        for _ in range(10):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            pr.pr_fine_propagate(sde, sched, 3, 1, n, 0, k, x, y)
            e1.record()
            e1.synchronize()
            best = min(best, 1e3 * e0.elapsed_time(e1))
        us[n] = best
    print(us, flush=True)
    assert us[64] < 0.7 * us[256], us
