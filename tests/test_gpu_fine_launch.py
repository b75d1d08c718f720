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
