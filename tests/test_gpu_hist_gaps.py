"""Histogram iterators and reweighting over empty tails, gaps wider than a
word of cells and grids at the edges of the waves' shares, bit for bit
against the oracle."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import coarse as OC
from oracle import histogram as H

pytestmark = pytest.mark.gpu

CELLS = [3, 16, 17, 63, 64, 65, 257, 1023, 1024]


def _masses(rng, I, pattern):
    r = rng.random(I) + 0.01
    if pattern == "tails":
        r[: I // 3] = 0.0
        r[I - I // 4:] = 0.0
    elif pattern == "left":
        r[: I - 1 - I // 8] = 0.0
    elif pattern == "wide":
        r[:] = 0.0
        r[[0, I // 2, I - 1]] = [0.2, 0.5, 0.3]
    elif pattern == "one":
        r[:] = 0.0
        r[I // 3] = 1.0
    elif pattern == "comb":
        r[1::2] = 0.0
    return r / r.sum()


PATTERNS = ["full", "tails", "left", "wide", "one", "comb"]


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("I", CELLS)
def test_jump_over_gaps(torch_dev, I):
    torch = torch_dev
    print(f"jump over gaps I={I}", flush=True)
    rng = np.random.default_rng(I)
    trip = [(a, b, c) for a in PATTERNS for b in PATTERNS for c in PATTERNS]
    rc, rf, rcs = (np.stack([_masses(rng, I, t[j]) for t in trip]) for j in range(3))
    k, g, og = len(trip), pr.Grid(n_cells=I), OC.Grid(I)
    out = torch.empty((k, I), dtype=torch.float64, device="cuda")
    ws = torch.empty(pr.pr_hist_jump_workspace_size(k, I), dtype=torch.uint8, device="cuda")
    for kind in (pr.PR_J_ADD, pr.PR_J_MULT, pr.PR_J_ROT, pr.PR_J_QUANTILE):
        pr.pr_hist_jump(kind, _dev(torch, rc), _dev(torch, rf), _dev(torch, rcs), k, g, out, ws)
        got = out.cpu().numpy()
        for s in range(0, k, 1 if I < 256 else 9):
            assert np.array_equal(got[s], H.jump(kind, rc[s], rf[s], rcs[s], og)), (kind, trip[s])


@pytest.mark.parametrize("I", CELLS)
def test_reweight_over_gaps(torch_dev, I):
    torch = torch_dev
    print(f"reweight over gaps I={I}", flush=True)
    rng = np.random.default_rng(100 + I)
    pairs = [(a, b) for a in PATTERNS for b in PATTERNS]
    k, n, g, og = len(pairs), 500, pr.Grid(n_cells=I), OC.Grid(I)
    rt = np.stack([_masses(rng, I, a) for a, _ in pairs])
    x = np.empty((k, n))
    for s, (_, b) in enumerate(pairs):  # particles in the cells that hold mass
        cells = rng.choice(I, size=n, p=_masses(rng, I, b))
        x[s] = -3.0 + (cells + 0.5) * (6.0 / I)
    w0 = H.equal_weights(n)
    rp = np.stack([H.hist_restrict(x[s], w0, og) for s in range(k)])
    ws = torch.empty(pr.pr_hist_match_workspace_size(n, k, I), dtype=torch.uint8, device="cuda")
    wo = torch.empty((k, n), dtype=torch.float64, device="cuda")
    pr.pr_hist_match(pr.PR_M_REWEIGHT, _dev(torch, rt), _dev(torch, rp), n, k, 1, g, _dev(torch, x),
                     _dev(torch, np.zeros((k, 1, n))), None, n, None, None, wo, ws)
    got = wo.cpu().numpy()
    for s in range(k):
        assert np.array_equal(got[s], H.reweight(rt[s], rp[s], x[s], w0, og)), pairs[s]
