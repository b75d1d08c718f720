"""GPU exponentials of the coarse generators against the oracle's, at the
edges of the product tiles (32 and 64), of a band as wide as the matrix and of
the squaring rule (none, odd, even)."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import coarse as OC
from oracle import iterate as OI
from oracle import particles as OP
from test_gpu_parity import _copy_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I", [3, 24, 25, 31, 32, 33, 64, 65, 383, 385])
# slices of 10 and 11 steps; mean: the largest rate times the shorter one
@pytest.mark.parametrize("mean", [0.2, 0.7, 1.5, 60.0, 1500.0])
def test_exponentials_match_oracle(I, mean):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"expm I={I} mean={mean}", flush=True)
    prop = OC.Propagator(OC.Grid(I), OP.Sde())
    K, S = 3, 31
    dt = mean / 10 / np.abs(np.diag(prop.A)).max()
    b = OI.slice_bounds(S, K)
    h = pr.pr_coarse_create(pr.Sde(), pr.Schedule(S, K, dt), pr.Grid(n_cells=I))
    try:
        for s in range(K):
            E = _copy_device(torch, pr.pr_coarse_matrix(h, s), I * I).reshape(I, I)
            # the bound of the existing coarse tests; entries are probabilities
            assert np.abs(E - prop.expm((b[s + 1] - b[s]) * dt)).max() < 1e-11, s
            assert np.abs(E.sum(0) - 1).max() < 1e-11, s
            assert E.min() >= 0.0, s
    finally:
        pr.pr_coarse_destroy(h)
