"""The FP32 pair of normals against 64 bits, particle by particle: one step
from the origin with unit noise coefficients returns the normals themselves."""
import numpy as np
import pytest

import paper_1912_09240_amd as pr
from oracle import particles as OP

pytestmark = pytest.mark.gpu


def _exact(w0, w2):
    """sqrt(-2 ln u) (cos, sin)(2 pi t) in 64 bits: u the top 24 bits of w0,
    halfway into their cell, rounded to single; t in 256ths by bits 4..11 of w2,
    in between by bits 12..31."""
    u = ((w0 >> 8).astype(np.float64) * 2.0 ** -24 + 2.0 ** -25).astype(np.float32).astype(np.float64)
    a = (((w2 >> 4) & 255) + (w2 >> 12).astype(np.float64) * 2.0 ** -20) * (np.pi / 128.0)
    r = np.sqrt(-2.0 * np.log(u))
    return r, r * np.cos(a), r * np.sin(a)


@pytest.mark.parametrize("seed", [0, 5, 9])
def test_pair_against_64_bits(seed):
    """Every normal within 3.1 x 2^-23 of its radius: the logarithm is 1 ulp off
    and scaled (1.5 x 2^-23 of it, half of that in the root), the root 1 ulp,
    the table's sine or cosine 2^-25, two roundings of the result 2^-24 each;
    truncation 1e-9.  2^22 particles reach radii 0 to 5.6 and every table entry."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = 2 ** 22
    print(f"FP32 normals seed={seed} n={n}", flush=True)
    x = torch.zeros(n, dtype=torch.float32, device="cuda")
    y = torch.zeros(n, dtype=torch.float32, device="cuda")
    sde = pr.Sde(lam=1.0, eps=1.0, beta=1.0, precision=pr.PR_F32)  # sqrt(2 dt / beta) = sqrt(2 dt / (beta eps)) = 1
    pr.pr_fine_propagate(sde, pr.Schedule(1, 1, 0.5), seed, 3, n, 0, 1, x, y)
    torch.cuda.synchronize()
    w = OP.blocks(seed, 3, 0, 0, 0, n)
    r, z0, z1 = _exact(w[:, 0].astype(np.uint64), w[:, 2].astype(np.uint64))
    bound = 3.1 * 2.0 ** -23 * r + 1e-8
    for got, want in ((x, z0), (y, z1)):
        err = np.abs(got.cpu().numpy().astype(np.float64) - want)
        print(f"  largest error {err.max():.3e}, of its bound {np.max(err / bound):.2f}", flush=True)
        assert (err <= bound).all(), (err / bound).argmax()
