"""Prime passes on the matrix cores and the small tiles of the run-time passes,
at the sizes where they change over: the smallest prime above 13, primes whose
outputs fill whole 16-row tiles and one more, prime passes after a radix pass
(twiddles, several butterflies a row), columns that do not fill a tile, lengths
left to the direct sum, and grids on either side of the small tiles."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

SHAPES = [(17, 19), (31, 29), (2, 37), (61, 34), (151, 4), (3, 302), (47, 95), (289, 5), (1021, 2), (2, 1021),
          (1361, 3), (2039, 2), (34, 17, 5), (3, 62, 31), (19, 2, 38), (2, 151, 3), (64, 1000), (1000, 16), (8, 96, 30)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_transform_pair(shape, prec):
    """Against numpy's transform in FP64.  Rounding: a transform of n points
    sums them pairwise in a few passes and, in a prime pass, R terms in one
    chain, whose error grows like sqrt(R) eps of the result's norm; 12 eps
    sqrt(largest prime) covers three axes of both directions."""
    from paper_2105_03297_amd import Homogenizer
    say("transform", shape, prec)
    dim = len(shape)
    hz = Homogenizer(shape, n_load=2, precision=prec)
    x = np.random.default_rng(5).standard_normal((2 * dim,) + shape)
    if prec == "fp32":
        x = x.astype(np.float32).astype(np.float64)
    X = hz.fft_forward(x).cpu().numpy().reshape((2 * dim,) + shape[:-1] + (shape[-1] // 2 + 1,))
    ref = np.fft.rfftn(x, axes=tuple(range(1, dim + 1)))
    back = hz.fft_inverse(ref.astype(np.complex64 if prec == "fp32" else np.complex128)).cpu().numpy().reshape(x.shape)
    hz.close()
    prime = max(p for n in shape for p in range(2, n + 1) if n % p == 0 and all(p % q for q in range(2, int(p ** 0.5) + 1)))
    bound = 12 * np.sqrt(prime) * (2.0 ** -24 if prec == "fp32" else 2.0 ** -53)
    assert np.linalg.norm(X - ref) <= bound * np.linalg.norm(ref)
    assert np.linalg.norm(back - x) <= bound * np.linalg.norm(x)


@pytest.mark.parametrize("shape", [(17, 31), (151, 38), (96, 1000), (3, 17, 34), (45, 50, 39)])
def test_solve_on_small_tiles_matches_direct_solve(shape):
    """C_eff is second order in the CG error: 1e-10 at tol 1e-10."""
    import microstructures as ms
    from gpu_util import random_material, rel
    from oracle import fe
    from paper_2105_03297_amd import Homogenizer
    say("solve", shape)
    lam, mu = random_material(shape, seed=2)
    loads = ms.unit_loads(len(shape))
    hz = Homogenizer(shape, n_load=len(loads))
    hz.set_material(lam=lam, mu=mu)
    out = hz.solve(loads, tol=1e-10, max_iter=500)
    hz.close()
    if np.prod(shape) < 20000:
        ref = fe.homogenize(None, None, loads, lam_mu=(lam, mu))["C_eff"]
    else:  # too large for the sparse direct solve: plain CG in C
        ref = fe.homogenize(None, None, loads, lam_mu=(lam, mu), method="ccg")["C_eff"]
    assert rel(out["C_eff"], ref) <= 1e-10
