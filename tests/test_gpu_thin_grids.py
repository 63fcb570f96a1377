"""Grids whose compile-time first-axis pass has fewer pencils than one of its
blocks (a long axis 0, a short rest): the solution against the oracle."""
import numpy as np
import pytest

from gpu_util import random_material, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(64, 4), (128, 5), (512, 2), (64, 3, 4), (64, 2, 2), (256, 2, 3)])
def test_thin_grid_matches_direct_solve(shape, prec):
    """C_eff is second order in the CG error and, in FP32, in the rounding of
    the fields: 1e-10 at tol 1e-10, 1e-5 (the bound of the FP32 parity tests)
    at tol 1e-5."""
    import microstructures as ms
    from oracle import fe
    from paper_2105_03297_amd import Homogenizer
    say("thin grid", shape, prec)
    lam, mu = random_material(shape, seed=41, prec=prec)
    loads = ms.unit_loads(len(shape))
    hz = Homogenizer(shape, n_load=len(loads), precision=prec)
    hz.set_material(lam=lam, mu=mu)
    out = hz.solve(loads, tol=1e-10 if prec == "fp64" else 1e-5, max_iter=500)
    hz.close()
    ref = fe.homogenize(None, None, loads, lam_mu=(lam, mu))
    assert all(r["status"] == 0 for r in out["report"])
    assert rel(out["C_eff"], ref["C_eff"]) <= (1e-10 if prec == "fp64" else 1e-5)
