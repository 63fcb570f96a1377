"""The 3D strain, stress, F and P fields, which a run of voxels stages in LDS
and writes together, at the edges of the runs (32 voxels of one row, or 64
consecutive ones) and in the group sizes of both precisions, against the
blocks formed from the displacement."""
import numpy as np
import pytest

from gpu_util import random_material, say

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2, 2), (3, 9, 31), (2, 8, 33), (5, 3, 64), (2, 17, 65), (3, 2, 97)]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_solve_fields(shape, prec):
    """e = sym(grad u) + Ebar and C e of the returned u: a few operations on
    numbers of the size of u/h and lam, mu, rounded to the plan's precision."""
    from oracle import fe
    from paper_2105_03297_amd import Homogenizer
    say("solve fields", shape, prec)
    lam, mu = random_material(shape, seed=5, prec=prec)
    A = np.random.default_rng(3).standard_normal((2, 3, 3)) * 0.01
    Eb = 0.5 * (A + np.swapaxes(A, 1, 2))
    hz = Homogenizer(shape, n_load=2, precision=prec)
    hz.set_material(lam=lam, mu=mu)
    out = hz.solve(Eb, tol=1e-5, max_iter=500, return_u=True, fields=True)
    hz.close()
    eps = 1e-13 if prec == "fp64" else 2e-6
    for l in range(2):
        u = out["u"][l].double().cpu().numpy().reshape(-1)
        e, s = (np.asarray(x) for x in fe.fields(u, lam, mu, Eb[l]))
        size = np.abs(e).max() + np.abs(u).max()
        ge = out["strain"][l].double().cpu().numpy().reshape(e.shape)
        gs = out["stress"][l].double().cpu().numpy().reshape(s.shape)
        assert np.abs(ge - e).max() <= eps * size
        assert np.abs(gs - s).max() <= 3 * eps * size * (lam + 2 * mu).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind", ["fe", "fd", "cd"])
@pytest.mark.parametrize("shape", [(2, 2, 2), (3, 5, 7), (4, 8, 6), (3, 5, 13)])
def test_finite_fields(shape, kind, prec):
    """P = F S with S = lam tr(E) I + 2 mu E of the returned F, the mean of F
    the prescribed one and the mean of P the reported one."""
    from paper_2105_03297_amd import Homogenizer
    say("finite fields", shape, kind, prec)
    lam, mu = random_material(shape, seed=5, prec=prec, emax=4.0)
    Fb = np.stack([np.eye(3) * 1.03, np.eye(3) + 0.01 * np.arange(9).reshape(3, 3) / 8])
    hz = Homogenizer(shape, n_load=2, precision=prec)
    hz.set_material(lam=lam, mu=mu)
    out = hz.finite_strain_solve(Fb, kind=kind, newton_tol=1e-4, equil_tol=0.0, cg_tol=1e-4, fields=True)
    hz.close()
    eps = 1e-13 if prec == "fp64" else 2e-6
    N = int(np.prod(shape))
    F = out["F"].double().cpu().numpy().reshape(2, N, -1, 3, 3)
    P = out["P"].double().cpu().numpy().reshape(2, N, -1, 3, 3)
    E = 0.5 * (np.swapaxes(F, -1, -2) @ F - np.eye(3))
    S = lam.reshape(1, N, 1, 1, 1) * np.trace(E, axis1=-2, axis2=-1)[..., None, None] * np.eye(3) + 2 * mu.reshape(1, N, 1, 1, 1) * E
    size = 10 * (lam + 2 * mu).max()
    assert np.abs(P - F @ S).max() <= eps * size
    assert np.abs(F.mean(axis=(1, 2)) - Fb).max() <= eps
    assert np.abs(P.mean(axis=(1, 2)) - np.asarray(out["P_mean"]).reshape(2, 3, 3)).max() <= eps * size
