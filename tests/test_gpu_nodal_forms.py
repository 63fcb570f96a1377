"""The finite-element kinds of the strain-space solvers run on nodal vectors:
parity at the edges of the kernels' tiles (31 nodes along the last axis, 7
along the middle one, 255 along a 2D row; compile-time and run-time last-axis
passes, odd and even lengths), FP32 at a tolerance near its rounding, and the
plan's own solution left alone."""
import numpy as np
import pytest

from gpu_util import random_material, say

pytestmark = pytest.mark.gpu


def _ebars(dim, L):
    A = np.random.default_rng(8).standard_normal((L, dim, dim)) * 0.01
    return 0.5 * (A + np.swapaxes(A, 1, 2))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,h", [((2, 2), None), ((17, 31), (0.7, 1.3)), ((9, 256), None), ((8, 257), None),
                                     ((2, 2, 2), None), ((5, 7, 31), None), ((4, 8, 32), (1.0, 0.5, 2.0)),
                                     ((3, 4, 128), None), ((64, 3, 4), None)])
def test_fe_strain_cg_on_nodal_vectors(shape, h, prec):
    """Every element strain against the oracle's direct solve.  The CG stops
    at a residual of tol in the energy norm of M = B^T B; with the material's
    contrast below 40 the strain error is below 40 tol ||e||.  FP32 adds the
    rounding of its fields, of order 2^-24 of the strain a sum of a few terms
    long: 1e-6."""
    from oracle import fe
    from paper_2105_03297_amd import Homogenizer
    dim = len(shape)
    say("fe strain cg", shape, h, prec)
    lam, mu = random_material(shape, seed=12, prec=prec)
    Eb = _ebars(dim, 2)
    tol = 1e-11 if prec == "fp64" else 1e-6
    hz = Homogenizer(shape, n_load=2, precision=prec, h=h)
    hz.set_material(lam=lam, mu=mu)
    out = hz.strain_cg_solve(Eb, kind="fe", tol=tol, max_iter=500, fields=True)
    got = out["strain"].cpu().numpy().astype(np.float64)
    hz.close()
    assert all(r["status"] == 0 for r in out["report"])
    K = fe.assemble(lam, mu, h)
    for l in range(2):
        u = fe.solve_direct(K, fe.load_vector(lam, mu, Eb[l], h), dim)
        ref, _ = fe.fields(u, lam, mu, Eb[l], h)
        ref = np.asarray(ref).reshape(got[l].shape)
        err = np.linalg.norm(got[l] - ref) / np.linalg.norm(ref)
        assert err <= 40 * tol + (1e-6 if prec == "fp32" else 1e-12), (l, err)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_plan_solution_survives_fe_strain_cg(prec):
    """feh_strain_cg_solve keeps its vectors in the caller's buffer: the
    sensitivities of the plan's last solve, and a repeated solve, are bitwise
    what they were."""
    import torch
    from paper_2105_03297_amd import Homogenizer
    say("plan solution", prec)
    shape = (6, 9, 34)
    lam, mu = random_material(shape, seed=3, prec=prec)
    Eb = _ebars(3, 6)
    hz = Homogenizer(shape, n_load=6, precision=prec)
    hz.set_material(lam=lam, mu=mu)
    a = hz.solve(Eb, tol=1e-5, return_u=True)
    w = np.diag(np.arange(1.0, 7.0))
    ga = hz.energy_sensitivity(w)
    hz.strain_cg_solve(Eb, kind="fe", tol=1e-5)
    gb = hz.energy_sensitivity(w)
    b = hz.solve(Eb, tol=1e-5, return_u=True)
    assert torch.equal(ga[0], gb[0]) and torch.equal(ga[1], gb[1])
    assert torch.equal(a["u"], b["u"]) and np.array_equal(a["energy"], b["energy"])
    hz.close()
