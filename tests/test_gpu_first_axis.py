"""The first-axis pass of 1024 points with the compile-time transform, and the
tile of general lengths, which takes as much LDS as the pass needs: against
the run-time pass, and against the oracle's direct solve."""
import numpy as np
import pytest

from gpu_util import random_material, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(1024, 2), (1024, 7), (1024, 64), (1024, 3, 4), (1024, 2, 9)])
def test_1024_points_match_runtime_pass(shape, prec):
    """Same butterflies, twiddles and inverse table: the two agree to rounding
    (bounds of the shorter compile-time lengths)."""
    import paper_2105_03297_amd as feh
    say("first axis 1024", shape, prec)
    lam, mu = random_material(shape, 17, prec)
    dim = len(shape)
    A = np.random.default_rng(2).standard_normal((2, dim, dim))
    Eb = 0.5 * (A + np.swapaxes(A, 1, 2))
    out = []
    for ct in (1, 0):
        h = feh.Homogenizer(shape, n_load=2, precision=prec)
        t = feh.feh_plan_tuning(h.plan)
        t["compile_time_transforms"] = ct
        feh.feh_plan_set_tuning(h.plan, t)
        h.set_material(lam=lam, mu=mu)
        o = h.solve(Eb, tol=1e-10 if prec == "fp64" else 1e-5, max_iter=3000, return_u=True)
        out.append((o["u"].double().cpu().numpy(), o["energy"], [r["iterations"] for r in o["report"]]))
        h.close()
    (ua, ea, ia), (ub, eb, ib) = out
    assert all(abs(x - y) <= 1 for x, y in zip(ia, ib))
    assert rel(ea, eb) < (1e-12 if prec == "fp64" else 1e-5)
    assert max(rel(ua[l], ub[l]) for l in range(2)) < (1e-10 if prec == "fp64" else 1e-3)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(1661, 3), (1030, 2), (151, 5), (2047, 4), (45, 2, 3), (313, 2, 4)])
def test_general_lengths_match_direct_solve(shape, prec):
    """u against the oracle's direct solve.  At a residual of tol in the energy
    norm and a contrast below 40, the strain energy error is below (40 tol)^2
    relative and the gradients' below 40 tol; FP32 adds the rounding of its
    fields, 1e-6 of the strain."""
    from oracle import fe
    import paper_2105_03297_amd as feh
    say("first axis general", shape, prec)
    lam, mu = random_material(shape, 12, prec)
    dim = len(shape)
    A = np.random.default_rng(2).standard_normal((2, dim, dim)) * 0.01
    Eb = 0.5 * (A + np.swapaxes(A, 1, 2))
    tol = 1e-10 if prec == "fp64" else 1e-6
    h = feh.Homogenizer(shape, n_load=2, precision=prec)
    h.set_material(lam=lam, mu=mu)
    o = h.solve(Eb, tol=tol, max_iter=3000, fields=True)
    got = o["strain"].double().cpu().numpy()
    h.close()
    assert all(r["status"] == 0 for r in o["report"])
    K = fe.assemble(lam, mu)
    for l in range(2):
        u = fe.solve_direct(K, fe.load_vector(lam, mu, Eb[l]), dim)
        ref, _ = fe.fields(u, lam, mu, Eb[l])
        ref = np.asarray(ref).reshape(got[l].shape)
        err = np.linalg.norm(got[l] - ref) / np.linalg.norm(ref)
        assert err <= 40 * tol + (1e-6 if prec == "fp32" else 1e-12), (l, err)
