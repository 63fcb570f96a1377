"""Solves that run in one workgroup per load case against the general path on
the same plan (a plan whose schedule was set takes that path): every kind of
length (packed and odd last axes, an odd half length, radices 2 to 13, larger
primes), the largest grids that fit, batched materials and iteration caps."""
import numpy as np
import pytest

from gpu_util import random_material, rel, say

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2), (2, 3), (3, 2), (5, 7), (8, 6), (16, 10), (17, 17), (13, 22), (11, 14), (26, 31), (37, 6), (23, 38),
          (48, 44), (4, 512), (600, 3)]


def _general(feh, hz):
    feh.feh_plan_set_tuning(hz.plan, feh.feh_plan_tuning(hz.plan))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_workgroup_solve(shape, prec):
    """Both paths are the same CG with other summation orders: u agrees to the
    rounding that CG amplifies, well below the tolerance it stops at."""
    import paper_2105_03297_amd as feh
    say("one workgroup", shape, prec)
    tol = 1e-10 if prec == "fp64" else 1e-5
    mats = [random_material(shape, 50 + b, prec) for b in range(2)]
    Eb = np.concatenate([feh.unit_loads(2)] * 2)
    hz = feh.Homogenizer(shape, n_load=3, n_batch=2, precision=prec, h=(1.0, 0.8))
    hz.set_material(lam=np.stack([m[0] for m in mats]), mu=np.stack([m[1] for m in mats]))
    a = hz.solve(Eb, tol=tol, return_u=True)
    cap = hz.solve(Eb, tol=0.0, max_iter=2, return_u=True)
    _general(feh, hz)
    b = hz.solve(Eb, tol=tol, return_u=True)
    capb = hz.solve(Eb, tol=0.0, max_iter=2, return_u=True)
    hz.close()
    for x, y, t in ((a, b, tol), (cap, capb, 1e-12 if prec == "fp64" else 1e-5)):
        for p, q in zip(x["report"], y["report"]):
            if max(p["rel_residual"], q["rel_residual"]) < 1e3 * (2.0 ** -53 if prec == "fp64" else 2.0 ** -24):
                continue  # at rounding: solved to the last bit or to zero: the cap at tol 0 may or may not be what ended it
            assert p["status"] == q["status"] and abs(p["iterations"] - q["iterations"]) <= 1
        un = float(y["u"].abs().max())
        assert float((x["u"] - y["u"]).abs().max()) <= 10 * t * un
        assert rel(x["energy"], y["energy"]) <= (1e-12 if prec == "fp64" else 1e-6)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,shape", [("fe", (17, 17)), ("fe", (12, 22)), ("fd", (13, 9)), ("cd", (7, 11)), ("cd", (8, 6)),
                                        ("ls", (15, 14)), ("fe", (2, 2)), ("fe", (40, 41))])
def test_one_workgroup_finite_strain(kind, shape, prec):
    """Two load steps of two load cases: the same Newton steps, F to the
    tolerance of the last CG."""
    import paper_2105_03297_amd as feh
    say("one workgroup finite", kind, shape, prec)
    lam, mu = random_material(shape, 7, prec, emax=4.0)
    Fbar = np.stack([np.diag([1.05, 1.02]), np.array([[1.03, 0.02], [-0.01, 1.04]])])
    tol = 1e-10 if prec == "fp64" else 1e-5
    kw = dict(kind=kind, n_steps=2, newton_tol=tol, equil_tol=tol, cg_tol=tol, fields=True)
    hz = feh.Homogenizer(shape, n_load=2, precision=prec)
    hz.set_material(lam=lam, mu=mu)
    a = hz.finite_strain_solve(Fbar, **kw)
    _general(feh, hz)
    b = hz.finite_strain_solve(Fbar, **kw)
    hz.close()
    for p, q in zip(a["report"], b["report"]):
        assert p["status"] == q["status"] == 0 and abs(p["newton_iterations"] - q["newton_iterations"]) <= 1
    assert float((a["F"] - b["F"]).abs().max()) <= 10 * tol
    assert rel(a["P_mean"], b["P_mean"]) <= 100 * tol


@pytest.mark.parametrize("shape", [(32, 32), (40, 20), (300, 4), (4, 300), (900, 2), (1024, 2), (31, 31), (17, 31)])
def test_residual_keeps_falling_in_fp32(shape):
    """The residual of an FP32 solve keeps to that of the general path well
    below the rounding of the first residual (6e-8), where nothing but the
    rounding of the day may enter it: at 1e-6 and 1e-7 both stop within an
    iteration of one another, and the displacements agree to FP32's rounding
    times the grid's length (the smallest eigenvalue's share of a long wave)."""
    import paper_2105_03297_amd as feh
    say("small fp32 residual", shape)
    lam, mu = random_material(shape, 12, "fp32")
    A = np.random.default_rng(2).standard_normal((2, 2, 2)) * 0.01
    Eb = 0.5 * (A + np.swapaxes(A, 1, 2))
    for tol in (1e-6, 1e-7):
        out = []
        for general in (False, True):
            h = feh.Homogenizer(shape, n_load=2, precision="fp32")
            if general:
                feh.feh_plan_set_tuning(h.plan, feh.feh_plan_tuning(h.plan))
            h.set_material(lam=lam, mu=mu)
            o = h.solve(Eb, tol=tol, max_iter=200, return_u=True)
            out.append(o)
            h.close()
        a, b = out
        assert all(r["status"] == 0 for r in b["report"])
        for x, y in zip(a["report"], b["report"]):
            assert x["status"] == 0 and abs(x["iterations"] - y["iterations"]) <= 1, (tol, x, y)
        ua, ub = (o["u"].double().cpu().numpy() for o in out)
        for l in range(2):
            assert np.linalg.norm(ua[l] - ub[l]) <= 6e-8 * max(shape) * 10 * np.linalg.norm(ub[l])
