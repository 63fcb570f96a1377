"""Small 2D grids by the general passes (the schedule's general_passes), which
larger grids take, against the one-launch solves and the oracle; and plans
whose own schedule is set again, or that were tuned, against untouched ones."""
import numpy as np
import pytest

from gpu_util import random_material, rel, say

pytestmark = pytest.mark.gpu

SHAPES = [(2, 2), (2, 3), (3, 2), (5, 7), (8, 6), (16, 10), (17, 17), (13, 22), (11, 14), (26, 31), (37, 6), (23, 38), (48, 44),
          (4, 512), (64, 4), (600, 3)]


def _plan(shape, prec, n_load, lam, mu, n_batch=1, h=None, **schedule):
    import paper_2105_03297_amd as feh
    hz = feh.Homogenizer(shape, n_load=n_load, n_batch=n_batch, precision=prec, h=h)
    if schedule:
        feh.feh_plan_set_tuning(hz.plan, dict(feh.feh_plan_tuning(hz.plan), **schedule))
        assert all(feh.feh_plan_tuning(hz.plan)[k] == v for k, v in schedule.items())
    hz.set_material(lam=lam, mu=mu)
    return hz


@pytest.mark.parametrize("layout", [None, 0, 1])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_launch_matches_general_passes(shape, prec, layout):
    """Two materials, to the tolerance and to a cap of two iterations.  The same
    CG with other summation orders: u agrees to the rounding that CG amplifies,
    well below the tolerance it stops at."""
    import paper_2105_03297_amd as feh
    say("general passes", shape, prec, layout)
    tol = 1e-10 if prec == "fp64" else 1e-5
    lam, mu = (np.stack(x) for x in zip(*(random_material(shape, 50 + b, prec) for b in range(2))))
    Eb = np.concatenate([feh.unit_loads(2)] * 2)
    more = {} if layout is None else {"first_per_load_case": layout}
    hs = [_plan(shape, prec, 3, lam, mu, 2, (1.0, 0.8)), _plan(shape, prec, 3, lam, mu, 2, (1.0, 0.8), general_passes=1, **more)]
    full = [h.solve(Eb, tol=tol, return_u=True) for h in hs]
    cap = [h.solve(Eb, tol=0.0, max_iter=2, return_u=True) for h in hs]
    for h in hs:
        h.close()
    for (a, b), t in ((full, tol), (cap, 1e-12 if prec == "fp64" else 1e-5)):
        for x, y in zip(a["report"], b["report"]):
            if max(x["rel_residual"], y["rel_residual"]) < 1e3 * (2.0 ** -53 if prec == "fp64" else 2.0 ** -24):
                continue  # solved to the last bit or to zero: the cap may or may not be what ended it
            assert x["status"] == y["status"] and abs(x["iterations"] - y["iterations"]) <= 1
        assert float((a["u"] - b["u"]).abs().max()) <= 10 * t * float(b["u"].abs().max())
        assert rel(a["energy"], b["energy"]) <= (1e-12 if prec == "fp64" else 1e-6)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(64, 4), (128, 5), (512, 2), (1024, 2), (17, 16), (48, 46)])
def test_general_passes_match_direct_solve(shape, prec):
    """C_eff is second order in the CG error and, in FP32, in the rounding of
    the fields: 1e-10 at tol 1e-10, 1e-5 (the bound of the FP32 parity tests)
    at tol 1e-5."""
    from oracle import fe
    import paper_2105_03297_amd as feh
    say("general passes, direct solve", shape, prec)
    lam, mu = random_material(shape, seed=41, prec=prec)
    hz = _plan(shape, prec, 3, lam, mu, general_passes=1)
    out = hz.solve(feh.unit_loads(2), tol=1e-10 if prec == "fp64" else 1e-5, max_iter=500)
    hz.close()
    assert all(r["status"] == 0 for r in out["report"])
    ref = fe.homogenize(None, None, feh.unit_loads(2), lam_mu=(lam, mu))
    assert rel(out["C_eff"], ref["C_eff"]) <= (1e-10 if prec == "fp64" else 1e-5)


@pytest.mark.parametrize("shape", [(32, 32), (40, 20), (300, 4), (4, 300), (900, 2), (31, 31), (17, 31)])
def test_residual_keeps_falling_in_fp32_as_by_the_passes(shape):
    """At 1e-6 and 1e-7 of the first residual both stop within an iteration of
    one another, and the displacements agree to FP32's rounding times the
    grid's length."""
    say("small fp32 residual, passes", shape)
    lam, mu = random_material(shape, 12, "fp32")
    A = np.random.default_rng(2).standard_normal((2, 2, 2)) * 0.01
    Eb = 0.5 * (A + np.swapaxes(A, 1, 2))
    hs = [_plan(shape, "fp32", 2, lam, mu), _plan(shape, "fp32", 2, lam, mu, general_passes=1)]
    for tol in (1e-6, 1e-7):
        a, b = (h.solve(Eb, tol=tol, max_iter=200, return_u=True) for h in hs)
        for x, y in zip(a["report"], b["report"]):
            assert x["status"] == y["status"] == 0 and abs(x["iterations"] - y["iterations"]) <= 1, (tol, x, y)
        ua, ub = (o["u"].double().cpu().numpy() for o in (a, b))
        for l in range(2):
            assert np.linalg.norm(ua[l] - ub[l]) <= 6e-8 * max(shape) * 10 * np.linalg.norm(ub[l])
    for h in hs:
        h.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,shape", [("fe", (17, 17)), ("fe", (12, 22)), ("fd", (13, 9)), ("cd", (7, 11)), ("cd", (8, 6)),
                                        ("ls", (15, 14)), ("fe", (2, 2)), ("fe", (2, 15)), ("fe", (40, 41))])
def test_finite_strain_matches_general_passes(kind, shape, prec):
    """Two load steps of sixteen load cases: the same Newton steps, F to the
    tolerance of the last CG."""
    say("finite, general passes", kind, shape, prec)
    lam, mu = random_material(shape, 7, prec, emax=4.0)
    rng = np.random.default_rng(3)
    Fbar = np.array([np.diag([1.05, 1.02]) + 0.02 * rng.standard_normal((2, 2)) for _ in range(16)])
    tol = 1e-10 if prec == "fp64" else 1e-5
    hs = [_plan(shape, prec, 16, lam, mu), _plan(shape, prec, 16, lam, mu, general_passes=1)]
    a, b = (h.finite_strain_solve(Fbar, kind=kind, n_steps=2, newton_tol=tol, equil_tol=tol, cg_tol=tol, fields=True) for h in hs)
    for h in hs:
        h.close()
    for x, y in zip(a["report"], b["report"]):
        assert x["status"] == y["status"] == 0 and abs(x["newton_iterations"] - y["newton_iterations"]) <= 1
    assert float((a["F"] - b["F"]).abs().max()) <= 10 * tol
    assert rel(a["P_mean"], b["P_mean"]) <= 100 * tol


@pytest.mark.parametrize("tuned", [False, True])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(32, 32), (17, 17), (45, 50, 39), (24, 20, 18)])
def test_own_schedule_set_again_repeats_bitwise(shape, prec, tuned):
    """A plan's reported schedule, set on it and on a new plan, gives the same
    numbers; a tuned plan of a grid that is solved in one launch gives those of
    an untouched one."""
    import torch
    import paper_2105_03297_amd as feh
    say("own schedule", shape, prec, tuned)
    dim = len(shape)
    lam, mu = random_material(shape, 3, prec)
    Eb = feh.unit_loads(dim)
    hz = _plan(shape, prec, len(Eb), lam, mu)
    untouched = hz.solve(Eb, tol=1e-5, return_u=True)
    schedule = hz.autotune(reps=1) if tuned else feh.feh_plan_tuning(hz.plan)
    a = hz.solve(Eb, tol=1e-5, return_u=True)
    feh.feh_plan_set_tuning(hz.plan, schedule)
    b = hz.solve(Eb, tol=1e-5, return_u=True)
    new = _plan(shape, prec, len(Eb), lam, mu, **schedule)
    c = new.solve(Eb, tol=1e-5, return_u=True)
    hz.close()
    new.close()
    assert torch.equal(a["u"], b["u"]) and torch.equal(a["u"], c["u"]) and np.array_equal(a["energy"], c["energy"])
    if not tuned or dim == 2:
        assert torch.equal(a["u"], untouched["u"])
