"""Finite strain on plans whose first-axis layout was set: load cases solved
together against each of them solved by itself."""
import numpy as np
import pytest

from gpu_util import random_material, rel, say

pytestmark = pytest.mark.gpu


def _solve(shape, Fbar, layout, prec, lam, mu, kind, tol):
    import paper_2105_03297_amd as feh
    hz = feh.Homogenizer(shape, n_load=len(Fbar), precision=prec)
    if layout is not None:
        t = feh.feh_plan_tuning(hz.plan)
        t["first_per_load_case"] = layout
        feh.feh_plan_set_tuning(hz.plan, t)
    hz.set_material(lam=lam, mu=mu)
    out = hz.finite_strain_solve(Fbar, kind=kind, newton_tol=tol, equil_tol=tol, cg_tol=tol, fields=True)
    hz.close()
    assert all(r["status"] == 0 for r in out["report"])
    return out


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("kind,shape", [("fe", (9, 40, 40)), ("fe", (10, 12, 12)), ("fd", (8, 40, 40)), ("cd", (9, 2001)),
                                        ("fe", (4, 2001))])
def test_load_cases_keep_to_themselves(kind, shape, prec):
    """Newton's last step is of at most the tolerance and leaves its square and
    the CG tolerance of that step; the bounds are those of the one-workgroup
    tests."""
    say("finite layouts", kind, shape, prec)
    dim = len(shape)
    lam, mu = random_material(shape, seed=23, prec=prec, emax=4.0)
    rng = np.random.default_rng(4)
    Fbar = np.array([np.eye(dim) * (1.02 + 0.01 * l) + 0.02 * rng.standard_normal((dim, dim)) for l in range(2)])
    tol = 1e-10 if prec == "fp64" else 1e-5
    alone = [_solve(shape, Fbar[l:l + 1], None, prec, lam, mu, kind, tol) for l in range(2)]
    for layout in (None, 0, 1):
        both = _solve(shape, Fbar, layout, prec, lam, mu, kind, tol)
        for l in range(2):
            assert abs(both["report"][l]["newton_iterations"] - alone[l]["report"][0]["newton_iterations"]) <= 1
            assert float((both["F"][l] - alone[l]["F"][0]).abs().max()) <= 10 * tol, (layout, l)
            assert rel(both["P_mean"][l], alone[l]["P_mean"][0]) <= 100 * tol, (layout, l)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,L", [((2, 2), 13), ((2, 3), 64), ((2, 9), 16), ((2, 15), 64), ((2, 15), 7), ((17, 17), 64)])
def test_many_load_cases_of_a_small_grid(shape, L, prec):
    """One workgroup per load case, some done long before others (from a plain
    stretch, at once, to six load steps' worth): each as it is by itself."""
    import paper_2105_03297_amd as feh
    say("finite small, many load cases", shape, L, prec)
    lam, mu = random_material(shape, seed=31, prec=prec, emax=4.0)
    rng = np.random.default_rng(9)
    Fbar = np.array([np.eye(2) * (1.0 + 0.05 * (l % 3)) + 0.02 * (l % 4) * rng.standard_normal((2, 2)) for l in range(L)])
    tol = 1e-10 if prec == "fp64" else 1e-5
    kw = dict(kind="fe", n_steps=6, newton_tol=tol, equil_tol=tol, cg_tol=tol, fields=True)
    hz = feh.Homogenizer(shape, n_load=L, precision=prec)
    hz.set_material(lam=lam, mu=mu)
    out = hz.finite_strain_solve(Fbar, **kw)
    hz.close()
    one = feh.Homogenizer(shape, n_load=1, precision=prec)
    one.set_material(lam=lam, mu=mu)
    for l in range(L):
        o = one.finite_strain_solve(Fbar[l:l + 1], **kw)
        # the same workgroup program on the same numbers
        assert bool((out["F"][l] == o["F"][0]).all()) and bool((out["P"][l] == o["P"][0]).all()), l
        assert out["report"][l] == o["report"][0], l
    one.close()
