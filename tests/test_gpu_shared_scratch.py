"""The table of inverses belongs to a buffer's contents, not to its address:
plans that take turns on the static scratch of feh_solve_noalloc, and a
workspace handed over a second time after other use."""
import numpy as np
import pytest

from gpu_util import random_material, say

pytestmark = pytest.mark.gpu


def _noalloc(feh, torch, plan, lam, mu, Eb):
    _, sm, W, rep = feh.feh_solve_noalloc(plan, lam.data_ptr(), mu.data_ptr(), Eb, 1e-10, 500)
    assert all(r["status"] == 0 for r in rep)
    return sm, W


def test_noalloc_plans_in_turn():
    """Bitwise the result of the first call, with another plan's solve (of
    another voxel size, hence other inverses) between the two."""
    import torch
    import paper_2105_03297_amd as feh
    say("noalloc in turn")
    shape = (64, 96)
    lam, mu = (torch.as_tensor(x, device="cuda") for x in random_material(shape, seed=5))
    Eb = feh.unit_loads(2)
    stream = torch.cuda.current_stream().cuda_stream
    a = feh.feh_plan_create(2, shape, None, 3, feh.FEH_FP64, stream)
    b = feh.feh_plan_create(2, shape, (1.0, 3.0), 3, feh.FEH_FP64, stream)
    first = _noalloc(feh, torch, a, lam, mu, Eb)
    _noalloc(feh, torch, b, lam, mu, Eb)
    again = _noalloc(feh, torch, a, lam, mu, Eb)
    assert np.array_equal(first[0], again[0]) and np.array_equal(first[1], again[1])
    feh.feh_plan_destroy(a)
    feh.feh_plan_destroy(b)


def test_workspace_set_again_after_other_use():
    import torch
    import paper_2105_03297_amd as feh
    say("workspace again")
    shape = (64, 96)
    lam, mu = (torch.as_tensor(x, device="cuda") for x in random_material(shape, seed=5))
    hz = feh.Homogenizer(shape, n_load=3)
    hz.set_material(lam=lam, mu=mu)
    a = hz.solve(feh.unit_loads(2), tol=1e-10)
    hz.workspace.fill_(0)
    torch.cuda.synchronize()
    feh.feh_plan_set_workspace(hz.plan, hz.workspace.data_ptr(), hz.workspace.numel())
    hz.set_material(lam=lam, mu=mu)
    b = hz.solve(feh.unit_loads(2), tol=1e-10)
    hz.close()
    assert np.array_equal(a["energy"], b["energy"])
