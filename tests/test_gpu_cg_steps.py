"""CG steps as amg_pcg_solve takes them (the next V-cycle launched ahead of the
test, its first smoother step taken with the update, short sums added by the
kernels that need them, scalars reported to pinned memory) against the
allocation-free solve, which takes the same steps one after the other and reads
its scalars back: the same bits, wherever a solve ends."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _problem(name):
    from workloads import config1_checkerboard_2d, layered_stack_3d, poisson_box, rotated_anisotropic_3d

    return {
        "one level": lambda: (poisson_box((20, 17), dirichlet="x0"), dict()),
        "two levels": lambda: (poisson_box((30, 31), dirichlet="x0"), dict(max_coarse=200)),
        "checker": lambda: (config1_checkerboard_2d(), dict(max_coarse=100)),
        "aniso": lambda: (rotated_anisotropic_3d(n=16, block=8), dict(max_coarse=100)),
        # more than 1,024 row blocks: sums by a kernel of their own
        "stack": lambda: (layered_stack_3d(n=46, repeats=4), dict(max_levels=16)),
    }[name]()


def _both(h, b, x0, **kw):
    import torch

    x, y = x0.clone(), x0.clone()
    _, i = h.solve(b, x, raise_on_error=False, **kw)
    _, j = h.solve_noalloc(b, y, raise_on_error=False, **kw)
    assert (i["status"], i["iterations"], i["rel_res"]) == (j["status"], j["iterations"], j["rel_res"])
    assert torch.equal(x, y)
    return x, i


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["one level", "two levels", "checker", "aniso", "stack"])
def test_solves_end_alike(name, precision):
    import torch

    import paper_2602_05686_amd as amg

    p, kw = _problem(name)
    h = amg.Hierarchy.from_problem(p, precision=precision, **kw)
    assert (h.level_form(0)["blocks"] > 1024) == (name == "stack")
    b = torch.as_tensor(p.b).cuda()
    zero = torch.zeros_like(b)
    start = torch.as_tensor(np.random.default_rng(3).standard_normal(p.n)).cuda()
    _, i = _both(h, b, zero, tol=1e-8, max_iter=200)
    assert i["status"] == "OK"
    for max_iter in (1, 2, 3, 7):  # at the cap, with and without a V-cycle foreseen
        for x0 in (zero, start):
            _, i = _both(h, b, x0, tol=1e-8, max_iter=max_iter)
            assert i["iterations"] <= max_iter
    for tol in (0.5, 1e-1, 1e-3, 1e-6):
        _both(h, b, start, tol=tol, max_iter=200)
    # from the solution: no step at all
    x, _ = _both(h, b, zero, tol=1e-10, max_iter=200)
    _, i = _both(h, b, x, tol=1e-8, max_iter=200)
    assert i["iterations"] == 0
    # a smaller system's solve between two of this one
    q, qkw = _problem("two levels")
    g = amg.Hierarchy.from_problem(q, precision=precision, **qkw)
    _both(g, torch.as_tensor(q.b).cuda(), torch.zeros(q.n, dtype=torch.float64, device="cuda"), tol=1e-8, max_iter=50)
    _both(h, b, zero, tol=1e-8, max_iter=200)
    g.close()
    h.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("name", ["checker", "stack"])
def test_true_residual_replaces_the_recurrence(name, precision):
    """A tolerance that the recurrence residual passes and the true one does not: the solve goes on from the true
    residual, past a V-cycle that may have been launched from the other."""
    import torch

    import paper_2602_05686_amd as amg

    p, kw = _problem(name)
    h = amg.Hierarchy.from_problem(p, precision=precision, **kw)
    b = torch.as_tensor(p.b).cuda()
    zero = torch.zeros_like(b)
    cap = 120
    _, i = _both(h, b, zero, tol=1e-16, max_iter=cap)
    assert i["status"] == "NOT_CONVERGED" and i["iterations"] == cap
    # the same steps with a tolerance out of reach: without replacement the
    # recurrence goes on falling, far below where the other solve has to start again
    _, j = _both(h, b, zero, tol=1e-300, max_iter=cap)
    assert j["iterations"] == cap and j["rel_res"] < 1e-30 and i["rel_res"] > 1e-16
    h.close()
