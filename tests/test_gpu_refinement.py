"""Mixed-precision solves across their refinement steps (the flexible CG carries its last
direction into the next step, and the last step goes as far as the tolerance needs): every
Krylov variant, inner tolerances on both sides of what FP32 can gain, tight and loose solve
tolerances, warm starts, against the oracle's residual and exact solution, and the same bits on a
repeated call (nothing carries over between calls)."""
import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, OPEN_BC, configs, uniform_mesh
from oracle.fv import FVMesh

from gpu_util import dev, host, plan_for, rel_err, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

MESHES = {
    "channel_n8": lambda: uniform_mesh((4, 3, 2), 0.25, 8, CHANNEL_BC),
    "open_n16": lambda: uniform_mesh((2, 1, 2), 0.5, 16, OPEN_BC),
    "three_level_n4": lambda: configs.multilevel_small()["mesh"],
}


@pytest.mark.parametrize("name", sorted(MESHES))
@pytest.mark.parametrize("opts", [
    dict(), dict(krylov=2), dict(krylov=0), dict(inner_tol=1e-2), dict(inner_tol=1e-5),
    dict(check_every=3), dict(coarse_solver=0), dict(tol=1e-12), dict(tol=1e-4), dict(tol=0.3)],
    ids=lambda o: "-".join(f"{k}={v}" for k, v in o.items()) or "default")
def test_solves_reach_the_tolerance(name, opts):
    m = MESHES[name]()
    fv = FVMesh(m)
    tol = opts.get("tol", 1e-10)
    plan = plan_for(m, "mixed", max_iter=200, **opts)
    b = fv.A @ np.random.default_rng(7).standard_normal(m.n_cells)
    p, rep = plan.poisson_solve(dev(b))
    assert rep.status == 0 and rep.final_rel_res <= tol
    assert abs(fv.residual_norm(host(p), b) - rep.final_rel_res) <= 0.05 * tol + 1e-13
    p2, rep2 = plan.poisson_solve(dev(b))
    assert np.array_equal(host(p), host(p2)) and rep2.history == rep.history
    # warm start from a perturbed solution
    g = host(p) * (1.0 + 1e-4 * np.random.default_rng(8).standard_normal(m.n_cells))
    p3, rep3 = plan.poisson_solve(dev(b), p=dev(g), use_guess=True)
    assert rep3.status == 0 and rep3.final_rel_res <= tol
    if tol <= 1e-10:
        assert rel_err(host(p), host(p3)) <= 1e-7
        assert rel_err(host(p), fv.solve(b)) <= 1e-7


@pytest.mark.parametrize("n", [2, 4, 8])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_solves_that_converge_at_once(n, precision):
    """A constant right-hand side on one open cube leaves a handful of unknowns by symmetry: CG
    ends in a few iterations with a residual that falls to rounding from one check to the next,
    which no earlier check predicts.  The cube's condition number (3 pi^2 against 12 n^2, the
    ghost at half a cell) times the solve tolerance bounds the error of p."""
    m = uniform_mesh((1, 1, 1), 0.5, n, OPEN_BC)
    fv = FVMesh(m)
    plan = plan_for(m, precision)
    b = np.full(m.n_cells, 3.0)
    p, rep = plan.poisson_solve(dev(b))
    assert rep.status == 0 and rep.final_rel_res <= 1e-10
    assert rel_err(host(p), fv.solve(b)) <= n * n * 1e-10
    p2, rep2 = plan.poisson_solve(dev(b))
    assert np.array_equal(host(p), host(p2)) and rep2.history == rep.history
