"""The search direction carried from one refinement step of a mixed solve into the next: it is only
worth carrying while FP32 rounding made little of the new residual.  On the rough right-hand side
of an adjoint solve (the seed of the kinetic energy) the first step leaves mostly rounding, and a
direction carried then, or with a tenth of rounding, costs iterations instead of saving them.  The
bound is the FP64 solve's count, which builds one Krylov space, and one iteration for every
refinement step after the first, which starts the next."""
import pytest
import torch

from bcm_inputs import CHANNEL_BC, OPEN_BC, uniform_mesh

from gpu_util import log, plan_for, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("dims", [(16, 4, 4), (16, 8, 8), (32, 8, 8)])
def test_carrying_does_not_cost_iterations(dims):
    m = uniform_mesh(dims, 1.0 / dims[1], 16, CHANNEL_BC)
    dt = 0.5 * float(m.h()[0])
    count = {}
    for precision in ("fp64", "mixed"):
        gen = torch.Generator(device="cuda").manual_seed(61)
        u = [0.1 * torch.rand(m.n_cells, generator=gen, device="cuda", dtype=torch.float64) - 0.05 for _ in range(3)]
        u[0] += 1.0
        plan = plan_for(m, precision)
        reps = []
        for _ in range(2):
            out = plan.project(u, None, 1.0, dt, 1.0)
            reps.append(out["report"])
            seed = plan.kinetic_energy(out["u_new"], 1.0, g_scale=1.0)[1]
            reps.append(plan.project_adjoint(u, None, seed, 1.0, dt, 1.0)[3])
            u = out["u_new"]
        count[precision] = reps
    log(f"  {dims}: " + ", ".join(f"{k} {[(r.n_outer, r.n_inner) for r in v]}" for k, v in count.items()))
    for f, x in zip(count["fp64"], count["mixed"]):
        assert f.status == 0 and x.status == 0
        assert x.n_inner <= f.n_inner + x.n_outer - 1


@pytest.mark.parametrize("seed,dims,n,opts", [
    (403, (3, 1, 4), 16, dict(post_sweeps=2, inner_tol=1e-2)),
    (507, (2, 2, 2), 16, dict(post_sweeps=3, inner_tol=1e-2)),
    (153, (2, 1, 2), 16, dict(post_sweeps=2, inner_tol=1e-2))])
def test_a_weak_v_cycle_converges_by_its_restarts(seed, dims, n, opts):
    """Without pre-smoothing and with the capped coarse CG flexible CG stagnates inside inner solves;
    a direction carried into the next one goes on stagnating, the restart does not."""
    for bc in (OPEN_BC, CHANNEL_BC, ("outflow", "inflow", "slip", "outflow", "inflow", "slip")):
        m = uniform_mesh(dims, 1.0, n, bc)
        plan = plan_for(m, "mixed", coarse_solver=0, pre_sweeps=0, prolong=0, **opts)
        for k in range(8):
            gen = torch.Generator(device="cuda").manual_seed(seed + 1000 * k)
            b = torch.randn(m.n_cells, generator=gen, device="cuda", dtype=torch.float64)
            for rhs in (b, plan.apply_laplacian(b)):
                _, rep = plan.poisson_solve(rhs)
                log(f"  {bc[0]} {dims} {k}: status {rep.status}, {rep.n_outer} steps, {rep.n_inner} iterations")
                assert rep.status == 0 and rep.final_rel_res <= 1e-10
