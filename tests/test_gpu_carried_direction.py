"""The search direction carried from one refinement step of a mixed solve into the next: it is only
worth carrying while FP32 rounding made little of the new residual.  On the rough right-hand side
of an adjoint solve (the seed of the kinetic energy) the first step leaves mostly rounding, and a
direction carried then, or with a tenth of rounding, costs iterations instead of saving them.  The
bound is the FP64 solve's count, which builds one Krylov space, and one iteration for every
refinement step after the first, which starts the next."""
import pytest
import torch

from bcm_inputs import CHANNEL_BC, uniform_mesh

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
