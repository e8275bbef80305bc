"""How far the last refinement step of a mixed solve goes: its target lies a factor 0.2 below the
tolerance, and FP32 rounding (at most a fifth of the target by the previous step's measure; here
allowed twice that) adds to it in square, sqrt(0.2^2 + (0.4 * 0.2)^2) = 0.2154 of the tolerance.  A
target with less margin leaves the solution further from the exact one at the same tolerance."""
import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, configs, uniform_mesh

from gpu_util import dev, plan_for, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

MESHES = {
    "channel_n4": lambda: uniform_mesh((9, 7, 5), 0.2, 4, CHANNEL_BC),
    "channel_n8": lambda: uniform_mesh((4, 3, 2), 0.25, 8, CHANNEL_BC),
    "odd_n8": lambda: uniform_mesh((21, 13, 11), 1.0 / 13.0, 8, CHANNEL_BC),
    "three_level_n4": lambda: configs.multilevel_small()["mesh"],
}


@pytest.mark.parametrize("rough", [False, True], ids=["operator_of_noise", "noise"])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_the_last_step_keeps_its_margin(name, rough):
    m = MESHES[name]()
    plan = plan_for(m, "mixed")
    for seed in (1, 2, 3):
        b = dev(np.random.default_rng(seed).standard_normal(m.n_cells))
        if not rough:
            b = plan.apply_laplacian(b)
        _, rep = plan.poisson_solve(b)
        assert rep.status == 0 and rep.final_rel_res <= 0.2154e-10, (seed, rep.final_rel_res)
