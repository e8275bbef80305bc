"""The momentum pass where its layout has edges: cubes with a neighbour or a wall on each side in
every combination of axes, units with empty slots, one-cube axes (both x halos from walls), for
every cube size and scheme, against the oracle.  Tolerances as in test_gpu_momentum.py: 1e-12
relative for H and the explicit steps (2e-6 with FP32 fields), 1e-11 for Crank-Nicolson solved
to 1e-13 (FP64 fields only: with FP32 fields the residual the sweeps can reach, not the pass,
sets the error)."""
import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, OPEN_BC, uniform_mesh, uniform_random_velocity
from oracle.momentum import step

from gpu_util import dev, host, plan_for, rel_err, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

MIXED = ("outflow", "inflow", "slip", "outflow", "inflow", "slip")


@pytest.mark.parametrize("precision", ["fp64", "mixed_f32fields"])
@pytest.mark.parametrize("n,dims,bc", [
    (16, (3, 3, 3), MIXED), (16, (1, 2, 3), CHANNEL_BC), (16, (2, 1, 1), OPEN_BC),
    (8, (5, 3, 3), MIXED), (8, (1, 1, 1), OPEN_BC), (8, (1, 3, 1), CHANNEL_BC),
    (4, (7, 3, 5), MIXED), (4, (1, 1, 3), CHANNEL_BC), (4, (2, 2, 2), OPEN_BC)])
def test_schemes_match_oracle(n, dims, bc, precision):
    m = uniform_mesh(dims, 0.25, n, bc)
    f32 = precision == "mixed_f32fields"
    u = uniform_random_velocity(m, 31, 0.6, (0.3, -0.2, 0.1)).reshape(3, -1)
    hp = uniform_random_velocity(m, 32, 2.0).reshape(3, -1)
    if f32:
        u, hp = (x.astype(np.float32).astype(np.float64) for x in (u, hp))
    h = float(m.h()[0])
    nu, U_in, dt = 0.3 * h, 0.7, 0.4 * h
    plan = plan_for(m, precision)
    ft = plan.field_dtype
    ud, hd = [dev(x, ft) for x in u], [dev(x, ft) for x in hp]
    tol = 2e-6 if f32 else 1e-12
    for scheme in ("euler", "ab2") if f32 else ("euler", "ab2", "cn"):
        r = plan.momentum(ud, U_in, dt, nu, scheme=scheme, want_h=True,
                          h_prev=hd if scheme == "ab2" else None, cn_tol=1e-13)
        ref, href = step(m, u, nu, U_in, dt, scheme, hp)
        got = np.stack([host(x) for x in r["u_tilde"]])
        geth = np.stack([host(x) for x in r["h"]])
        assert rel_err(geth, href) <= tol, scheme
        assert rel_err(got, ref) <= (1e-11 if scheme == "cn" else tol), scheme
        assert r["report"].status == 0
