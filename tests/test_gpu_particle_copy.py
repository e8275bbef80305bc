"""The copy u* = u~ of the particle forcing: whole fields of every cube size, 16-byte aligned
buffers (one kernel), buffers that are not, and an output laid over another component's input
(copies in turn).  One particle touches each cell once, so the fields are the same bits on every
route, and u~ exactly away from its support."""
import numpy as np
import pytest
import torch

from bcm_inputs import CHANNEL_BC, uniform_mesh, uniform_random_velocity

from gpu_util import dev, host, plan_for, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("n,dims", [(2, (1, 1, 1)), (2, (5, 3, 3)), (4, (3, 3, 3)), (8, (5, 2, 1)), (16, (3, 2, 1))])
@pytest.mark.parametrize("precision", ["fp64", "mixed_f32fields"])
def test_every_cell_is_copied_once(n, dims, precision):
    m = uniform_mesh(dims, 0.5, n, CHANNEL_BC)
    plan = plan_for(m, precision)
    u = uniform_random_velocity(m, 11, 0.5, (1.0, 0.0, 0.0)).reshape(3, -1)
    if m.n_cells < 27:                    # no support fits: the plain copy
        X, moved = torch.zeros(0, 3, dtype=torch.float64, device="cuda"), 0
    else:
        X, moved = dev(np.array([[0.25 * d + 0.01 for d in dims]])), 27
    dt = plan.field_dtype
    result = {}
    for off in (0, 1, 3):
        bufs = [torch.full((m.n_cells + 8,), -7.0, dtype=dt, device="cuda") for _ in range(6)]
        src, out = [b[off:off + m.n_cells] for b in bufs[:3]], [b[off:off + m.n_cells] for b in bufs[3:]]
        for d in range(3):
            src[d].copy_(dev(u[d], dt))
        plan.ib_force(src, X, 0.01, 1.0, Us=(0.0, 0.0, 0.0), out=out)
        result[off] = [host(o) for o in out]
        for d in range(3):
            assert np.count_nonzero(result[off][d] != host(src[d])) <= moved
            assert np.array_equal(host(src[d]), host(dev(u[d], dt)))
            b = host(bufs[3 + d])
            assert np.all(b[:off] == -7.0) and np.all(b[off + m.n_cells:] == -7.0)
    for off in (1, 3):
        assert all(np.array_equal(a, b) for a, b in zip(result[0], result[off]))


def test_output_over_another_component():
    m = uniform_mesh((2, 2, 2), 0.5, 8, CHANNEL_BC)
    plan = plan_for(m, "fp64")
    u = uniform_random_velocity(m, 12, 0.5, (1.0, 0.0, 0.0)).reshape(3, -1)
    src = [dev(v) for v in u]
    out = [plan.empty(), src[0], plan.empty()]
    plan.ib_force(src, torch.zeros(0, 3, dtype=torch.float64, device="cuda"), 0.01, 1.0, out=out)
    assert all(np.array_equal(host(o), v) for o, v in zip(out, u))
