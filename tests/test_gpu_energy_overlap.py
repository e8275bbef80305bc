"""The kinetic-energy objective and its seed where outputs lie over inputs: in place (component by
component, the batched loop's case), over another component (cell by cell), and apart, on cube
sizes on both sides of the batched loop's limit.  Same sums in every case that does not change
its own input; 1e-13 against numpy covers a sum of 3 x 8192 squares (n eps = 6e-12 at the
very most, 1e-15 for a tree of partial sums)."""
import ctypes

import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, uniform_mesh, uniform_random_velocity

from gpu_util import dev, host, plan_for, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _call(plan, u, g, rho=1.3, scale=0.7):
    J = ctypes.c_double()
    arr = ctypes.c_void_p * 3
    st = plan._lib.bcm_kinetic_energy(plan.handle, arr(*[x.data_ptr() for x in u]), rho, scale,
                                      ctypes.byref(J), arr(*[x.data_ptr() for x in g]), None)
    assert st == 0
    return J.value


@pytest.mark.parametrize("n,dims", [(16, (2, 1, 1)), (8, (2, 2, 2)), (4, (3, 2, 1)), (2, (1, 1, 1))])
@pytest.mark.parametrize("precision", ["fp64", "mixed_f32fields"])
def test_seed_over_inputs(n, dims, precision):
    m = uniform_mesh(dims, 0.5, n, CHANNEL_BC)
    plan = plan_for(m, precision)
    dt = plan.field_dtype
    u0 = uniform_random_velocity(m, 21, 0.5, (1.0, 0.0, 0.0)).reshape(3, -1)
    fresh = lambda: [dev(v, dt) for v in u0]  # noqa: E731
    u, g = fresh(), [plan.empty() for _ in range(3)]
    J = _call(plan, u, g)
    V = float(m.h()[0]) ** 3
    x = np.stack([host(v).astype(np.float64) for v in u])
    assert abs(J - 0.5 * 1.3 * V * (x * x).sum()) <= 1e-13 * J
    u = fresh()
    assert _call(plan, u, u) == J                       # in place
    assert all(np.array_equal(host(a), host(b)) for a, b in zip(u, g))
    u = fresh()
    over = [plan.empty(), plan.empty(), u[0]]           # written after its cells are read
    assert _call(plan, u, over) == J
    assert all(np.array_equal(host(a), host(b)) for a, b in zip(over, g))
