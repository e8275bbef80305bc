"""Cube-graph multigrid on meshes whose graph rows are wide (2:1 interfaces): a coarse cube with
finer neighbours on all six sides (24 couplings), one refined cube (9), and a checkerboard of
coarse and refined cubes (more wide nodes of one colour than a pass takes at once), smoothed by
one workgroup and by the multi-workgroup kernels.  Tolerances: the solve's own 1e-10 with the
rounding of the oracle's norm on top, and for p the conditioning that the other solver tests
allow."""
import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, OPEN_BC
from bcm_inputs.mesh import build_mesh
from oracle.fv import FVMesh

from gpu_util import dev, host, plan_for, rel_err, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def _mesh(dims, n, bc, pick):
    def refine(level, lo, hi):
        return pick(*(int(round(float(v) / 0.5)) for v in lo))
    return build_mesh(dims, 0.5, n, bc, refine=refine, max_level=1)


MESHES = {
    "coarse_centre": lambda: _mesh((3, 3, 3), 4, OPEN_BC, lambda i, j, k: (i, j, k) != (1, 1, 1)),
    "fine_centre": lambda: _mesh((5, 3, 3), 4, CHANNEL_BC, lambda i, j, k: (i, j, k) == (2, 1, 1)),
    "checkerboard": lambda: _mesh((10, 8, 8), 2, CHANNEL_BC, lambda i, j, k: (i + j + k) % 2 == 1),
}


@pytest.mark.parametrize("name", sorted(MESHES))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("split", [-1, 0])
def test_wide_rows(name, precision, split):
    m = MESHES[name]()
    fv = FVMesh(m)
    b = np.random.default_rng(31).standard_normal(m.n_cells)
    p, rep = plan_for(m, precision, graph_split=split).poisson_solve(dev(b))
    p = host(p)
    assert rep.status == 0 and fv.residual_norm(p, b) <= 1.2e-10
    assert rel_err(p, fv.solve(b)) <= 1e-7
