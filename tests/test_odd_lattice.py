"""Box lattices with odd cube counts: the cube-graph hierarchy coarsens them to the size of the
dense bottom solve (host check of every level's operator), and the solves on them converge like
those on even lattices and agree with the oracle."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, OPEN_BC, uniform_mesh
from gpu_util import dev, host, plan_for, rel_err, requires_gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1808_04099_amd", "csrc")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("lattice_check") / "lattice_check")
    subprocess.run([gxx, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "lattice_check.cpp"),
                    os.path.join(CSRC, "mesh.cpp"), os.path.join(CSRC, "coarse.cpp"), "-o", out],
                   check=True, capture_output=True, timeout=300)
    return out


@pytest.mark.parametrize("open_all", [0, 1])
@pytest.mark.parametrize("dims", [(21, 13, 11), (5, 5, 5), (17, 9, 1), (10, 10, 10), (99, 1, 1),
                                  (16, 8, 8), (13, 13, 2)])
def test_hierarchy(checker, dims, open_all):
    r = subprocess.run([checker, *map(str, dims), str(open_all)], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr


# 12 iterations is what the even lattices of the same size need to 1e-10 (10 to 12); 16 leaves a
# third on top.  Errors: the residual bound 1e-10 times the conditioning that the other solver
# tests allow (1e-7 relative).
@pytest.mark.gpu
@requires_gpu
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("dims,bc", [((7, 5, 3), CHANNEL_BC), ((9, 5, 5), OPEN_BC),
                                     ((35, 3, 1), CHANNEL_BC)])
def test_solve_on_odd_lattice(dims, bc, precision):
    from oracle import UniformGrid
    m = uniform_mesh(dims, 0.25, 4, bc)
    b = np.random.default_rng(11).standard_normal(m.n_cells)
    plan = plan_for(m, precision)
    p, rep = plan.poisson_solve(dev(b))
    ug = UniformGrid(m)
    ref = ug.to_cubes(ug.solve(ug.to_global(b))).reshape(-1)
    assert rep.status == 0 and rep.final_rel_res <= 1e-10
    assert rep.n_inner <= 16, rep
    assert rel_err(host(p), ref) <= 1e-7
