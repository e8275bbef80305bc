"""The 16^3 kernels of the face-velocity output and of the adjoint against the oracle, on a
single-level channel, an open box and a two-level mesh (2:1 faces on every axis): every face
value, cells in cubes without a body (whose u* is not stored), u_s as constants and as fields,
accumulated alpha cotangents, with and without a body.  Tolerances of test_gpu_projection.py and
test_gpu_adjoint.py: 1e-7 relative (solves at 1e-12), 1e-5 with FP32 fields."""
import numpy as np
import pytest

from bcm_inputs import CHANNEL_BC, OPEN_BC, build_mesh, uniform_mesh, uniform_random_velocity
from oracle import projection as OP
from oracle.fv import FVMesh

from gpu_util import dev, host, plan_for, rel_err, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

MIXED = ("inflow", "outflow", "slip", "outflow", "inflow", "slip")
MESHES = {
    "channel": lambda: uniform_mesh((3, 2, 1), 0.5, 16, CHANNEL_BC),
    "open": lambda: uniform_mesh((1, 2, 2), 0.5, 16, OPEN_BC),
    "two_level": lambda: build_mesh((2, 2, 2), 0.5, 16, MIXED, max_level=1,
                                    refine=lambda lv, lo, hi: bool(np.all(lo < 0.2))),
}


def _case(name, f32, body):
    m = MESHES[name]()
    rng = np.random.default_rng(41)
    u = uniform_random_velocity(m, 42, 0.4, (1.0, 0.0, 0.0)).reshape(3, -1)
    alpha = np.zeros((m.n_cubes, m.n ** 3))
    if body:
        alpha[::2] = rng.uniform(0.0, 1.0, alpha[::2].shape)   # every other cube holds the body
    alpha = alpha.ravel()
    us = rng.standard_normal((3, m.n_cells))
    if f32:
        u, alpha, us = (x.astype(np.float32).astype(np.float64) for x in (u, alpha, us))
    return m, u, alpha, us


def _cell_faces(fv, U):
    """Face values on the minus and plus side of every cell along each axis ([3][2][cells]; the
    coarse side of a 2:1 face has the mean of its four sub-faces)."""
    out = np.zeros((3, 2, fv.n_cells))
    cnt = np.zeros((3, 2, fv.n_cells))
    for side, cell in ((1, fv.L), (0, fv.R)):
        ok = cell >= 0
        np.add.at(out, (fv.axis[ok], side, cell[ok]), U[ok])
        np.add.at(cnt, (fv.axis[ok], side, cell[ok]), 1)
    return out / cnt


@pytest.mark.parametrize("precision", ["fp64", "mixed_f32fields"])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_face_velocities(name, precision):
    f32 = precision == "mixed_f32fields"
    m, u, alpha, us = _case(name, f32, True)
    n = m.n
    fv = FVMesh(m)
    plan = plan_for(m, precision, tol=1e-12)
    ft = plan.field_dtype
    U_in, dt, rho = 0.9, 0.01, 1.1
    r = plan.project([dev(x, ft) for x in u], dev(alpha, ft), U_in, dt, rho,
                     us=[dev(x, ft) for x in us], face_u=True)
    ref = OP.project(fv, u, alpha, us, U_in, dt, rho)
    tol = 1e-5 if f32 else 1e-7
    assert rel_err(np.stack([host(x) for x in r["u_new"]]), ref["u_new"]) <= tol
    want = _cell_faces(fv, ref["U_new"]).reshape(3, 2, m.n_cubes, n, n, n)
    for d in range(3):
        sh = [m.n_cubes] + [n + (1 if 2 - a == d else 0) for a in range(3)]
        got = host(r["face_u"][d]).reshape(sh)
        ax = 3 - d
        lo, hi = np.take(got, range(n), axis=ax), np.take(got, range(1, n + 1), axis=ax)
        scale = np.abs(want[d]).max()
        assert np.abs(lo - want[d, 0]).max() <= tol * scale, d
        assert np.abs(hi - want[d, 1]).max() <= tol * scale, d


@pytest.mark.parametrize("body", [True, False])
@pytest.mark.parametrize("precision", ["fp64", "mixed_f32fields"])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_adjoint(name, precision, body):
    f32 = precision == "mixed_f32fields"
    m, u, alpha, us = _case(name, f32, body)
    rng = np.random.default_rng(43)
    gu = rng.standard_normal((3, m.n_cells))
    gp = rng.standard_normal(m.n_cells)
    ga0 = rng.standard_normal(m.n_cells)
    if f32:
        gu, ga0 = (x.astype(np.float32).astype(np.float64) for x in (gu, ga0))
    U_in, dt, rho = 0.9, 0.02, 1.1
    fv = FVMesh(m)
    plan = plan_for(m, precision, tol=1e-12)
    ft = plan.field_dtype
    ud, gd = [dev(x, ft) for x in u], [dev(x, ft) for x in gu]
    tol = 1e-5 if f32 else 1e-7
    for us_np, us_dev in (((0.1, 0.0, -0.05), (0.1, 0.0, -0.05)), (us, [dev(x, ft) for x in us])):
        g_ut, g_us, gU, lam = OP.project_adjoint(fv, u, alpha, us_np, U_in, dt, rho, gu, gp=gp)
        for acc in (False, True) if body else (False,):
            g_u, g_a, g_U, rep, lam_g = plan.project_adjoint(
                ud, dev(alpha, ft) if body else None, gd, U_in, dt, rho, us=us_dev, g_p=dev(gp),
                want_lambda=True, accumulate=acc, g_alpha=dev(ga0, ft) if acc else None,
                g_U_in=2.5 if acc else 0.0)
            assert rep.status == 0
            assert rel_err(np.stack([host(x) for x in g_u]), g_ut) <= tol
            assert rel_err(host(lam_g), lam) <= tol
            assert abs(g_U - (2.5 if acc else 0.0) - gU) <= tol * max(abs(gU), 1.0)
            if body:
                g_al = OP.alpha_gradient(g_us, u, us_np) + (ga0 if acc else 0.0)
                assert rel_err(host(g_a), g_al) <= tol
