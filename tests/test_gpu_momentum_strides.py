"""The momentum pass on more units than it has workgroups (2048), where a workgroup takes a second
unit, and on fields of 4 GiB and more, where its byte offsets have 64 bits.  Explicit steps against
the oracle (1e-12 relative, the bound of every explicit FP64 step); Crank-Nicolson by its equation,
with the oracle's H: the residual of the result at the tolerance asked for (1e-12, and rounding
1e-13 beside it), and the reported norm of the first iterate's residual to 1e-9."""
import numpy as np
import pytest
import torch

from bcm_inputs import CHANNEL_BC, OPEN_BC, uniform_mesh, uniform_random_velocity
from oracle.momentum import MomentumGrid

from gpu_util import dev, host, log, plan_for, rel_err, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("n,dims", [(4, (33, 33, 31)), (16, (13, 13, 13))])
def test_workgroups_that_take_two_units(n, dims):
    m = uniform_mesh(dims, 0.25, n, CHANNEL_BC)
    u = uniform_random_velocity(m, 41, 0.6, (0.3, -0.2, 0.1)).reshape(3, -1)
    hp = uniform_random_velocity(m, 42, 2.0).reshape(3, -1)
    h = float(m.h()[0])
    nu, U_in, dt = 0.3 * h, 0.7, 0.4 * h
    plan = plan_for(m, "fp64")
    mg = MomentumGrid(m)
    ug = [mg.to_global(x) for x in u]
    Hu = mg.H(ug, ug, nu, U_in)
    cubes = lambda g: np.stack([mg.to_cubes(x).reshape(-1) for x in g])
    norm = lambda g: np.sqrt(sum(float((x * x).sum()) for x in g))
    log(f"  {m.n_cubes} cubes of {n}^3: oracle ready")
    ud, hd = [dev(x) for x in u], [dev(x) for x in hp]
    r = plan.momentum(ud, U_in, dt, nu, scheme="ab2", want_h=True, h_prev=hd)
    href = cubes(Hu)
    assert rel_err(np.stack([host(x) for x in r["h"]]), href) <= 1e-12
    assert rel_err(np.stack([host(x) for x in r["u_tilde"]]), u + dt * (1.5 * href - 0.5 * hp)) <= 1e-12
    rhs = [a + 0.5 * dt * b for a, b in zip(ug, Hu)]

    def residual(x):
        Hx = mg.H(x, ug, nu, U_in)
        return [a + 0.5 * dt * b - c for a, b, c in zip(rhs, Hx, x)]

    one = plan.momentum(ud, U_in, dt, nu, scheme="cn", cn_max_iter=1, want_h=True)
    assert rel_err(np.stack([host(x) for x in one["h"]]), href) <= 1e-12
    first = residual([a + dt * b for a, b in zip(ug, Hu)])     # of the Euler predictor
    want = norm(first) / norm(rhs)
    assert abs(one["report"].final_rel_res - want) <= 1e-9 * want
    log("  first iterate checked")
    full = plan.momentum(ud, U_in, dt, nu, scheme="cn", cn_tol=1e-12)
    assert full["report"].status == 0
    got = [mg.to_global(host(x)) for x in full["u_tilde"]]
    assert norm(residual(got)) <= (1e-12 + 1e-13) * norm(rhs)


def test_fields_beyond_four_gib():
    """132651 cubes of 16^3 in FP64 (4.05 GiB a field).  A cube's result depends on its
    neighbours alone (8 cells away after three sweeps), so sampled cubes are compared with small
    meshes around them, which the pass with 32-bit offsets solves: the first and last cubes in
    memory, those on both sides of the 4 GiB line, and some between."""
    D = 51
    m = uniform_mesh((D, D, D), 1.0 / D, 16, OPEN_BC)
    assert m.n_cells * 8 > 0xFFFFFFFF
    torch.cuda.empty_cache()
    q = np.rint(m.origin * D).astype(int)
    at = {tuple(v): c for c, v in enumerate(q)}
    h = float(m.h()[0])
    nu, dt = 0.3 * h, 0.4 * h
    plan = plan_for(m, "fp64")
    gen = torch.Generator(device="cuda").manual_seed(43)
    u = [torch.rand(m.n_cells, generator=gen, device="cuda", dtype=torch.float64) - 0.5 for _ in range(3)]
    out = [torch.empty_like(x) for x in u]
    line = (1 << 32) // (4096 * 8)
    rng = np.random.default_rng(44)
    sample = [0, line - 1, line, line + 1, m.n_cubes - 1] + [int(c) for c in rng.integers(0, m.n_cubes, 5)]
    for scheme, its in (("euler", 0), ("cn", 3)):
        log(f"  {scheme} on {m.n_cells} cells")
        plan.momentum(u, 0.0, dt, nu, scheme=scheme, cn_tol=1e-15, cn_max_iter=its, out=out)
        for c in sample:
            lo, hi = np.maximum(q[c] - 1, 0), np.minimum(q[c] + 1, D - 1)
            sub = uniform_mesh(tuple(int(v) for v in hi - lo + 1), 1.0 / D, 16, OPEN_BC)
            sq = np.rint(sub.origin * D).astype(int)
            of = [at[tuple(v + lo)] for v in sq]
            su = [torch.cat([x[4096 * k:4096 * (k + 1)] for k in of]) for x in u]
            r = plan_for(sub, "fp64").momentum(su, 0.0, dt, nu, scheme=scheme, cn_tol=1e-15, cn_max_iter=its)
            k = of.index(c)
            for a, b in zip(out, r["u_tilde"]):
                assert rel_err(host(a[4096 * c:4096 * (c + 1)]), host(b[4096 * k:4096 * (k + 1)])) <= 1e-12, (scheme, c)
    del plan, u, out
    torch.cuda.empty_cache()
