"""The copy u* = u~ of the particle forcing on fields of more than 8192 workgroups' first round
(134 MB), with a number of 16-byte words that is no multiple of a workgroup's 1024: every cell of
each component, and nothing around it."""
import pytest
import torch

from bcm_inputs import CHANNEL_BC, uniform_mesh

from gpu_util import plan_for, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]


def test_every_cell_of_a_field_beyond_one_round():
    m = uniform_mesh((33, 33, 31), 0.25, 8, CHANNEL_BC)
    words = m.n_cells * 8 // 16
    assert words > 8192 * 1024 and words % 1024 != 0
    plan = plan_for(m, "fp64")
    gen = torch.Generator(device="cuda").manual_seed(51)
    u = [torch.rand(m.n_cells, generator=gen, device="cuda", dtype=torch.float64) for _ in range(3)]
    buf = [torch.full((m.n_cells + 16,), -7.0, device="cuda", dtype=torch.float64) for _ in range(3)]
    out = [b[8:-8] for b in buf]
    none = torch.zeros(0, 3, dtype=torch.float64, device="cuda")
    plan.ib_force(u, none, 0.01, 1.0, out=out)
    for a, b, o in zip(u, buf, out):
        assert torch.equal(a, o)
        assert bool((b[:8] == -7.0).all()) and bool((b[-8:] == -7.0).all())
