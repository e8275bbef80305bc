"""The codec on more cubes than one round of its scans takes: 16767 cubes of 4^3 are three rounds
of the offset scan (8192 sizes each, the last one partial), seventeen of the verdict's, and more
units than the encoder and the decoder have workgroups.  The stream equals the oracle's byte for
byte, the decoded field bit for bit, and a value that is not finite, or a damaged cube, is seen in
each of the rounds."""
import numpy as np
import pytest

from bcm_inputs import OPEN_BC, uniform_mesh
from oracle import codec as C

from gpu_util import dev, host, plan_for, requires_gpu

pytestmark = [pytest.mark.gpu, requires_gpu]

STEP = 1e-2


@pytest.fixture(scope="module")
def case():
    m = uniform_mesh((27, 27, 23), 1.0 / 27.0, 4, OPEN_BC)
    rng = np.random.default_rng(21)
    # sizes that differ from cube to cube, empty ones among them
    x = rng.standard_normal((m.n_cubes, 64)) * 10.0 ** rng.integers(-4, 4, (m.n_cubes, 1))
    return m, x.ravel(), plan_for(m, "fp64")


def test_stream_and_decoded_field(case):
    m, x, plan = case
    ref = C.compress(x, 4, m.n_cubes, STEP)
    s = plan.compress(dev(x), STEP)
    assert s.cpu().numpy().tobytes() == ref
    assert np.array_equal(host(plan.decompress(s)), C.decompress(ref))


@pytest.mark.parametrize("cube", [0, 8191, 8192, 16383, 16384, 16766])
def test_a_bad_cube_in_any_round_is_reported(case, cube):
    from paper_1808_04099_amd import BCMError
    m, x, plan = case
    y = x.copy()
    y[64 * cube + 5] = np.nan
    with pytest.raises(BCMError, match="not finite|non-finite"):
        plan.compress(dev(y), STEP)
    s = plan.compress(dev(x), STEP).clone()
    offs = np.frombuffer(s.cpu().numpy().tobytes(), dtype="<u8", count=m.n_cubes + 1, offset=32)
    good = host(plan.decompress(s)).reshape(m.n_cubes, 64)
    s[32 + 8 * (m.n_cubes + 1) + int(offs[cube])] = 33      # a group width beyond 32
    out = plan.empty(plan.field_dtype)
    with pytest.raises(BCMError, match="malformed"):
        plan.decompress(s, out=out)
    got = host(out).reshape(m.n_cubes, 64)
    assert not got[cube].any()
    rest = np.arange(m.n_cubes) != cube
    assert np.array_equal(got[rest], good[rest])
