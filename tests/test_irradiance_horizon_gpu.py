"""The irradiance sums leave out groups of four source texels behind a wavefront's
horizon: output sizes with and without 8 x 8 tiles, source counts that are no multiple
of four or of the 256 a wavefront tests at once, chunks of one group and empty ones,
light from one direction only, and source texels that are no finite numbers (which
reach every output, also those that they lie behind)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2012_03325_amd import synth
from tests.parity_util import assert_interval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _run(env, irr, src):
    from paper_2012_03325_amd import frame as fr
    p = dict(irr_size=irr, irr_src_size=src, pref_size=2, pref_levels=1, pref_samples=2, lut_size=2, lut_samples=2)
    ibl = fr.DeviceIBL(env, **p)
    ibl.irr.fill_(float("nan"))
    ibl.scratch.fill_(255)
    ibl.precompute()
    torch.cuda.synchronize()
    return ibl.irr.cpu().numpy()[..., :3], p


# 6, 150, 486 and 24576 sources; 264600 in 1024 chunks of 259, the last of which starts past the end
@pytest.mark.parametrize("irr,src", [(8, 1), (8, 5), (16, 9), (24, 16), (40, 8), (7, 9), (2, 5), (16, 64), (4, 210)])
@pytest.mark.parametrize("spot", [0, 1])
def test_irradiance_horizon(irr, src, spot):
    size = max(src, 2)
    env = np.array(synth.env_sky_gradient(size))
    if spot:  # dark but for one texel of +X and one of -Y
        env[..., :3] = 0.0
        env[0, size // 2, size // 3, :3] = (1000.0, 1.0, 0.001)
        env[3, 0, size - 1, :3] = (0.5, 250.0, 3.0)
    got, p = _run(env, irr, src)
    ref = O.precompute_ibl(env, **p)["irradiance"][..., :3]
    # the parity tolerance of sums of float32 terms; a texel near a spot's horizon takes a cosine that
    # float32 knows to 2^-23 of 1 only, times the spot's weight
    atol = 1000.0 * 4 / (6 * src * src) * 2.0 ** -21 if spot else 0.0
    assert_interval(f"irradiance {irr} from {src}", got, ref, ref, rtol=1e-4, atol=atol)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_irradiance_of_a_non_finite_texel(value):
    env = np.array(synth.env_sky_gradient(16))
    env[2, 3, 4, 1] = value
    got, _ = _run(env, 16, 16)
    assert not np.isfinite(got[..., 1]).any()
    assert np.isfinite(got[..., 0]).all() and np.isfinite(got[..., 2]).all()
