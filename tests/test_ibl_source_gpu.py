"""The irradiance source by segments of one face or of all six: sizes on both sides of
the line (16384 threads a face), from one texel a face to the environment's own size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from tests.parity_util import assert_interval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("size,src", [(64, 1), (12, 3), (40, 5), (128, 16), (128, 32), (256, 32), (128, 128),
                                      (129, 129), (2, 1)])
def test_source(size, src):
    from paper_2012_03325_amd import frame as fr
    env = np.random.default_rng(size + src).uniform(0.0, 4.0, (6, size, size, 4)).astype(np.float32)
    env[1] *= 3.0
    env[4, : size // 2] *= 5.0
    p = dict(irr_size=3, irr_src_size=src, pref_size=2, pref_levels=1, pref_samples=1, lut_size=2, lut_samples=1)
    ref = O.precompute_ibl(env, **p)["irradiance"][..., :3]
    ibl = fr.DeviceIBL(env, **p)
    ibl.irr.fill_(float("nan"))
    ibl.scratch.fill_(255)
    ibl.precompute()
    torch.cuda.synchronize()
    # the tolerance of the tables' parity tests for sums of float32 terms
    assert_interval(f"irradiance from 6x{src}^2", ibl.irr.cpu().numpy()[..., :3], ref, ref, rtol=1e-4)
