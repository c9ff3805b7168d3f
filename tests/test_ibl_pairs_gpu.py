"""The plain prefilter from the environment itself and from its copy in pairs of texels:
sizes on both sides of the choice (more than 32 samples and at least half a lookup a texel of
the environment), against the oracle."""
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


# (environment, prefilter, levels, samples): lookups a texel from 0.44 to 0.53, 32 and 33 samples, ragged tables
@pytest.mark.parametrize("size,pref,levels,samples", [(64, 16, 2, 34), (64, 16, 2, 31), (64, 12, 2, 50), (32, 8, 2, 40), (32, 8, 2, 33),
                                                      (32, 32, 3, 32), (32, 32, 3, 33), (48, 20, 3, 129),
                                                      (48, 8, 2, 129), (2, 2, 1, 64), (6, 4, 2, 200)])
def test_prefilter(size, pref, levels, samples):
    from paper_2012_03325_amd import frame as fr
    env = np.random.default_rng(size + samples).uniform(0.0, 4.0, (6, size, size, 4)).astype(np.float32)
    env[2] *= 4.0
    p = dict(irr_size=2, irr_src_size=3 if size % 3 == 0 else 2, pref_size=pref, pref_levels=levels,
             pref_samples=samples, lut_size=2, lut_samples=1)
    ref = O.precompute_ibl(env, **p)
    ibl = fr.DeviceIBL(env, **p)
    ibl.pref.fill_(float("nan"))
    ibl.scratch.fill_(255)
    ibl.precompute()
    torch.cuda.synchronize()
    for m, (g, r, rh) in enumerate(zip(ibl.pref_levels(), ref["prefiltered"], ref["prefiltered_hi"])):
        assert_interval(f"prefiltered {m}", g.cpu().numpy()[..., :3], r[..., :3], rh[..., :3])
