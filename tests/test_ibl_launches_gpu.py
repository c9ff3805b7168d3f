"""The image-based-lighting launches at the sizes where their split changes:
mip chains of one, two and three launches (and none), blocks of less than a whole
chain step, BRDF-table sample counts at which the table leaves the integral launch
or its LDS rows, one level only, and cubes that are no power of two."""
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


def _p(irr=4, src=8, pref=8, levels=3, samples=32, lut=8, lut_samples=32, fis=0):
    return dict(irr_size=irr, irr_src_size=src, pref_size=pref, pref_levels=levels, pref_samples=samples, lut_size=lut,
                lut_samples=lut_samples, pref_fis=fis)


CASES = [(2, _p(levels=1, fis=1)), (2, _p(src=2, levels=1)), (4, _p(levels=2, fis=1)), (8, _p(fis=1)),
         (32, _p(pref=32, levels=5, fis=1)), (64, _p(pref=16, levels=4, samples=700, fis=1)),
         (128, _p(pref=16, levels=4, samples=900, fis=1)), (2048, _p(src=16, pref=16, levels=4, samples=2, fis=1)),
         (48, _p(irr=5, src=12, pref=20, levels=3, samples=65)), (16, _p(irr=33, src=16, levels=1)),
         (16, _p(lut=33, lut_samples=1023)), (16, _p(lut=33, lut_samples=1025)), (16, _p(lut=5, lut_samples=2048)),
         (16, _p(lut=5, lut_samples=2049)), (16, _p(levels=3, samples=129))]


@pytest.mark.parametrize("size,p", CASES)
def test_ibl_launch_edges(size, p):
    from paper_2012_03325_amd import frame as fr
    env = synth.env_sky_gradient(size)
    ref = O.precompute_ibl(env, **p)
    ibl = fr.DeviceIBL(env, **p)
    for t in (ibl.irr, ibl.pref, ibl.lut):
        t.fill_(float("nan"))
    ibl.scratch.fill_(255)  # nothing may depend on what the scratch held
    ibl.precompute()
    torch.cuda.synchronize()
    # tolerances of the IBL parity tests: 1e-4 for sums of float32 terms, 2e-6 absolute for the O(1) table
    assert_interval("irradiance", ibl.irr.cpu().numpy()[..., :3], ref["irradiance"][..., :3],
                    ref["irradiance"][..., :3], rtol=1e-4)
    for m, (g, r, rh) in enumerate(zip(ibl.pref_levels(), ref["prefiltered"], ref["prefiltered_hi"])):
        assert_interval(f"prefiltered {m}", g.cpu().numpy()[..., :3], r[..., :3], rh[..., :3])
    assert_interval("table", ibl.lut.cpu().numpy(), ref["lut"], ref["lut"], rtol=1e-4, atol=2e-6)
    assert not np.isnan(ibl.pref.cpu().numpy()).any() and not np.isnan(ibl.irr.cpu().numpy()).any()
