"""SSAO's two depth sources at their borders: images of up to 3 * 2^19 pixels
(3 * 2^20 in a batch) gather the full-resolution depth, larger ones a compact
copy.  Raw and blurred AO against the FP64 oracle on both sides, for even and odd
sizes (an odd plane's last element is half a pair), and batches that take other
sources than the single views, or mix them, bitwise equal to those."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2012_03325_amd import synth
from tests.parity_util import AO_ATOL, assert_interval

pytestmark = pytest.mark.gpu

_views = {}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    _views.clear()
    torch.cuda.synchronize()


def _device_view(w, h):
    from paper_2012_03325_amd import frame as fr
    if (w, h) not in _views:
        v = synth.config_reduced(w, h, seed=31, shadow_size=0, env_size=8, ssao_n=9, n_spheres=32)
        v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
        ibl = fr.DeviceIBL(v.env, **v.ibl)
        ibl.precompute()
        _views[(w, h)] = v, fr.DeviceView(v, ibl)
    return _views[(w, h)]


# direct; direct; compact; compact (in a batch direct); compact
SIZES = [(2048, 768), (1537, 1023), (2049, 768), (1537, 2045), (1539, 2045)]


@pytest.mark.parametrize("w,h", SIZES)
def test_ssao_depth_source(w, h):
    v, dv = _device_view(w, h)
    g = v.gbuf
    lo, hi = O.ssao_raw(g["depth"], g["normal"], v.cam, v.ssao_kernel, v.ssao_noise, v.ssao_radius, v.ssao_bias)
    blo, bhi = O.ssao_blur(lo, hi, g["depth"], v.blur_tau)
    dv.ssao(blur=False)
    assert_interval(f"raw {w}x{h}", dv.ao.cpu().numpy(), lo, hi, rtol=0.0, atol=AO_ATOL)
    dv.ssao(blur=True)
    assert_interval(f"blurred {w}x{h}", dv.ao.cpu().numpy(), blo, bhi, rtol=0.0, atol=AO_ATOL)


@pytest.mark.parametrize("sizes", [SIZES[1:] + [(33, 17)], SIZES[:4] + [(2048, 1536)]])  # mixed; all direct
@pytest.mark.parametrize("kw", [dict(), dict(ssao_tile=1), dict(ssao_tile=2), dict(persistent=16)])
def test_batch_mixes_depth_sources(sizes, kw):
    from paper_2012_03325_amd import frame as fr
    dvs = [_device_view(w, h)[1] for w, h in sizes]
    solo = []
    for dv in dvs:
        dv.ssao()
        solo.append(dv.ao.clone())
        dv.ao.fill_(-1)
    fr.DeviceBatch(dvs, fr.make_schedule(**kw)).render()
    torch.cuda.synchronize()
    for dv, ao in zip(dvs, solo):
        assert np.array_equal(dv.ao.cpu().numpy(), ao.cpu().numpy())
