"""SSAO's blur in a batch, by columns (61 of them by eight rows a wavefront), where a
single view's raw AO and blur are two kernels: half-resolution widths one short of,
at and one past whole tiles, heights with a remainder of none, one and two rows,
bitwise against the single view, and that against the FP64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2012_03325_amd import synth
from tests.parity_util import AO_ATOL, assert_interval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


# half-resolution 548 x 322, 549 x 320, 550 x 321 (61 * 9 = 549), and a compact depth copy
@pytest.mark.parametrize("w,h,n", [(1096, 643, 33), (1098, 640, 33), (1099, 641, 33), (2074, 767, 3)])
@pytest.mark.parametrize("half", [0, 1])
def test_ssao_blur_columns(w, h, n, half):
    from paper_2012_03325_amd import epb as E, frame as fr
    v = synth.config_reduced(w, h, seed=47, shadow_size=0, env_size=8, ssao_n=n, n_spheres=32)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    t = E.EPB_F16 if half else E.EPB_F32
    dv = fr.DeviceView(v, ibl, gdtype=t, ao_dtype=t, hdr_dtype=t)
    dv.ssao()
    one = dv.ao.clone()
    if not half:
        g = v.gbuf
        lo, hi = O.ssao_raw(g["depth"], g["normal"], v.cam, v.ssao_kernel, v.ssao_noise, v.ssao_radius, v.ssao_bias)
        blo, bhi = O.ssao_blur(lo, hi, g["depth"], v.blur_tau)
        assert_interval(f"blurred {w}x{h}", one.cpu().numpy(), blo, bhi, rtol=0.0, atol=AO_ATOL)
    for kw in (dict(), dict(persistent=8)):
        dv.ao.fill_(-1)
        fr.DeviceBatch([dv], fr.make_schedule(**kw)).render()
        torch.cuda.synchronize()
        assert np.array_equal(one.cpu().numpy(), dv.ao.cpu().numpy()), kw
