"""SSAO's raw values and blur in one kernel: 8 x 8 tiles while an image has at most
256 of them, 13 x 13 tiles up to a line on size and sample count, two kernels
beyond.  Blurred AO against the FP64 oracle at the edges of tiles and on both sides
of each line, and bitwise against a batch of the same view (which keeps the two
kernels)."""
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


# 8 x 8 tiles: one texel, a remainder of one, whole tiles, the most tiles; 13 x 13 tiles: one
# tile row more, remainders of one, whole tiles; one kernel / two kernels: 64 / 65 samples with
# one wavefront per SIMD more; two kernels
@pytest.mark.parametrize("w,h,n,half", [
    (1, 1, 9, 0), (17, 33, 8, 1), (32, 16, 17, 0), (256, 256, 9, 1),
    (258, 256, 9, 0), (391, 417, 7, 1), (416, 390, 16, 0),
    (800, 600, 64, 1), (800, 600, 65, 0), (1280, 720, 33, 1)])
def test_ssao_one_kernel(w, h, n, half):
    from paper_2012_03325_amd import epb as E, frame as fr
    v = synth.config_reduced(w, h, seed=37, shadow_size=0, env_size=8, ssao_n=n, n_spheres=32)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    g = v.gbuf
    lo, hi = O.ssao_raw(g["depth"], g["normal"], v.cam, v.ssao_kernel, v.ssao_noise, v.ssao_radius, v.ssao_bias)
    blo, bhi = O.ssao_blur(lo, hi, g["depth"], v.blur_tau)
    dv = fr.DeviceView(v, ibl)
    dv.ssao()
    one = dv.ao.cpu().numpy()
    assert_interval(f"blurred {w}x{h} n={n}", one, blo, bhi, rtol=0.0, atol=AO_ATOL)
    dt = E.EPB_F16 if half else E.EPB_F32
    dv = fr.DeviceView(v, ibl, gdtype=dt, ao_dtype=dt, hdr_dtype=dt)
    dv.ao.fill_(-1)
    dv.ssao()
    one = dv.ao.clone()
    dv.ao.fill_(-1)
    fr.DeviceBatch([dv]).render()
    torch.cuda.synchronize()
    assert np.array_equal(one.cpu().numpy(), dv.ao.cpu().numpy())
