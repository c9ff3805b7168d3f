"""Compositing without a pyramid on images of more than 1536 strips, which takes a kernel
of its own: the single view's image bitwise equal to a batch's, which takes the general one."""
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03325_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("tonemap", [0, 1])
@pytest.mark.parametrize("w,h", [(1024, 769), (1031, 781), (16384, 56), (63, 12297)])
def test_no_bloom(w, h, tonemap, half):
    from paper_2012_03325_amd import epb as E, frame as fr
    v = synth.config_reduced(w, h, seed=43, shadow_size=0, env_size=8, ssao_n=2, n_spheres=16)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    v.tonemap = E.EPB_TONEMAP_REINHARD if tonemap else E.EPB_TONEMAP_ACES
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    t = E.EPB_F16 if half else E.EPB_F32
    dv = fr.DeviceView(v, ibl, gdtype=t, ao_dtype=t, hdr_dtype=t, bloom_levels=1)
    dv.render()
    one = dv.ldr.clone()
    dv.ldr.fill_(7)
    fr.DeviceBatch([dv]).render()
    torch.cuda.synchronize()
    assert torch.equal(one, dv.ldr)
