"""Compositing by half strips (up to 1536 strips of 64 x 8 pixels in one image) and by
whole ones: heights that leave a strip one row, its first half, a row of its second
half and all rows, both sides of the line, every pyramid depth and storage type.
The single view's image bitwise equal to a batch's, which takes whole strips."""
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
@pytest.mark.parametrize("w,h,levels", [
    (64, 1, 6), (65, 4, 5), (63, 5, 4), (130, 12, 3), (64, 13, 2), (97, 40, 6), (33, 21, 1),
    (1024, 768, 6), (1024, 769, 6)])
def test_half_strips_equal_whole_strips(w, h, levels, half):
    from paper_2012_03325_amd import epb as E, frame as fr
    v = synth.config_reduced(w, h, seed=41, shadow_size=0, env_size=8, ssao_n=2, n_spheres=16)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    t = E.EPB_F16 if half else E.EPB_F32
    dv = fr.DeviceView(v, ibl, gdtype=t, ao_dtype=t, hdr_dtype=t, bloom_levels=levels)
    dv.render()
    one = dv.ldr.clone()
    dv.ldr.fill_(7)
    fr.DeviceBatch([dv]).render()
    torch.cuda.synchronize()
    assert torch.equal(one, dv.ldr)
