"""epb_shade_post on both sides of the image size up to which it forms bloom level 1
in the shading pass (3 * 2^20 pixels): HDR, 8-bit image and bloom scratch bitwise
those of epb_shade followed by epb_bloom_tonemap."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03325_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h", [(2048, 1536), (2049, 1536)])
@pytest.mark.parametrize("half", [False, True])
def test_shade_post_at_the_line(w, h, half):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2012_03325_amd import epb as E
    from paper_2012_03325_amd import frame as fr
    v = synth.config_reduced(w, h, seed=23, shadow_size=64, env_size=8, ssao_n=1, n_spheres=16, n_lights=2)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    t = E.EPB_F16 if half else E.EPB_F32
    dv = fr.DeviceView(v, ibl, gdtype=t, ao_dtype=t, hdr_dtype=t)
    dv.ssao()
    got = []
    for fused in (False, True):
        for x in (dv.hdr, dv.ldr, dv.postp.scratch):
            x.view(torch.uint8).fill_(0x3F)
        if fused:
            dv.shade_post()
        else:
            dv.shade()
            dv.bloom_tonemap()
        torch.cuda.synchronize()
        got.append([x.view(torch.uint8).cpu().numpy().copy() for x in (dv.hdr, dv.ldr, dv.postp.scratch)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
