"""The shading pass's tile order: every tile is shaded exactly once for tile
counts around a round of chunks (512 tiles), one workgroup per tile and looping
workgroups, and the images are those of the other tile shapes."""
import numpy as np
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


# tiles of 32 x 8: 7, 511, 512, 513, 1024 and 1031 (one row)
@pytest.mark.parametrize("w,h", [(32 * 7, 8), (32 * 73, 8 * 7), (32 * 32, 8 * 16), (32 * 27 - 5, 8 * 19 - 3),
                                 (32 * 32 - 31, 8 * 32 - 7), (16384, 8 * 2 + 1)])
def test_every_tile_once(w, h):
    from paper_2012_03325_amd import frame as fr
    v = synth.config_reduced(w, h, seed=17, shadow_size=32, env_size=8, ssao_n=1, n_spheres=12, n_lights=2)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    dv = fr.DeviceView(v, ibl)
    dv.hdr.fill_(float("nan"))
    dv.render()
    hdr = dv.hdr.cpu().numpy()
    assert np.isfinite(hdr).all()
    for kw in (dict(), dict(shade_tile=1), dict(shade_tile=2), dict(blocks_per_cu=1), dict(fuse_bloom=1)):
        dv.hdr.fill_(float("nan"))
        fr.DeviceBatch([dv], fr.make_schedule(**kw)).render()
        torch.cuda.synchronize()
        assert np.array_equal(dv.hdr.cpu().numpy(), hdr), kw
