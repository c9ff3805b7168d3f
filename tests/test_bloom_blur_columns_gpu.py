"""The bloom blur's tiles (60 columns by four rows a wavefront in a single view, eight
in a batch): level sizes of one texel, below, at and beyond a tile's columns and
rows, against the FP64 oracle, and the batch bitwise equal to the single view."""
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


# level 1 of 1 x 1, 3 x 2, 59 x 15, 60 x 16, 61 x 17, 62 x 31, 120 x 32, 121 x 33, 64 x 65 texels
@pytest.mark.parametrize("w,h", [(1, 1), (5, 3), (118, 30), (120, 32), (122, 34), (124, 61), (240, 64), (241, 65),
                                 (127, 130)])
@pytest.mark.parametrize("half", [0, 1])
def test_bloom_blur_columns(w, h, half):
    from paper_2012_03325_amd import epb as E, frame as fr
    v = synth.config_reduced(w, h, seed=43, shadow_size=0, env_size=8, ssao_n=2, n_spheres=16)
    v.ibl = dict(irr_size=4, irr_src_size=8, pref_size=8, pref_levels=2, pref_samples=16, lut_size=8, lut_samples=16)
    ibl = fr.DeviceIBL(v.env, **v.ibl)
    ibl.precompute()
    t = E.EPB_F16 if half else E.EPB_F32
    dv = fr.DeviceView(v, ibl, gdtype=t, ao_dtype=t, hdr_dtype=t)
    dv.render()
    if not half:
        ref = O.bloom_tonemap(dv.hdr.cpu().numpy().astype(np.float64), levels=6, threshold=v.bloom_threshold,
                              strength=v.bloom_strength, exposure=v.exposure, gamma=v.gamma, tonemap=v.tonemap,
                              want_pyramid=True)
        for l, (g, r) in enumerate(zip(dv.pyramid(), ref["pyramid"])):
            gg = g.cpu().numpy()[..., :3].transpose(2, 0, 1)
            # sums of float32 terms at rtol 1e-5; near the threshold the bright pass takes the difference
            # of luminances of order 1, each known to a few 2^-24
            assert_interval(f"level {l + 1}", gg, r, r, rtol=1e-5, atol=1e-6)
    one = dv.ldr.clone()
    for kw in (dict(), dict(persistent=8)):
        dv.ldr.fill_(7)
        fr.DeviceBatch([dv], fr.make_schedule(**kw)).render()
        torch.cuda.synchronize()
        assert torch.equal(one, dv.ldr), kw
