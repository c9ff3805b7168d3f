"""The ray caster's depth map and G-buffer of the same camera, which take differently
shaped regions on large images: the same depths, in either attribute type."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2012_03325_amd import epb as E
from paper_2012_03325_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


# regions of 32 x 16 and 16 x 32 cut by the edges, on both sides of the line for few spheres and large images
@pytest.mark.parametrize("n,w,h", [(0, 1024, 1024), (1, 1025, 1025), (300, 1039, 1009), (1024, 2048, 513),
                                   (1025, 1025, 1025), (300, 1023, 1025), (300, 31, 16), (64, 16384, 65)])
def test_depth_map_equals_gbuffer(n, w, h):
    from paper_2012_03325_amd import frame as fr
    sc = synth.make_spheres(np.random.default_rng(n + w), n, True)
    d = fr.DeviceScene(sc)
    cam = synth.look_at((0, 3.5, 8.5), (0, 0, 0), (0, 1, 0), 45, w, h)
    depth = torch.full((h, w), float("nan"), device="cuda")
    d.render_depth(cam, depth)
    full, half = d.render_gbuffer(cam), d.render_gbuffer(cam, E.EPB_F16)
    torch.cuda.synchronize()
    assert not torch.isnan(depth).any()
    assert torch.equal(depth, full["depth"]) and torch.equal(depth, half["depth"])
    for k in ("normal", "albedo", "roughness", "metalness"):
        assert torch.equal(full[k].half(), half[k]), k
