"""The ray caster where a wavefront meets most of 64 spheres, which it then takes two at a
time: clusters within some pixels of a large image, odd and even numbers of them, equal
hits among them, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as O
from paper_2012_03325_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _cast(sc, cam):
    from paper_2012_03325_amd import frame as fr
    g = {k: v.cpu().numpy() for k, v in fr.DeviceScene(sc).render_gbuffer(cam).items()}
    torch.cuda.synchronize()
    return g


@pytest.mark.parametrize("n,away", [(33, 60.0), (64, 60.0), (65, 60.0), (97, 20.0), (500, 8.0), (1023, 8.0),
                                    (1024, 30.0)])
def test_cluster(n, away):
    sc = synth.make_spheres(np.random.default_rng(n), n, True)
    cam = synth.look_at((0, 3.5 * away / 8.5, away), (0, 0, 0), (0, 1, 0), 45, 1025, 1024)
    ref = O.raycast(sc, cam)
    ok = ref["ambiguous"] == 0
    g = _cast(sc, cam)
    depth = ref["depth"].astype(np.float32)
    hit = ok & np.isfinite(depth)
    assert np.array_equal(np.isfinite(g["depth"])[ok], np.isfinite(depth)[ok])
    # the double-precision depth rounded to float32 (one unit for the order of its operations)
    assert np.abs(g["depth"][hit].view(np.int32) - depth[hit].view(np.int32)).max() <= 1
    for k in ("albedo", "roughness", "metalness"):
        assert np.array_equal(g[k][..., ok], ref[k].astype(np.float32)[..., ok]), k


def test_equal_hits_in_a_cluster():
    """Every sphere three times over, in shuffled order: the first copy's material wins."""
    rng = np.random.default_rng(5)
    base = synth.make_spheres(rng, 300, False)
    order = rng.permutation(900) % 300
    first = np.array([np.nonzero(order == k)[0][0] for k in range(300)])
    sc = synth.SphereScene(base.centers[order], base.radii[order], rng.uniform(0, 1, (900, 3)),
                           rng.uniform(0.05, 1, 900), np.zeros(900))
    one = synth.SphereScene(base.centers, base.radii, sc.albedo[first], sc.roughness[first], np.zeros(300))
    cam = synth.look_at((0, 15, 40), (0, 0, 0), (0, 1, 0), 45, 1025, 1024)
    a, b = _cast(sc, cam), _cast(one, cam)
    assert np.isfinite(a["depth"]).any()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
