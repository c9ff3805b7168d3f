"""The environment chain of filtered sampling over three launches, which only the
largest cube has: one sample of the roughest level along each texel's direction
reads the chain's last level, whose four texels a face are the face's quadrants."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.parity_util import assert_interval

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _solid_angles(n):
    c = (2.0 * np.arange(n + 1) - n) / n
    x, y = np.meshgrid(c, c)
    a = np.arctan2(x * y, np.sqrt(x * x + y * y + 1.0))
    return a[1:, 1:] - a[1:, :-1] - a[:-1, 1:] + a[:-1, :-1]


@pytest.mark.parametrize("size", [1024, 2048, 4096])  # the last level from launch 2, 2 and 3
def test_last_level_of_the_chain(size):
    from paper_2012_03325_amd import frame as fr
    small = 256
    env = np.random.default_rng(size).uniform(0.0, 4.0, (6, small, small, 4)).astype(np.float32)
    p = dict(irr_size=2, irr_src_size=64, pref_size=4, pref_levels=2, pref_samples=1, lut_size=2, lut_samples=1,
             pref_fis=1)
    rep = size // small  # (a texel's parts share its colour and add up to its solid angle)
    ibl = fr.DeviceIBL(env.repeat(rep, 1).repeat(rep, 2), **p)
    ibl.pref.fill_(float("nan"))
    ibl.scratch.fill_(255)
    ibl.precompute()
    torch.cuda.synchronize()
    w = _solid_angles(small)[None, :, :, None]
    quadrants = lambda v: v.reshape(v.shape[0], 2, small // 2, 2, small // 2, -1).sum((2, 4))
    ref = quadrants(env[..., :3].astype(np.float64) * w) / quadrants(w)
    # an N.L-weighted mean of one sample with N.L = 1: the chain's value (the tables' tolerance)
    assert_interval(f"last level of 6x{size}^2", ibl.pref_levels()[1].cpu().numpy()[..., :3], ref, ref)
