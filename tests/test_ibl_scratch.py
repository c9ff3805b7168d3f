"""Scratch sizes of the image-based-lighting precompute."""
import pytest

from paper_2012_03325_amd import epb as E

SIZES = [8, 16, 32, 64, 128, 256, 512, 1024, 2048, 4096]


def _bytes(size, fis, irr=32, src=64, pref=128, levels=5, samples=1024, lut=64, lut_samples=64):
    p = E.epb_ibl_params(irr, src, pref, levels, samples, lut, lut_samples, fis)
    return E.epb_scratch_bytes(E.EPB_OP_PRECOMPUTE_IBL, size, size, p)


@pytest.mark.parametrize("pref,levels", [(8, 1), (8, 3), (16, 2), (32, 4), (64, 3), (128, 5), (512, 7)])
def test_filtered_asks_for_no_less_than_plain(pref, levels):
    """A buffer sized for filtered sampling serves plain sampling of the same sizes too."""
    for size in SIZES:
        for irr, samples in ((2, 1), (32, 64), (64, 4096)):
            if (min(size, pref) >> (levels - 1)) < 2:
                continue  # levels of less than 2x2
            plain, filtered = (_bytes(size, fis, irr, 64, pref, levels, samples) for fis in (0, 1))
            assert plain > 0 and filtered >= plain


@pytest.mark.parametrize("fis", [0, 1])
@pytest.mark.parametrize("pref,levels,samples", [(8, 1, 64), (8, 3, 16), (32, 3, 33), (128, 2, 64), (128, 4, 1024)])
def test_a_larger_environment_asks_for_no_less(pref, levels, samples, fis):
    """A buffer sized for the largest environment serves smaller ones too, for more samples fewer."""
    sizes = [s for s in SIZES if (min(s, pref) >> (levels - 1)) >= 2]
    asked = [_bytes(s, fis, 32, 8, pref, levels, samples) for s in sizes]
    assert min(asked) > 0 and asked == sorted(asked)
    for s in sizes:
        asked = [_bytes(s, fis, 32, 8, pref, levels, n) for n in (1, 16, 32, 33, 64, 500, 4096)]
        assert asked == sorted(asked)
