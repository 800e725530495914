"""Merges in a frame of more than 2^23 vertex slots with many vertices per
merge disc, which sorts its merge grid by eight depths instead of two classes:
photon paths against smaller frames of the same view, which have the two.  The
images estimate the same radiance, and the merges grow with the pixels squared
(twice as wide, so four times the photons, each with four times the vertices)."""
import numpy as np
import pytest

from neb_inputs import tiny_box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


def _render(neb, px, length):
    g = neb.Renderer(tiny_box(width=px, height=px, max_path_len=length),
                     density_mode=neb.DENSITY_RADIUS, density_radius=0.01)
    g.render(1)
    img, st = g.image_host().astype(np.float64), g.stats()
    g.close()
    return img, st


@pytest.mark.parametrize("length", [9, 12])
def test_large_frame_agrees_with_small(neb, length):
    small, large = 512, 1040  # 2.1 and 8.7 M vertex slots at length 9
    a, sa = _render(neb, small, length)
    b, sb = _render(neb, large, length)
    q = large / small
    assert large * large * (length - 1) > 1 << 23 > small * small * (length - 1)
    # paths of independent pixels: relative deviations of the counts are below 1 %
    assert abs(sb["vertices"] / sa["vertices"] / q ** 2 - 1) < 0.01
    assert abs(sb["photons"] / sa["photons"] / q ** 2 - 1) < 0.01
    assert abs(sb["merges"] / sa["merges"] / q ** 4 - 1) < 0.02
    ma, mb = a.mean((0, 1)), b.mean((0, 1))
    assert np.all(np.abs(mb - ma) < 0.02 * ma)
