"""Renders from cameras so far away that every slab of the tree is one
distance and its empty child slots are entered like the others
(tests/test_bvh_walk_host.py has the walk by itself): black images, no
vertex, no photon, and a context that renders as before afterwards."""
import numpy as np
import pytest

from neb_inputs import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


@pytest.mark.parametrize("wh", [(33, 17), (300, 256)])
@pytest.mark.parametrize("eye", [(1e37, 2e37, 3e37), (-3e38, 3e38, -3e38), (0.5, 0.5, 3e38)])
def test_far_camera_sees_nothing(neb, eye, wh):
    near = scenes.tiny_box(width=wh[0], height=wh[1])
    g = neb.Renderer(near.with_settings(camera=scenes._camera(eye, (0.5, 0.5, 0.5), (0, 1, 0), 60.0)),
                     density_mode=neb.DENSITY_ANALYTIC, rho0=3000.0, cam_weight=1.0)
    g.render(2)
    img, st = g.image_host(), g.stats()
    g.close()
    assert st["camera_rays"] == 2 * wh[0] * wh[1]
    assert st["vertices"] == st["photons"] == st["events"] == 0
    assert np.all(img == 0.0)
