"""Photon merges over candidate lists of every length: merge radii from a
few candidates per photon up to half the box, where a wave's list runs over
many of the windows it is walked in, with path lengths on both sides of the
depth classes' border and an image that leaves part of a wave idle.  The
merge images against the FP64 oracle (analytic density, the same rho on
both sides; one percent relative RMSE, the bound of the other element by
element comparisons)."""
import numpy as np
import pytest

from neb_inputs import tiny_box
from parity import rel_rmse, technique_errors

pytestmark = pytest.mark.gpu

RHO0 = 3000.0


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


@pytest.mark.parametrize("radius,wh,L", [(0.004, (33, 17), 5), (0.03, (24, 24), 6), (0.2, (24, 24), 5),
                                         (0.2, (24, 23), 8), (0.5, (20, 20), 9)])
def test_list_lengths(neb, oracle, radius, wh, L):
    sc = tiny_box(width=wh[0], height=wh[1], max_path_len=L).with_settings(merge_radius=radius)
    g = neb.Renderer(sc, density_mode=neb.DENSITY_ANALYTIC, rho0=RHO0, cam_weight=1.0, light_photons=512)
    g.render(2)
    img, tech, st = g.image_host().astype(np.float64), g.technique_images_host(), g.stats()
    g.close()
    o = oracle.render(sc, n_iter=2, density_mode=oracle.DENSITY_ANALYTIC, rho0=RHO0, cam_weight=1.0,
                      light_photons=512)
    assert st["merges"] == pytest.approx(o["stats"]["merges"], rel=5e-3, abs=2)
    if radius >= 0.2:
        assert st["candidates"] > 4096 * (st["photon_items"] / 64)  # lists beyond a window
    assert rel_rmse(img, o["mean"]) < 0.01
    for t, v in technique_errors(tech, o["tech"], 2).items():
        assert v < 0.01, (t, v)
