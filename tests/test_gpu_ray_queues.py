"""Closest hits over queues at the lengths where their launches change: 16
rays per wave, up to which a queue is dealt out (4 096 and 4 097 rays with one
block per CU of 256), one to eight rays for a wave, and frames just above 65 536
pixels, whose launches never deal and whose later bounces are shorter than
their grids.  View paths and next-event visibility against the FP64 oracle."""
import time

import numpy as np
import pytest

from neb_inputs import box_room, city_lots
from parity import path_agreement, rel_rmse, scene_diag

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


@pytest.mark.parametrize("wh,blocks", [((64, 64), 1), ((241, 17), 1), ((1, 1), 8), ((2, 1), 8), ((3, 1), 8), ((8, 1), 8),
                                       ((9, 1), 8), ((257, 256), 8), ((257, 256), 1)])
def test_paths_and_visibility(neb, oracle, wh, blocks):
    sc = city_lots(width=wh[0], height=wh[1])
    g = neb.Renderer(sc, flags=neb.FLAG_RECORD_PATHS | neb.FLAG_NO_PHOTONS)
    cfg = g.launch_config()
    cfg.update(trace_blocks_per_cu=blocks, nee_blocks_per_cu=blocks)
    g.set_launch_config(**cfg)
    g.render(1)
    rec, img, st = g.records(), g.image_host().astype(np.float64), g.stats()
    g.close()
    o = oracle.render(sc, n_iter=1, record=True, enable_photons=False)
    frac, same = path_agreement(rec, o["records"], scene_diag(sc))
    # FP32 and FP64 part ways on about one path in 5000
    assert frac == 1.0 if len(same) < 100 else frac >= 0.999, frac
    assert abs(st["nee_visible"] - o["stats"]["nee_visible"]) <= max(1, 1e-3 * o["stats"]["nee_visible"])
    if o["mean"].sum() > 0:
        assert rel_rmse(img, o["mean"]) < 0.01


def _medians(neb, frames):
    """Seconds of eight iterations of each frame, the frames in turn."""
    import torch
    rs = []
    for w, h in frames:
        sc = box_room(n_tris=300, n_lights=2, res=w, spp=4, seed=4, scene_id=1).with_settings(width=w, height=h)
        rs.append(neb.Renderer(sc, flags=neb.FLAG_NO_PHOTONS))
        rs[-1].render(8)
    t = [[] for _ in rs]
    for _ in range(25):
        for k, r in enumerate(rs):
            torch.cuda.synchronize()
            s = time.perf_counter()
            r.render(8)
            torch.cuda.synchronize()
            t[k].append(time.perf_counter() - s)
    for r in rs:
        r.close()
    return [sorted(x)[len(x) // 2] for x in t]


def test_blocks_without_rays_cost_nothing(neb):
    # 65 536 pixels: grids of eight rays a wave, queues too long to be dealt;
    # 256 pixels more, and the grids are of 64 rays a wave.  The blocks without
    # a ray took an eighth of the iteration.
    dealt, undealt = _medians(neb, [(256, 256), (256, 257)])
    assert dealt < 1.08 * undealt, (dealt, undealt)
