"""Closest-hit launch shapes at the limits of a configuration: what a stack
alone would leave room for is accepted as before, and reported as the blocks
that are resident beside what the lanes of a block exchange."""
import numpy as np
import pytest

from neb_inputs import city_lots

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


@pytest.mark.parametrize("stack,accepted,resident", [(32, 20, 17), (48, 13, 12), (64, 10, 9)])
def test_blocks_per_cu(neb, stack, accepted, resident):
    sc = city_lots(width=61, height=67)
    images = []
    for blocks in (accepted, -1, 1):
        g = neb.Renderer(sc, flags=neb.FLAG_NO_PHOTONS)
        cfg = g.launch_config()
        cfg.update(bvh_stack=stack, trace_blocks_per_cu=blocks, nee_blocks_per_cu=blocks)
        g.set_launch_config(**cfg)
        got = g.launch_config()
        assert got["trace_blocks_per_cu"] == got["nee_blocks_per_cu"] == (1 if blocks == 1 else resident)
        if blocks == accepted:
            for name in ("trace_blocks_per_cu", "nee_blocks_per_cu"):
                with pytest.raises(Exception):
                    g.set_launch_config(**dict(cfg, **{name: accepted + 1}))
        g.render(1)
        images.append(g.image_host())
        g.close()
    for img in images[1:]:
        assert np.allclose(img, images[0], rtol=1e-5, atol=1e-6)
