"""Bucket tables of every number of scan tiles (one, two, a few, many; 4096
keys each): fixed-radius counts over points on a lattice whose spacing is
beyond the radius, so that a count is the number of points at one place, a
whole number that has to be met."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


@pytest.mark.parametrize("n", [1, 1024, 4096, 8191, 8192, 65537, 524288, 1100000])
def test_counts_are_exact(neb, n):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    cell = torch.randint(0, 64, (n, 3), generator=g, device="cuda")
    p = cell.float() / 64
    R = float(np.float32(0.4 / 64))
    key = (cell[:, 0] * 64 + cell[:, 1]) * 64 + cell[:, 2]
    want = torch.bincount(key, minlength=64 ** 3)[key]
    out = torch.empty(n, device="cuda")
    calls = [lambda: neb.point_density(p, p, neb.DENSITY_RADIUS, R, 8)]
    if n <= 524288:
        calls += [lambda: neb.point_density_noalloc(p, p, neb.DENSITY_RADIUS, R, 8, out)] * 2
    for call in calls:
        got = call().double() * (math.pi * R * R)
        assert torch.equal(got.round().long(), want)
