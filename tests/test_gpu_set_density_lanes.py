"""Point-set densities where the number of lanes that share a query changes
(up to 4 096, 16 384 and 65 536 queries) and where the number of distances
kept does (k = 4, 8), against FP64 brute force; and the same densities inside
a render, whose queries run in bucket order, against neb_point_density's."""
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


def _reference(p, q, R, k):
    """FP64 count within R and k-th smallest squared distance of each query."""
    import torch
    m, dk = [], []
    for a in q.double().split(4096):
        d2 = torch.cdist(a, p.double(), compute_mode="donot_use_mm_for_euclid_dist") ** 2
        m.append((d2 < R * R).sum(1))
        dk.append(torch.topk(d2, k, dim=1, largest=False).values[:, -1])
    return torch.cat(m).double(), torch.cat(dk)


@pytest.mark.parametrize("n_query,k", [(1, 1), (63, 4), (4096, 5), (4097, 8), (16384, 9), (16385, 16), (65536, 2),
                                       (65537, 7)])
def test_lane_counts(neb, n_query, k):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n_query)
    n = 3001
    p = torch.rand(n, 3, generator=g, device="cuda") * torch.tensor([1.0, 0.02, 1.0], device="cuda")
    p[: n // 3] = p[: n // 3] * 0.05 + 0.4  # a dense corner: buckets of hundreds
    q = p[torch.randint(0, n, (n_query,), generator=g, device="cuda")].clone()
    q[1::2] += 0.01
    R = float(np.float32(0.04))
    m, dk = _reference(p, q, R, k)
    area = math.pi * R * R
    out = torch.empty(n_query, device="cuda")
    for call in (neb.point_density, lambda *a: neb.point_density_noalloc(*a, out)):
        c = call(p, q, neb.DENSITY_RADIUS, R, 8).double() * area
        near = (c - m).abs()
        # a distance within FP32 rounding of R counts on either side
        assert (near > 0.5).double().mean() <= 1e-3 and near.max() <= 1.5
        r = call(p, q, neb.DENSITY_KNN, R, k).double()
        want = torch.where(m >= k, k / (math.pi * dk), m / area)
        # squared distances carry a few FP32 roundings
        bad = (r - want).abs() > 1e-5 * want + 1e-12
        assert bad.double().mean() <= 1e-3
