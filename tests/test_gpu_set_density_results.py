"""Point-set densities, each result by itself, where the number of lanes that
share a query changes (up to 4 096, 16 384 and 65 536 queries) and where the
number of distances kept does (k = 4, 8): against FP64 brute force over the same
FP32 points.  And renders whose densities keep 4, 8 and 16 distances against
the oracle, and scenes of different k in one batch, which keep as many as the
largest asks for, against the same scenes alone."""
import math

import numpy as np
import pytest

from neb_inputs import tiny_box

pytestmark = pytest.mark.gpu

# a squared distance: three differences (half an ulp each, doubled by the
# square), three products, two sums; the radius's square one more: 6 x 2^-24
EDGE = 1e-6
# the estimate: that distance's error, a product and a quotient
REL = 2e-6


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


def _reference(p, q, R, k):
    """FP64 counts within R, on both sides of the rounding of R^2, and the k-th
    smallest squared distance of each query."""
    import torch
    lo, hi, dk = [], [], []
    for a in q.double().split(4096):
        d2 = ((a[:, None, :] - p.double()[None]) ** 2).sum(2)
        lo.append((d2 < R * R * (1 - EDGE)).sum(1))
        hi.append((d2 < R * R * (1 + EDGE)).sum(1))
        dk.append(torch.topk(d2, k, dim=1, largest=False).values[:, -1])
    return torch.cat(lo).double(), torch.cat(hi).double(), torch.cat(dk)


@pytest.mark.parametrize("n_query,k", [(1, 1), (63, 4), (64, 3), (4096, 5), (4097, 8), (16384, 9), (16385, 16), (65536, 2),
                                       (65537, 7), (65537, 16)])
def test_every_result(neb, n_query, k):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n_query + k)
    n = 3001
    p = torch.rand(n, 3, generator=g, device="cuda") * torch.tensor([1.0, 0.02, 1.0], device="cuda")
    p[: n // 3] = p[: n // 3] * 0.05 + 0.4  # a dense corner: buckets of hundreds
    q = p[torch.randint(0, n, (n_query,), generator=g, device="cuda")].clone()
    q += (torch.rand(n_query, 3, generator=g, device="cuda") - 0.5) * 0.02
    R = float(np.float32(0.04))
    lo, hi, dk = _reference(p, q, R, k)
    area = math.pi * R * R
    out = torch.empty(n_query, device="cuda")
    for call in (neb.point_density, lambda *a: neb.point_density_noalloc(*a, out)):
        count = call(p, q, neb.DENSITY_RADIUS, R, 8).double() * area
        assert bool(((count > lo - 0.01) & (count < hi + 0.01)).all())
        r = call(p, q, neb.DENSITY_KNN, R, k).double()
        nearest = k / (math.pi * dk)
        by_distance = (hi >= k) & ((r - nearest).abs() <= REL * nearest)
        by_count = (lo < k) & (r * area > lo - 0.01) & (r * area < hi + 0.01)
        wrong = torch.nonzero(~(by_distance | by_count))
        assert wrong.numel() == 0, (wrong[:5].flatten().tolist(), wrong.shape[0])


@pytest.mark.parametrize("k", [3, 8, 16])
def test_render_matches_oracle(neb, oracle, k):
    sc = tiny_box()
    n_iter, R = 4, 0.05
    g = neb.Renderer(sc, density_mode=neb.DENSITY_KNN, density_radius=R, knn_k=k)
    g.render(n_iter)
    img, st = g.image_host().astype(np.float64), g.stats()
    g.close()
    o = oracle.render(sc, n_iter=n_iter, density_mode=5, density_radius=float(np.float32(R)), knn_k=k)
    assert o["tech"]["P"].sum() > 0.05 * o["sum"].sum()
    assert float(np.sqrt(np.mean((img - o["mean"]) ** 2)) / np.mean(o["mean"])) < 0.01
    assert st["photons"] == pytest.approx(o["stats"]["photons"], rel=2e-3)


def test_mixed_k_equals_alone(neb):
    scenes = [tiny_box(width=48, height=40, max_path_len=5, seed=1),
              tiny_box(width=64, height=64, max_path_len=4, seed=9).with_settings(scene_id=5),
              tiny_box(width=33, height=57, max_path_len=5, seed=3).with_settings(scene_id=6)]
    per = [{"density_radius": 0.05, "knn_k": k} for k in (3, 16, 8)]
    B = neb.BatchRenderer(scenes, density_mode=neb.DENSITY_KNN, per_scene=per)
    B.render(3)
    for s, sc in enumerate(scenes):
        A = neb.Renderer(sc, density_mode=neb.DENSITY_KNN, **per[s])
        A.render(3)
        ta, tb = A.technique_images_host(), B.technique_images_host(s)
        for t in ("e", "E", "P"):
            a, b = ta[t].astype(np.float64), tb[t].astype(np.float64)
            assert np.all(np.abs(a - b) <= 1e-4 * np.abs(a) + 1e-6 * max(np.abs(a).max(), 1e-30)), (s, t)
        A.close()
    B.close()
