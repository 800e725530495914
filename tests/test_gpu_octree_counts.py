"""Concurrent octree deposits against the one-thread path where no leaf
fills: the trees must be equal word for word, whatever wave a deposit falls
into (scattered points, every lane of a wave at one leaf, one leaf hit by
all waves, points outside the box), for counts around a wave and a block,
over several calls, on a tree of one block and a grown one.  Then on leaves
that do fill: the ledger and every block's parent."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LO, HI = np.zeros(3, np.float32), np.ones(3, np.float32)


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _points(kind, n, seed):
    rng = np.random.default_rng(seed)
    p = rng.random((n, 3)).astype(np.float32)
    if kind == "runs":  # 64 consecutive points in one place, others next to it
        p = np.repeat(p[:(n + 63) // 64], 64, axis=0)[:n]
    elif kind == "one":
        p[:] = (0.31, 0.71, 0.12)
    elif kind == "outside":
        p[::3] += 2.0
    return p


@pytest.mark.parametrize("grown", [0, 9, 4000])
@pytest.mark.parametrize("kind", ["scattered", "runs", "one", "outside"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 900])
def test_counts_equal_one_thread(neb, kind, n, grown):
    a, b = neb.DeviceOctree(LO, HI, 1 << 14), neb.DeviceOctree(LO, HI, 1 << 14)
    for t in (a, b):
        if grown:
            t.increment(_dev(_points("scattered", grown, 1)), single_thread=True)
        t.set_iteration(250)  # a leaf holds 1 000
        for call in range(2):
            t.increment(_dev(_points(kind, n // (1 + call) or 1, 2 + call)[:450]), single_thread=t is b)
    (na, ia), (nb, ib) = a.export(), b.export()
    assert ia == ib and ia["lost"] == 0
    assert np.array_equal(na, nb)


@pytest.mark.parametrize("capacity,n", [(8, 100), (64, 5000), (1 << 16, 40000)])
def test_ledger_over_calls(neb, capacity, n):
    t = neb.DeviceOctree(LO, HI, capacity)
    total = 0
    for it in range(1, 7):
        t.set_iteration(it)
        p = _points("runs" if it % 2 else "scattered", n, it)
        t.increment(_dev(p), single_thread=it == 3 and n < 10000)
        total += n
        nodes, info = t.export()
        assert info["lost"] == 0 and info["ledger"] == info["deposits"] == total
        ptr = -nodes[nodes < 0]
        assert np.all((ptr - 1) % 8 == 0) and len(np.unique(ptr)) == len(ptr)
        assert np.all(nodes[nodes >= 0] >= 0) and 8 * len(ptr) + 1 == info["allocated"]
