"""Deposits into large octrees.  A call of few points costs what its points
cost, not what the tree does, so the counts of such calls wait in a second word
per node: they must be seen by densities, exports, the one-thread path and
the splits of later calls, and join the nodes without a change.  A call
whose points all lie outside the box and are many joins them and counts
nothing.  And a tree's memory is all there when it has been created."""
import time

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


def _points(n, seed, lo=0.0, hi=1.0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.rand(n, 3, generator=g, device="cuda") * (hi - lo) + lo


def _grown(neb, capacity, n, iteration):
    t = neb.DeviceOctree(LO, HI, capacity)
    t.increment(_points(n, 5))
    t.set_iteration(iteration)
    return t


def _leaves(nodes):
    return int((nodes[nodes >= 0].astype(np.int64) & 0x3FFFFFFF).sum())


def _seconds(call, rounds=5, calls=100):
    import torch
    best = float("inf")
    for _ in range(rounds):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(calls):
            call()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / calls)
    return best


def test_few_points_cost_the_same_in_a_large_tree(neb):
    small, large = _grown(neb, 1 << 14, 20000, 900), _grown(neb, 1 << 25, 80000000, 900)
    p = _points(100, 1)
    a, b = _seconds(lambda: small.increment(p)), _seconds(lambda: large.increment(p))
    # 128 MB of second words take 50 us or more to read, the call 20
    assert b < 1.5 * a + 10e-6, (a, b)


def test_memory_is_there_from_the_start(neb):
    import torch
    p = _points(100, 1)
    t = neb.DeviceOctree(LO, HI, 1 << 26)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    t.increment(p)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] < 64 << 20  # the queues of deferred points


@pytest.mark.parametrize("iteration,n,single", [(250, 1, False), (250, 700, False), (1, 5000, False), (2, 60000, False),
                                                (250, 1, True), (250, 700, True), (1, 5000, True)])
def test_waiting_counts_are_seen(neb, iteration, n, single):
    import torch
    t = _grown(neb, 8 << 20, 3000000, iteration)  # room for every split
    q = torch.cat([_points(20000, 9), _points(20000, 8, 0.4, 0.41)])
    nrm = torch.nn.functional.normalize(_points(40000, 7, -1.0, 1.0), dim=1)
    before, info = t.export()
    assert info["overflow"] == 0 and info["allocated"] > max(1 << 20, 16 * n)
    assert info["ledger"] == info["deposits"] == 3000000
    d0 = t.density(q, nrm)
    for call in range(3):  # into a corner, whose leaves split and split again where the iteration is low
        t.increment(_points(n, 20 + call, 0.4, 0.41), single_thread=single and call == 1)
    nodes, info = t.export()
    assert info["ledger"] == info["deposits"] == 3000000 + 3 * n and info["lost"] == 0
    blocks = int((nodes < 0).sum()) - int((before < 0).sum())
    assert _leaves(nodes) == _leaves(before) + 3 * n + 4 * iteration * blocks
    assert blocks > 0 or iteration > 2 or n < 100
    robust, plain = t.density(q, nrm), t.density(q, nrm, robust=False)
    assert n < 100 or (d0 != robust).any()
    t.increment(torch.full((1 << 20, 3), 2.0, device="cuda"))  # joins the counts, deposits nothing
    after, info2 = t.export()
    assert np.array_equal(nodes, after)
    assert info2["ledger"] == info["ledger"] and info2["rejected"] == info["rejected"] + (1 << 20)
    assert torch.equal(robust, t.density(q, nrm)) and torch.equal(plain, t.density(q, nrm, robust=False))


def test_clear_with_waiting_counts(neb):
    t = _grown(neb, 3 << 20, 3000000, 250)
    t.increment(_points(1000, 1))
    t.clear_counters()
    nodes, info = t.export()
    assert info["ledger"] == info["deposits"] == 0 and not nodes[nodes >= 0].any()
    t.set_iteration(250)
    t.increment(_points(1000, 2))
    nodes, info = t.export()
    assert info["ledger"] == info["deposits"] == 1000 == _leaves(nodes)


@pytest.mark.parametrize("capacity,n", [(8, 5), (1 << 12, 3000), (1 << 20, 1000003), (3 << 20, 2000000)])
def test_ledger_sums_the_leaves(neb, capacity, n):
    nodes, info = _grown(neb, capacity, n, 900).export()
    blocks = (info["allocated"] - 1) // 8  # all of iteration 1
    assert _leaves(nodes) - 4 * blocks == info["ledger"] == info["deposits"] == n
    assert info["lost"] == 0
