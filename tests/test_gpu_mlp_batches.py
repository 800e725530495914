"""Training batches at the edges of the training kernel's 16-sample tiles,
of its blocks (2 048 tiles at once, then several per wave) and of the
weight-gradient slices (512 samples):
gradient per tensor and loss against the FP64 reference with the same bf16
operand rounding, and an Adam step that follows that gradient."""
import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def neb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1909_00573_amd import neb as N
    N.lib()
    return N


@pytest.mark.parametrize("n", [1, 15, 17, 128, 511, 512, 513, 32768, 32769, 32768 + 129])
def test_gradient_at_edges(neb, n):
    import torch
    rng = np.random.default_rng(n)
    th = M.init_params(5).astype(np.float32)
    q = rng.uniform(0, 1, (n, 3)).astype(np.float32)
    nn = rng.normal(size=(n, 3))
    nn = (nn / np.linalg.norm(nn, axis=1, keepdims=True)).astype(np.float32)
    t = (np.sin(3 * q[:, 0]) + nn[:, 2]).astype(np.float32)
    Q, N_, T = (torch.from_numpy(a).cuda() for a in (q, nn, t))
    m = neb.Mlp(init=th, max_batch=n)
    g, loss = m.gradient(Q, N_, T)
    g = g.cpu().numpy().astype(np.float64)
    lref, gref = M.loss_and_grad(th.astype(np.float64), M.encode(q.astype(np.float64), nn.astype(np.float64)),
                                 t.astype(np.float64), bf16=True)
    assert loss == pytest.approx(lref, rel=2e-3)
    # bf16 deltas and activations, FP32 sums: the bounds of the 1000-sample
    # gradient test; a single sample's flipped rounding is 2^-8 of its share
    tol = 1e-2 if n >= 100 else 3e-2
    G, R = M.unflatten(g), M.unflatten(gref)
    for name, _ in M.SHAPES:
        a, b = np.asarray(G[name]).ravel(), np.asarray(R[name]).ravel()
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b) + 1e-12, name
    m.train_step(Q, N_, T, lr=1e-3)
    step = m.params().astype(np.float64) - th
    sure = np.abs(gref) > 1e-2 * np.abs(gref).max()
    # the first step is lr g / (|g| + eps)
    assert np.allclose(step[sure], -1e-3 * np.sign(gref[sure]), rtol=0, atol=2e-5)
    m.close()
