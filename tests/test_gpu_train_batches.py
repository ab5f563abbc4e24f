"""Fused training pass at the edges of its batch shapes: one block of rows, an
odd number of 32-row blocks, splits that do not divide evenly, batches of
more blocks than CUs. Gradients against the
FP64 network (bf16 operands carry 2^-9 each; norm-wise errors of a few of
those, independent of the batch: 2e-2), rows through an index list against
the same rows in order (bitwise)."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_2470_amd import lbmp
    lbmp.load_library()
    return lbmp


@pytest.mark.parametrize("B", [32, 96, 544, 1056, 16384, 16416])
def test_gradients_and_indexed_rows(lb, B):
    import torch
    params = mlp.init_params(7)
    flat = np.concatenate([p.ravel() for p in params])
    rng = np.random.default_rng(B)
    x = rng.normal(size=(B, 6))
    t = np.sin(x[:, 0]) + 0.3 * x[:, 1] * x[:, 2]
    xd, td = (torch.tensor(v, dtype=torch.float32, device="cuda") for v in (x, t))
    sg = lb.Surrogate(B, seed=0)
    sg.set_params(flat)
    g, loss = sg.gradients(xd, td, B)
    lref, gref = mlp.loss_and_grads(params, x, t)
    assert abs(loss / lref - 1) < 2e-2
    k = 0
    for ref in gref:
        a = g[k:k + ref.size].reshape(ref.shape)
        k += ref.size
        assert np.linalg.norm(a - ref) < 2e-2 * np.linalg.norm(ref)
    # the rows scattered over a longer table and picked by index: the same step
    n = B + 37
    idx = torch.tensor(np.random.default_rng(1).permutation(n)[:B].astype(np.int32), device="cuda")
    X = torch.full((n, 6), float("nan"), device="cuda")
    Y = torch.full((n,), float("nan"), device="cuda")
    X[idx.long()], Y[idx.long()] = xd, td
    other = lb.Surrogate(B, seed=0)
    other.set_params(flat)
    for _ in range(3):
        la = sg.train_step(xd, td, None, B, 1e-3, want_loss=True)
        lo = other.train_step(X, Y, idx, B, 1e-3, want_loss=True)
        assert la == lo
    assert np.array_equal(sg.get_params(), other.get_params())
    sg.free()
    other.free()
