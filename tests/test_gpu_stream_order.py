"""Order between the caller's current stream and a handle's: with the current
stream idle (nothing to wait for, no event), busy, the handle's own, and being
captured (fork and join become part of the graph)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_2470_amd import lbmp
    lbmp.load_library()
    return lbmp


@pytest.mark.parametrize("where", ["null", "side", "own"])
def test_busy_idle_and_own_stream(lb, where):
    import torch
    sg = lb.Surrogate(1024, seed=3)
    x0 = torch.rand((4096, 6), device="cuda")
    ref = sg.predict(x0).clone()
    torch.cuda.synchronize()
    stream = {"null": torch.cuda.default_stream(), "side": torch.cuda.Stream(), "own": sg.stream}[where]
    with torch.cuda.stream(stream):
        for busy in (False, True, True, False):
            y = torch.rand((2048, 2048), device="cuda")
            torch.cuda.synchronize()
            x = torch.zeros_like(x0)
            torch.cuda.synchronize()
            if busy:   # x holds its values only after these products
                for _ in range(30):
                    y = (y @ y) / 2048.0
            x.copy_(x0 + 0.0 * y[:1, :6])
            if not busy:
                stream.synchronize()
            got = (sg.predict(x) * 1.0).cpu()   # read on the current stream, without a synchronisation
            assert torch.equal(got, ref.cpu())
    sg.free()


def test_predict_in_a_captured_graph(lb):
    import torch
    sg = lb.Surrogate(1024, seed=3)
    x, out = torch.rand((300, 6), device="cuda"), torch.empty(300, device="cuda")
    sg.predict(x, out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        z = x * 2.0
        sg.predict(z, out)
        w = out + 1.0
    for seed in range(4):
        x.copy_(torch.rand((300, 6), device="cuda", generator=torch.Generator("cuda").manual_seed(seed)))
        g.replay()
        torch.cuda.synchronize()
        ref = sg.predict(x * 2.0)
        assert torch.equal(w, ref + 1.0)
    sg.free()


def test_training_on_rows_still_being_written(lb):
    import torch
    rng = np.random.default_rng(1)
    x = torch.tensor(rng.normal(size=(1024, 6)), dtype=torch.float32, device="cuda")
    y = torch.tensor(rng.normal(size=1024), dtype=torch.float32, device="cuda")
    a, b = lb.Surrogate(1024, seed=5), lb.Surrogate(1024, seed=5)
    for _ in range(5):
        a.train_step(x, y, None, 1024, 1e-3)
        a.sync()
    xs = torch.zeros_like(x)
    m = torch.rand((2048, 2048), device="cuda")
    torch.cuda.synchronize()
    for _ in range(30):
        m = (m @ m) / 2048.0
    xs.copy_(x + 0.0 * m[:1, :6])
    for _ in range(5):
        b.train_step(xs, y, None, 1024, 1e-3)
    assert np.array_equal(a.get_params(), b.get_params())
