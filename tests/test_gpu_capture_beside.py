"""Propagation and training steps issued while a graph is being captured on a
stream that is not theirs, on this thread or another: they run eagerly, and the
capture goes on. (The steps ask whether the current stream is idle; a query in
the default capture mode would fail and invalidate the capture.) Also steps
that are themselves captured, and the current stream idle, busy or the
handle's own."""
import threading

import numpy as np
import pytest

from paper_1303_2470_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_2470_amd import lbmp
    lbmp.load_library()
    return lbmp


class Runs:
    """A propagation and a training run, and the same ones stepped eagerly."""

    def __init__(self, lb):
        import torch
        rng = np.random.default_rng(1)
        self.lb = lb
        self.x = torch.tensor(rng.normal(size=(1024, 6)), dtype=torch.float32, device="cuda")
        self.y = torch.tensor(rng.normal(size=1024), dtype=torch.float32, device="cuda")
        m = inputs.random_mask(12, 10, 9, 0.2, seed=3)
        self.flow = lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.02, seed=4))
        self.mp, self.mp_ref = self.start(), self.start()
        self.sg, self.sg_ref = lb.Surrogate(1024, seed=5), lb.Surrogate(1024, seed=5)
        torch.cuda.synchronize()

    def start(self):
        return self.lb.mp_init(self.flow, {"D_b": 0.05, "k_a": [0.02], "k_d": [0.01]}, 64, 40)

    def step(self, n=2):
        self.lb.mp_step_n(self.mp, n)
        self.train()

    def train(self):
        self.sg.train_step(self.x, self.y, None, 1024, 1e-3)

    def check(self, steps, trains):
        import torch
        torch.cuda.synchronize()
        self.lb.mp_step_n(self.mp_ref, steps)
        for _ in range(trains):
            self.sg_ref.train_step(self.x, self.y, None, 1024, 1e-3)
        a, b = self.lb.mp_vacf(self.mp, 0), self.lb.mp_vacf(self.mp_ref, 0)
        assert self.lb.mp_steps_done(self.mp) == self.lb.mp_steps_done(self.mp_ref)
        assert np.array_equal(a["Z"], b["Z"])
        assert np.array_equal(self.sg.get_params(), self.sg_ref.get_params())


@pytest.fixture()
def runs(lb):
    r = Runs(lb)
    yield r
    for h in (r.mp, r.mp_ref, r.sg, r.sg_ref, r.flow):
        h.free()


@pytest.mark.parametrize("where", ["side stream", "thread", "thread, side stream"])
def test_steps_beside_a_capture(runs, where):
    import torch
    side, z, failed = torch.cuda.Stream(), torch.zeros(8, device="cuda"), []

    def body():
        try:
            if "side" in where:
                with torch.cuda.stream(side):
                    runs.step()
            else:
                runs.step()
        except Exception as e:  # raised again below, outside the capture
            failed.append(e)

    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        z.add_(1)
        if "thread" in where:
            t = threading.Thread(target=body)
            t.start()
            t.join()
        else:
            body()
        z.add_(1)
    assert not failed, failed
    for k in range(3):
        g.replay()
        runs.step()
        torch.cuda.synchronize()
        assert bool((z == 2 * (k + 1)).all())
    runs.check(2 * 4, 4)


@pytest.mark.parametrize("own", [True, False])
def test_captured_steps(runs, own):
    """Steps captured on the handle's own stream, and forked from another one
    and joined: a replay does what the eager steps do."""
    import torch
    for h, call in ((runs.mp, lambda: runs.lb.mp_step_n(runs.mp, 3)), (runs.sg, runs.train)):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=h.stream if own else torch.cuda.Stream()):
            call()
            if not own:
                torch.cuda.current_stream().wait_stream(h.stream)
        g.replay()
        torch.cuda.synchronize()
    runs.check(3, 1)


@pytest.mark.parametrize("where", ["null", "side", "own"])
@pytest.mark.parametrize("busy", [False, True])
def test_rows_written_on_the_current_stream(runs, where, busy):
    """A training step waits for rows that the current stream still writes."""
    import torch
    stream = {"null": torch.cuda.default_stream(), "side": torch.cuda.Stream(), "own": runs.sg.stream}[where]
    m = torch.rand((2048, 2048), device="cuda")
    xs = torch.zeros_like(runs.x)
    torch.cuda.synchronize()
    rows, runs.x = runs.x, xs
    with torch.cuda.stream(stream):
        if busy:
            for _ in range(30):
                m = (m @ m) / 2048.0
            xs.copy_(rows + 0.0 * m[:1, :6])
        else:
            xs.copy_(rows)
            stream.synchronize()
        for _ in range(3):
            runs.step(1)
    torch.cuda.synchronize()
    runs.x = rows
    runs.check(3, 3)
