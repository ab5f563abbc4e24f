"""Step kernels of launch-bound runs on lattices that are mostly solid: the flat
kernel's work grows with the lattice, variant 0's with its fluid nodes, so the
choice must not cost a capillary in a large block of solid the time of the
whole block. (Timed: the least of several runs against variant 0's, which used
to be 0.5 to 0.7 of the chosen kernel's.) And the choice on either side of its
lines."""
import time

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


def capillary(n, nz, r):
    m = np.ones((nz, n, n), dtype=np.uint8)
    y, x = np.indices((n, n))
    m[:, (x - (n - 1) / 2) ** 2 + (y - (n - 1) / 2) ** 2 <= r * r] = 0
    return m


def at_rest(lb, m):
    return lb.lb_flow_from_velocity(m, np.zeros((3,) + m.shape))


def species(S):
    return {"D_b": 0.05, "k_a": [0.01] * S, "k_d": [0.02] * S}


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("shape,S", [((128, 64, 8), 3), ((64, 128, 8), 2)])
def test_time_of_a_capillary(lb, monkeypatch, shape, S, prec):
    import torch
    monkeypatch.setenv("LBMP_TUNE_CACHE", "")
    fl = at_rest(lb, capillary(*shape))
    best, out = {}, {}
    for tile in (None, f"0,1,{S}"):
        monkeypatch.delenv("LBMP_TILE", raising=False)
        if tile:
            monkeypatch.setenv("LBMP_TILE", tile)
        mp = lb.mp_init(fl, species(S), prec, 2000)
        t = []
        for _ in range(6):
            t0 = time.perf_counter()
            lb.mp_step_n(mp, 256)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        best[tile], out[tile] = min(t), lb.mp_state(mp, 0, S - 1)
        mp.free()
    fl.free()
    assert best[None] < 1.25 * best[f"0,1,{S}"], best
    for a, b in zip(out[None], out[f"0,1,{S}"]):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("prec,nz,plan", [(32, 32, (9, 1)), (32, 33, (9, 4)), (32, 64, (9, 4)), (32, 65, (0, 1)),
                                          (64, 16, (9, 1)), (64, 17, (9, 4)), (64, 32, (9, 4)), (64, 33, (0, 1))])
def test_choice(lb, monkeypatch, prec, nz, plan):
    monkeypatch.setenv("LBMP_TUNE_CACHE", "")
    monkeypatch.delenv("LBMP_TILE", raising=False)
    fl = at_rest(lb, capillary(64, nz, 8))  # 4,096 nodes and 208 fluid ones a plane
    for init, want in ((lb.mp_init, plan), (lb.mp_uptake_init, (9, 1))):
        mp = init(fl, species(2), prec, 4)
        st = lb.mp_stats(mp, 0)
        assert (st["kernel_variant"], st["tile_k"]) == want
        mp.free()
    fl.free()
