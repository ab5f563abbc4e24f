"""The recorded sums do not depend on how the steps of a run are split into
calls: a step's sums are added in one order, whether the next launch of the
same call, the end of the call or of a replayed chunk of steps records them.
Lattices of some hundred tiles and of more than 2,048 (summed in two stages),
where a pair's tiles outnumber the threads that add them."""
import numpy as np
import pytest

from paper_1303_2470_amd import inputs

pytestmark = pytest.mark.gpu

T = 150  # 64-step chunks are replayed from 128 steps in one call on


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_2470_amd import lbmp
    lbmp.load_library()
    return lbmp


def _same(a, b):
    for k in ("Z", "D", "mass"):
        assert np.array_equal(a[k], b[k]), k


@pytest.mark.parametrize("shape", [(64, 44, 38), (64, 136, 80)], ids=["hundreds", "thousands"])
@pytest.mark.parametrize("tile,prec", [("4,2,2", 32), ("6,2,2", 32), ("6,4,2", 32), ("8,2,2", 32), ("9,1,1", 32),
                                       ("9,2,1", 64)])
def test_sums_do_not_depend_on_the_calls(lb, monkeypatch, tile, prec, shape):
    m = inputs.random_mask(*shape, 0.2, seed=41)
    fl = lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.02, seed=42))
    sp = {"D_b": 0.05, "k_a": [0.01, 0.05], "k_d": [0.02, 0.004]}
    monkeypatch.setenv("LBMP_TILE", tile)

    def start():
        mp = lb.mp_init(fl, sp, prec, T)
        assert lb.mp_stats(mp, 0)["kernel_variant"] == int(tile[0])
        return mp

    a = start()
    lb.mp_step_n(a, T)
    ref = lb.mp_vacf(a, 0)
    a.free()
    b = start()
    for n in (1, 2, 64, 30, 53):
        lb.mp_step_n(b, n)
    _same(lb.mp_vacf(b, 0), ref)
    b.free()
    c = start()
    lb.mp_step_n(c, 61)
    buf = lb.mp_save(c)
    c.free()
    d = start()
    lb.mp_load(d, buf)
    lb.mp_step_n(d, T - 61)
    _same(lb.mp_vacf(d, 0), ref)
    d.free()
    fl.free()
