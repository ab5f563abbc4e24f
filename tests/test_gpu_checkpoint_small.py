"""Checkpoint and resume with the step kernels of small lattices: a run stopped,
saved, loaded into a new handle (of the same kernel, or of another one) and
continued, against the uninterrupted run; the resident kernel also across the
limit of steps in one launch."""
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


SPECIES = {"D_b": 0.05, "k_a": [0.0, 0.01, 0.05], "k_d": [0.1, 0.02, 0.004]}


def flow(lb):
    m = inputs.random_mask(13, 11, 9, 0.3, seed=51)
    return lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.02, seed=52))


def states(lb, h):
    return [lb.mp_state(h, 0, s) for s in range(3)]


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("mode,tile,other", [("vacf", "9,1,1", "9,4,1"), ("vacf", "9,2,1", "0,1,3"),
                                             ("vacf", "10,1,1", "9,1,1"), ("uptake", "9,1,1", "0,1,3"),
                                             ("uptake", "10,1,1", "9,1,1")])
def test_resume(lb, monkeypatch, mode, tile, other, prec):
    fl = flow(lb)
    T, n = 140, 53
    init = lb.mp_init if mode == "vacf" else lb.mp_uptake_init

    def start(t):
        monkeypatch.setenv("LBMP_TILE", t)
        h = init(fl, SPECIES, prec, T)
        assert lb.mp_stats(h, 0)["kernel_variant"] == int(t.split(",")[0])
        return h

    def series(h):
        if mode == "vacf":
            r = lb.mp_vacf(h, 0)
            return {k: r[k] for k in ("Z", "D", "mass")}
        r = lb.mp_uptake(h, 0)
        return {k: r[k] for k in ("mobile", "adsorbed")}

    a = start(tile)
    lb.mp_step_n(a, T)
    ref, sref = series(a), states(lb, a)
    a.free()
    b = start(tile)
    lb.mp_step_n(b, n)
    buf = lb.mp_save(b)
    b.free()
    for t in (tile, other):
        c = start(t)
        lb.mp_load(c, buf)
        assert lb.mp_steps_done(c) == n
        lb.mp_step_n(c, T - n)
        got = series(c)
        # every kernel's fields are bitwise the same; its sums group nodes in
        # its own way, so between kernels the series agree to rounding
        for (X, Xa), (Xr, Xar) in zip(states(lb, c), sref):
            assert np.array_equal(X, Xr) and np.array_equal(Xa, Xar)
        for k in ref:
            if t == tile:
                assert np.array_equal(got[k], ref[k]), k
            else:
                np.testing.assert_allclose(got[k], ref[k], rtol=1e-11, atol=1e-15)
        c.free()
    fl.free()


def test_resident_kernel_across_launches(lb, monkeypatch):
    fl = flow(lb)
    monkeypatch.setenv("LBMP_TILE", "10,1,1")
    T = 4096 + 37  # one more launch than fits
    a = lb.mp_init(fl, SPECIES, 64, T)
    lb.mp_step_n(a, T)
    b = lb.mp_init(fl, SPECIES, 64, T)
    lb.mp_step_n(b, 4095)
    c = lb.mp_init(fl, SPECIES, 64, T)
    lb.mp_load(c, lb.mp_save(b))
    lb.mp_step_n(c, T - 4095)
    assert np.array_equal(lb.mp_vacf(a, 0)["D"], lb.mp_vacf(c, 0)["D"])
    for (X, Xa), (Xr, Xar) in zip(states(lb, c), states(lb, a)):
        assert np.array_equal(X, Xr) and np.array_equal(Xa, Xar)
    for h in (a, b, c):
        h.free()
    fl.free()
