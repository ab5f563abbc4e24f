"""Gathered chunks on lattices whose last stretch of fluid nodes is cut short
by its halo: the stepped fields equal variant 4's bitwise, and so does the next
quantity's first node, where a chunk past the last fluid node would store. (The
partition itself is checked on the CPU for the same lattices.)"""
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


@pytest.mark.parametrize("nh", [1, 2])
@pytest.mark.parametrize("mask", [lambda: inputs.random_mask(79, 52, 13, 0.05, seed=2),
                                  lambda: inputs.random_mask(83, 85, 9, 0.1, seed=0),
                                  lambda: inputs.bulk_mask(97, 12, 13),
                                  lambda: inputs.sphere_pack(65, 6, 0.5, seed=1)],
                         ids=["79x52x13", "83x85x9", "97x12x13", "65^3"])
def test_fields_equal_the_haloed_block(lb, monkeypatch, mask, nh):
    m = mask()
    fl = lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.01, seed=9))
    sp = {"D_b": 0.05, "k_a": [0.02, 0.3], "k_d": [0.01, 0.5]}
    monkeypatch.setenv("LBMP_GATHER_NH", str(nh))
    got = {}
    for tile in ("8,2,2", "4,2,2"):
        monkeypatch.setenv("LBMP_TILE", tile)
        mp = lb.mp_init(fl, sp, 32, 12)
        assert lb.mp_stats(mp, 0)["kernel_variant"] == int(tile[0])
        lb.mp_step_n(mp, 12)
        got[tile] = [lb.mp_state(mp, 0, s) for s in range(2)]
        mp.free()
    for (X, Xa), (Xr, Xar) in zip(got["8,2,2"], got["4,2,2"]):
        assert np.array_equal(X, Xr) and np.array_equal(Xa, Xar)
    fl.free()
