"""Tables of the gathered chunks (built on the device) where they can go
wrong: chunks cut short by their halo, last chunks of a few nodes, lattices of
one column (a node is its own neighbour), tiles beyond the lattice. A wrong
arrival slot, halo quad or interface index changes the stepped fields, which
must equal variant 4's bitwise."""
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


def _checkerboard(n):
    z, y, x = np.indices((n, n, n))
    return ((x + y + z) % 2).astype(np.uint8)


MASKS = {
    "column": lambda: inputs.slit_mask(1, 1, 34),
    "one node": lambda: inputs.random_mask(3, 3, 3, 1.0, seed=1),
    "plane": lambda: inputs.random_mask(130, 1, 2, 0.2, seed=2),
    "bulk 33x5x9": lambda: inputs.bulk_mask(33, 5, 9),
    "random 40^3 0.3": lambda: inputs.random_mask(40, 40, 40, 0.3, seed=3),
    "random 40^3 0.6": lambda: inputs.random_mask(40, 40, 40, 0.6, seed=4),
    "random 48^3 0.95": lambda: inputs.random_mask(48, 48, 48, 0.95, seed=5),
    "checkerboard 24^3": lambda: _checkerboard(24),
    "spheres 50^3": lambda: inputs.sphere_pack(50, 6, 0.4, seed=6),
}


@pytest.mark.parametrize("nh", [1, 2])
@pytest.mark.parametrize("name", MASKS)
def test_fields_equal_the_haloed_block(lb, monkeypatch, name, nh):
    m = MASKS[name]()
    fl = [lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.01, seed=9))]
    m2 = inputs.random_mask(19, 8, 6, 0.4, seed=8)  # a second geometry after it in the same handle
    fl.append(lb.lb_flow_from_velocity(m2, inputs.random_velocity(m2, 0.01, seed=10)))
    sp = [{"D_b": 0.05, "k_a": [0.02, 0.3], "k_d": [0.01, 0.5]}] * 2
    monkeypatch.setenv("LBMP_GATHER_NH", str(nh))
    got = {}
    for tile in ("8,2,2", "4,2,2"):
        monkeypatch.setenv("LBMP_TILE", tile)
        mp = lb.mp_init(fl, sp, 32, 12)
        assert lb.mp_stats(mp, 0)["kernel_variant"] == int(tile[0])
        lb.mp_step_n(mp, 12)
        got[tile] = [lb.mp_state(mp, g, s) for g in range(2) for s in range(2)], lb.mp_vacf(mp, 0)
        mp.free()
    for (X, Xa), (Xr, Xar) in zip(got["8,2,2"][0], got["4,2,2"][0]):
        assert np.array_equal(X, Xr) and np.array_equal(Xa, Xar)
    for k, v in got["4,2,2"][1].items():
        np.testing.assert_allclose(got["8,2,2"][1][k], v, rtol=1e-12, atol=1e-18)


@pytest.mark.parametrize("tile", ["8,2,2", "4,2,2", "3,1,1", "0,1,2", "9,4,1"])
@pytest.mark.parametrize("name", ["plane", "bulk 33x5x9", "random 48^3 0.95"])
def test_workspace_content_does_not_matter(lb, monkeypatch, tile, name):
    """The workspace the allocator hands out holds NaNs: the same series as
    from a workspace of zeros."""
    import torch
    m = MASKS[name]()
    fl = lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.01, seed=9))
    sp = {"D_b": 0.05, "k_a": [0.02, 0.3], "k_d": [0.01, 0.5]}
    monkeypatch.setenv("LBMP_TILE", tile)
    empty, got = torch.empty, []
    for v in (0, 255):  # bytes of 255 are NaNs in FP32 and FP64
        monkeypatch.setattr(torch, "empty", lambda *a, **k: empty(*a, **k).fill_(v))
        mp = lb.mp_init(fl, sp, 32, 9)
        monkeypatch.setattr(torch, "empty", empty)
        lb.mp_step_n(mp, 9)
        got.append((lb.mp_vacf(mp, 0), lb.mp_state(mp, 0, 1)))
        mp.free()
    for k in got[0][0]:
        assert np.array_equal(got[0][0][k], got[1][0][k]), k
    assert all(np.array_equal(a, b) for a, b in zip(got[0][1], got[1][1]))
