"""Step kernels of launch-bound sizes: one block per tile, species and quantity
group (variant 9) and whole fields resident in LDS over many steps (variant
10). Both do variant 0's arithmetic with its rounding bits, so the stored
fields must equal variant 0's bitwise; the recorded sums add the same terms in
another order (FP64: a few units in the last place of the largest term)."""
import numpy as np
import pytest

import oracle
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


def _medium(nf, seed):
    """A lattice of ragged shape with exactly nf fluid nodes, and a velocity."""
    nx, ny = 13, 7
    nz = max(2, -(-int(1.3 * nf) // (nx * ny)))
    m = np.ones(nx * ny * nz, dtype=np.uint8)
    m[np.random.default_rng(seed).permutation(m.size)[:nf]] = 0
    m = m.reshape(nz, ny, nx)
    return m, inputs.random_velocity(m, 0.02, seed=seed + 1)


KA = np.array([0.0, 0.02, 0.3])
KD = np.array([0.1, 0.01, 0.5])


def _run(lb, monkeypatch, tile, flows, prec, pieces, uptake=False):
    monkeypatch.setenv("LBMP_TILE", tile)
    sp = [{"D_b": 0.05, "k_a": KA, "k_d": KD} for _ in flows]
    mp = (lb.mp_uptake_init if uptake else lb.mp_init)(flows, sp, prec, sum(pieces))
    monkeypatch.delenv("LBMP_TILE")
    assert lb.mp_stats(mp, 0)["kernel_variant"] == int(tile.split(",")[0])
    for n in pieces:
        lb.mp_step_n(mp, n)
    out = []
    for g in range(len(flows)):
        r = lb.mp_uptake(mp, g) if uptake else lb.mp_vacf(mp, g)
        out.append((r, [lb.mp_state(mp, g, s) for s in range(len(KA))]))
    mp.free()
    return out


def _same(a, b):
    for (ra, fa), (rb, fb) in zip(a, b):
        for s in range(len(KA)):
            assert np.array_equal(fa[s][0], fb[s][0]) and np.array_equal(fa[s][1], fb[s][1]), s
        for k in ra:
            assert np.abs(ra[k] - rb[k]).max() <= 1e-12 * np.abs(rb[k]).max(), k


@pytest.mark.parametrize("uptake", [False, True])
@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("nf", [1, 32, 64, 65, 128, 129, 256, 300, 512, 513, 1024, 1025, 1536, 2048])
def test_resident_equals_direct(lb, monkeypatch, nf, prec, uptake):
    if prec == 64 and nf > 1536:
        pytest.skip("beyond the FP64 limit (refused, see below)")
    m, u = _medium(nf, nf)
    fl = lb.lb_flow_from_velocity(m, u)
    pieces = (1, 2, 30)
    ref = _run(lb, monkeypatch, "0,1,3", [fl], prec, pieces, uptake)
    _same(_run(lb, monkeypatch, "10,1,1", [fl], prec, pieces, uptake), ref)


@pytest.mark.parametrize("prec", [32, 64])
def test_resident_batch_and_long_calls(lb, monkeypatch, prec):
    """Geometries of different sizes in one handle; a call longer than one launch's steps."""
    flows = [lb.lb_flow_from_velocity(*_medium(nf, 7)) for nf in (40, 700, 5)]
    ref = _run(lb, monkeypatch, "0,1,3", flows, prec, (4500,))
    _same(_run(lb, monkeypatch, "10,1,1", flows, prec, (4500,)), ref)


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("tile", ["9,1,1", "9,2,1", "9,4,1"])
def test_flat_equals_direct(lb, monkeypatch, tile, prec):
    """Ragged lattices (a last block of few nodes, a block without fluid), two geometries."""
    m1, u1 = _medium(3000, 3)
    m2 = inputs.random_mask(70, 9, 7, 0.3, seed=21)
    m2[2:5] = 1                                      # several solid planes: whole blocks without fluid
    flows = [lb.lb_flow_from_velocity(m1, u1), lb.lb_flow_from_velocity(m2, inputs.random_velocity(m2, 0.02, seed=5))]
    ref = _run(lb, monkeypatch, "0,1,3", flows, prec, (3, 150))
    _same(_run(lb, monkeypatch, tile, flows, prec, (3, 150)), ref)
    if tile == "9,1,1":
        ref = _run(lb, monkeypatch, "0,1,3", flows, prec, (3, 40), uptake=True)
        _same(_run(lb, monkeypatch, tile, flows, prec, (3, 40), uptake=True), ref)


def test_chosen_by_size_and_oracle(lb):
    """Without a pinned tile: resident up to its node limit, flat above it, both against the oracle."""
    for nf, variant in ((1500, 10), (1600, 9)):
        m, u = _medium(nf, 11)
        fl = lb.lb_flow_from_velocity(m, u)
        mp = lb.mp_init(fl, {"D_b": 0.05, "k_a": KA, "k_d": KD}, 64, 100)
        assert lb.mp_stats(mp, 0)["kernel_variant"] == variant
        lb.mp_step_n(mp, 100)
        out = lb.mp_vacf(mp, 0)
        for s in range(3):
            ref = oracle.vacf(m, u, 0.6, KA[s], KD[s], 100)
            D = oracle.d_of_t(ref["Z"], ref["V"])
            assert (np.abs(out["D"][s] - D) / np.maximum(np.abs(D), 5e-5)).max() < 1e-10
        mp.free()


@pytest.mark.parametrize("tile,prec,nf,uptake", [("10,1,1", 32, 2049, False), ("10,1,1", 64, 1537, False),
                                                 ("10,2,1", 64, 100, False), ("9,3,1", 64, 100, False),
                                                 ("9,1,2", 64, 100, False), ("9,2,1", 64, 100, True)])
def test_refused_tiles(lb, monkeypatch, tile, prec, nf, uptake):
    fl = lb.lb_flow_from_velocity(*_medium(nf, 2))
    monkeypatch.setenv("LBMP_TILE", tile)
    with pytest.raises(lb.LbmpError) as e:
        (lb.mp_uptake_init if uptake else lb.mp_init)(fl, {"D_b": 0.05, "k_a": KA, "k_d": KD}, prec, 10)
    assert e.value.status == -1
