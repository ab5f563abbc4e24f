"""D(t) and Z(t) read back in windows (scan over the recorded sums in
double-double): windows across the scan's stretches of 512 times must equal
the whole series bitwise, and the whole series a plain FP64 sum of its own Z."""
import math

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


@pytest.mark.parametrize("steps", [0, 1, 63, 511, 512, 513, 1100])
def test_windows_and_sum(lb, steps):
    m = inputs.random_mask(9, 7, 6, 0.3, seed=3)
    fl = lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.02, seed=4))
    mp = lb.mp_init(fl, {"D_b": 0.05, "k_a": [0.01, 0.2], "k_d": [0.02, 0.1]}, 64, steps + 5)
    lb.mp_step_n(mp, steps)
    full = lb.mp_vacf(mp, 0)
    assert full["Z"].shape == (2, 3, steps + 1)
    for s in range(2):
        for g in range(3):
            V, Z = full["vbar"][s, g], full["Z"][s, g]
            terms = [0.5 * (Z[0] - V * V)] + [z - V * V for z in Z[1:]]
            # Z itself is rounded: each term is off by at most ulp(Z) / 2 + ulp(V^2) / 2
            tol = 2e-16 * sum(abs(z) + V * V for z in Z) + 1e-300
            for t in {0, 1, 511, 512, 513, steps} & set(range(steps + 1)):
                assert abs(full["D"][s, g, t] - math.fsum(terms[:t + 1])) <= tol, (s, g, t)
    for t0, n in ((0, 0), (0, 1), (steps, 1), (steps // 2, steps - steps // 2 + 1), (min(steps, 500), min(30, steps + 1 - min(steps, 500)))):
        w = lb.mp_vacf(mp, 0, t0, n)
        assert np.array_equal(w["Z"], full["Z"][:, :, t0:t0 + n]) and np.array_equal(w["D"], full["D"][:, :, t0:t0 + n])
        assert np.array_equal(w["mass"], full["mass"]) and np.array_equal(w["vbar"], full["vbar"])
    with pytest.raises(lb.LbmpError):
        lb.mp_vacf(mp, 0, steps, 2)
    mp.free()


def test_state_of_charged_geometries(lb):
    """mp_state's reference weights belong to the geometry asked for (two
    charged ones and a neutral one in a handle): at the start the density is
    the Eq. 11 weight exp(-beta mu) / Z up to the source of the first step,
    zero for a bulk lattice at rest."""
    m = inputs.bulk_mask(6, 5, 4)
    fl = [lb.lb_flow_from_velocity(m, np.zeros((3,) + m.shape)) for _ in range(3)]
    b = [np.random.default_rng(i).uniform(-0.3, 0.3, m.shape) for i in range(2)]
    mp = lb.mp_init(fl, [{"D_b": 0.02, "k_a": [0.0], "k_d": [0.5]}] * 3, 64, 3, beta_mu_ex=[b[0], None, b[1]])
    for g, mu in ((0, b[0]), (1, np.zeros(m.shape)), (2, b[1])):
        X, Xa = lb.mp_state(mp, g, 0)
        w = np.exp(-mu)
        assert np.abs(X[0] - w / w.sum()).max() < 1e-15
        assert (Xa == 0).all()
    mp.free()
