"""The static flow solve at its limit, whose scratch has no room for tiled
populations, against the solve with all the room it asks for: the same
velocities in a comparable time (both stored so that a wave's accesses are
contiguous; 17 and 12 ms on this lattice, where populations stored node by node
took 49)."""
import time

import numpy as np
import pytest

from paper_1303_2470_amd import inputs

pytestmark = pytest.mark.gpu


def test_populations_without_tiles():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_2470_amd import lbmp as lb
    m = inputs.bulk_mask(233, 50, 30)  # two nodes short of the limit, 196 short of full tiles
    assert m.size == lb.lb_flow_static_max_nodes() - 2
    args = dict(tau=0.9, force=(1e-6, 2e-6, 0.0), tol=0.0, max_steps=600, allow_unconverged=True)
    best, u = {}, {}
    for solve in (lb.lb_flow_solve_static, lb.lb_flow_solve):
        t = []
        for _ in range(4):
            t0 = time.perf_counter()
            f = solve(m, **args)
            t.append(time.perf_counter() - t0)
            u[solve] = f.velocity()
            f.free()
        best[solve] = min(t)
    assert np.array_equal(u[lb.lb_flow_solve_static], u[lb.lb_flow_solve])
    assert best[lb.lb_flow_solve_static] < 2.5 * best[lb.lb_flow_solve], best
