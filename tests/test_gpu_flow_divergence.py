"""A flow solve that diverges says so (LBMP_ENUMERIC) in each of its forms: one
block for the whole solve, the pull table and the node map. Once a flow is NaN everywhere the maxima of the residual must not drop
them: a residual of zero would read as converged."""
import numpy as np
import pytest

from paper_1303_2470_amd import inputs

pytestmark = pytest.mark.gpu

LBMP_ENUMERIC = -7


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1303_2470_amd import lbmp
    lbmp.load_library()
    return lbmp


MASKS = {
    "one block": lambda: inputs.random_mask(9, 9, 9, 0.1, seed=2),
    "table": lambda: inputs.random_mask(32, 32, 30, 0.1, seed=3),
    "map": lambda: inputs.random_mask(64, 64, 64, 0.1, seed=4),
}


@pytest.mark.parametrize("check_every", [1, 100])
@pytest.mark.parametrize("name", MASKS)
def test_a_diverging_flow_is_refused(lb, name, check_every):
    with pytest.raises(lb.LbmpError) as e:
        lb.lb_flow_solve(MASKS[name](), tau=0.501, force=(0.7, 0.4, 0.2), tol=1e-8, max_steps=4000,
                         check_every=check_every)
    assert e.value.status == LBMP_ENUMERIC


@pytest.mark.parametrize("name", MASKS)
def test_an_ordinary_flow_is_not(lb, name):
    fl = lb.lb_flow_solve(MASKS[name](), tau=0.8, force=(1e-6, 0.0, 0.0), tol=1e-4, max_steps=20000)
    u = fl.velocity()
    assert fl.converged and np.isfinite(u).all() and np.abs(u).max() > 0.0
    fl.free()
