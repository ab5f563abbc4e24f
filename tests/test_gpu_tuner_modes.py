"""Plans of the tile tuner: a VACF and an uptake handle on the same medium with
the same species move different quantities and may need different plans, so
each has its own entry, in the process and in the cache file."""
import json

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


@pytest.mark.parametrize("prec", [32, 64])
@pytest.mark.parametrize("first", ["vacf", "uptake"])
def test_each_mode_keeps_its_plan(lb, monkeypatch, tmp_path, first, prec):
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("LBMP_TUNE_CACHE", str(cache))
    monkeypatch.delenv("LBMP_TILE", raising=False)
    # a shape of its own for every case: plans are also kept in the process
    m = inputs.random_mask(50, 41 + 2 * (prec == 64) + (first == "vacf"), 36, 0.2, seed=71)
    fl = lb.lb_flow_from_velocity(m, inputs.random_velocity(m, 0.01, seed=72))
    sp = {"D_b": 0.05, "k_a": [0.02, 0.05], "k_d": [0.01, 0.004]}
    init = {"vacf": lb.mp_init, "uptake": lb.mp_uptake_init}
    other = "uptake" if first == "vacf" else "vacf"
    plans = {}
    for mode in (first, other, first, other):
        h = init[mode](fl, sp, prec, 10)
        st = lb.mp_stats(h, 0)
        plans.setdefault(mode, []).append((st["kernel_variant"], st["tile_k"], st["species_per_block"]))
        lb.mp_step_n(h, 3)
        h.free()
    fl.free()
    lines = [json.loads(s) for s in cache.read_text().splitlines()]
    assert len(lines) == 2 and lines[0]["key"] != lines[1]["key"]
    for mode, e in zip((first, other), lines):
        plan = (e["variant"], e["K"], e["species_per_block"])
        assert plans[mode] == [plan, plan], mode
