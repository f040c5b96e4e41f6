"""The launch-shape tuner against the untuned solve: the shipped shapes leave 2D
grids alone that take the cooperative path without one, and tuning such a grid
keeps no shape."""
import json
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COOP_CELLS = 1 << 22        # the default of ng_set_coop


def test_shipped_shapes_are_for_larger_grids():
    with open(os.path.join(ROOT, "paper_1805_03442_amd", "tuning.json")) as f:
        keys = json.load(f)
    assert keys
    for k in keys:
        dim, nx, ny = re.fullmatch(r"(\d)d_\w+_(\d+)x(\d+)", k).groups()
        # a bucket's smallest grid is half its size
        assert dim == "1" or int(nx) * int(ny) / 2 > COOP_CELLS, k


@pytest.mark.gpu
@pytest.mark.parametrize("n", [256, 1024])
def test_tuning_keeps_only_what_beats_the_untuned_solve(n, tmp_path):
    from paper_1805_03442_amd import autotune, ng
    path = str(tmp_path / "tuning.json")
    stale = {autotune.key(n, n, ng.NG_FP32): dict(rows=4, waves=1, step_ms=1.0), "1d_fp32_64x1": dict(rows=1, waves=1, step_ms=1.0)}
    with open(path, "w") as f:
        json.dump(stale, f)
    print("tuning", n, flush=True)
    r = autotune.tune(n, n, ng.NG_FP32, steps=20, candidates=[(4, 1), (8, 4)], path=path)
    assert r["untuned_us_per_step"] < r["us_per_step"] and not r["kept"]
    assert autotune.lookup(n, n, ng.NG_FP32, path) is None
    assert autotune.lookup(64, 1, ng.NG_FP32, path) == (1, 1)
    from paper_1805_03442_amd import workloads as wl
    gas = dict(wl.BASE_GAS, Q_T=2.0)
    s = ng.Solver(gas, n, n, W=wl.uniform_state(gas, n, n), precision=ng.NG_FP32)
    assert not autotune.apply(s, path) and not autotune.apply(s)
    s.close()
