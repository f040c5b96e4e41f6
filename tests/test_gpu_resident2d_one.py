"""GPU: the 2D cooperative path on one workgroup (60x4 is the largest grid there),
bit for bit against one launch per step: a source that drives the ghosts, and a
rejected step."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu


def both(ng, gas, W, prec, steps, **kw):
    out = []
    for coop in (-1, 0):
        s = ng.Solver(gas, 60, 4, W=W, precision=prec, **kw)
        s.set_coop(coop)
        if coop == 0:
            s.set_small_limit(0)
        s.step(steps)
        s.step(7)
        d = s.diagnostics()
        out.append(([d[k] for k in ("t", "dt_last", "steps", "status", "flags", "smax", "rho_min", "p_min")], s.conserved()))
        s.close()
    assert out[0][0] == out[1][0]
    assert np.array_equal(out[0][1], out[1][1])
    return dict(zip(("t", "dt_last", "steps", "status"), out[0][0]))


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp64", "fp32", "mixed"])
def test_source(prec):
    from paper_1805_03442_amd import ng
    gas = wl.results_gas(0.5)
    print("one workgroup, source", prec, flush=True)
    d = both(ng, gas, wl.uniform_state(gas, 60, 4), prec, 50, bc=(3, 1, 2, 2), source=(1e-2, 0.1))
    assert d["status"] == 0 and d["steps"] == 57


@pytest.mark.parametrize("prec", [0, 1, 2], ids=["fp64", "fp32", "mixed"])
def test_rejected_step(prec):
    from paper_1805_03442_amd import ng
    gas = dict(wl.BASE_GAS, Q0=0.0, I0=0.12 * 60, I_rho=1.0, I_T=0.0)
    W = wl.uniform_state(gas, 60, 4)
    W[0] += 0.1 * np.sin(2 * np.pi * (np.arange(60) + 0.5) / 60)[None, :]
    print("one workgroup, rejected", prec, flush=True)
    d = both(ng, gas, W, prec, 300)
    assert d["status"] == ng.NG_EPHYS and 0 < d["steps"] < 300
