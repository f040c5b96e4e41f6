"""GPU: the cooperative path's launch shapes and endings (ng_resident.hip),
bit for bit against one launch per step.

Sizes sit at the edges of the shape's rules: one workgroup and two, a ragged
last segment of one cell, the most cells that stay in LDS and one more (they
then stay in the state buffers)."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}
# most cells in LDS: 156 KB hold two copies of w-cell segments with halos,
# on 256 CUs
LDS64 = (156 * 1024 // 64 - 4) // 60 * 60 * 256
LDS32 = (156 * 1024 // 32 - 4) // 60 * 60 * 256
CASES = [("fp64", 181), ("fp64", 240), ("fp64", 241), ("fp64", 481), ("fp32", 480), ("fp32", 481),
         ("mixed", 541), ("fp64", LDS64), ("fp64", LDS64 + 1), ("fp32", LDS32),
         ("fp32", LDS32 + 1), ("mixed", LDS64 + 1)]


def pair(ng, gas, n, W, prec, **kw):
    a = ng.Solver(gas, n, 1, W=W, precision=PREC[prec], **kw)
    b = ng.Solver(gas, n, 1, W=W, precision=PREC[prec], **kw)
    b.set_coop(0)
    b.set_small_limit(0)
    return a, b


def same(a, b, totals=True):
    da, db = a.diagnostics(), b.diagnostics()
    for key in ("t", "dt_last", "dt_next", "steps", "status", "flags", "smax", "rho_min", "p_min"):
        assert da[key] == db[key] or (np.isnan(da[key]) and np.isnan(db[key])), key
    if totals:
        # sums of the same numbers in another order
        for q in (0, 3, 4):
            assert da["total"][q] == pytest.approx(db["total"][q], rel=1e-12)
    assert np.array_equal(a.conserved(), b.conserved())
    return da


@pytest.mark.parametrize("ends", ["periodic", "walls", "source"])
@pytest.mark.parametrize("prec,n", CASES, ids=lambda v: str(v))
def test_shapes_equal_one_launch_per_step(prec, n, ends):
    from paper_1805_03442_amd import ng
    gas, kw = dict(wl.BASE_GAS, Q_T=2.0), {}
    if ends == "walls":
        kw = dict(bc=(1, 1, 0, 0))
    elif ends == "source":
        gas, kw = wl.results_gas(0.5), dict(bc=(3, 2, 0, 0), source=(1e-2, 0.1))
    x = (np.arange(n) + 0.5) / n
    W = wl.uniform_state(gas, n)
    W[0] += 1e-2 * np.sin(2 * np.pi * 3 * x)
    W[1] = 0.1 * np.cos(2 * np.pi * x)
    print(prec, n, ends, flush=True)
    a, b = pair(ng, gas, n, W, prec, **kw)
    for steps in (1, 6, 7):     # launches of both parities, one after another
        a.step(steps)
        b.step(steps)
        assert same(a, b)["status"] == 0
    a.close()
    b.close()


@pytest.mark.parametrize("scheme", [0, 1], ids=["muscl", "csph"])
@pytest.mark.parametrize("n", [200, 3000, 100003])
def test_rejected_step_keeps_the_last_state(n, scheme):
    """A sink strong enough to take the pressure below zero within a hundred
    steps, first where the gas is densest: the step is rejected by every
    workgroup, with the state, totals and flags of the step before."""
    from paper_1805_03442_amd import ng
    gas = dict(wl.BASE_GAS, Q0=0.0, I0=0.12 * n, I_rho=1.0, I_T=0.0)
    W = wl.uniform_state(gas, n)
    W[0] += 0.1 * np.sin(2 * np.pi * (np.arange(n) + 0.5) / n)
    print(n, scheme, flush=True)
    a, b = pair(ng, gas, n, W, "fp64", scheme=scheme, riemann=1)
    a.step(200)
    b.step(200)
    d = same(a, b)
    assert d["status"] == ng.NG_EPHYS and d["steps"] < 200
    a.close()
    b.close()
