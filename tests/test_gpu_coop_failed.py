"""GPU: a solve that has failed keeps its status, flags and last state through
later cooperative launches over it, as it does with one launch per step: alone
in 1D and 2D, rejected by the priming pass of a batch, and beside solves that
go on."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu


def failing(nx, ny=1):
    """A sink that takes the pressure below zero, first where the gas is densest."""
    gas = dict(wl.BASE_GAS, Q0=0.0, I0=0.12 * nx, I_rho=1.0, I_T=0.0)
    W = wl.uniform_state(gas, nx, ny)
    W[0] += 0.1 * np.sin(2 * np.pi * (np.arange(nx) + 0.5) / nx)[None, :]
    return gas, W


def sound(n):
    gas = dict(wl.BASE_GAS, Q_T=2.0)
    W = wl.uniform_state(gas, n)
    W[0, 0] += 1e-2 * np.sin(2 * np.pi * 2 * (np.arange(n) + 0.5) / n)
    return gas, W


def same(a, b):
    for key in ("t", "dt_last", "steps", "status", "flags", "smax", "rho_min", "p_min"):
        assert a[key] == b[key], key


@pytest.mark.parametrize("shape", [(200, 1), (3000, 1), (150, 131)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_lone_solve_keeps_its_failure(shape):
    from paper_1805_03442_amd import ng
    nx, ny = shape
    gas, W = failing(nx, ny)
    print("failed solve", shape, flush=True)
    res = []
    for coop in (-1, 0):
        s = ng.Solver(gas, nx, ny, W=W, precision=ng.NG_FP64)
        s.set_coop(coop)
        s.step(300)
        first, U = s.diagnostics(), s.conserved()
        assert first["status"] == ng.NG_EPHYS and first["flags"] & 4
        s.step(5)
        s.step(1)
        same(s.diagnostics(), first)
        assert np.array_equal(s.conserved(), U)
        res.append((first, U))
        s.close()
    same(res[0][0], res[1][0])
    assert np.array_equal(res[0][1], res[1][1])


@pytest.mark.parametrize("prec", ["fp64", "fp32", "mixed"])
def test_failed_member_beside_others(prec):
    """Members of one and of several workgroups, one of each rejected on the way;
    the others go on, each as with one launch per step."""
    from paper_1805_03442_amd import ng
    p = dict(fp64=ng.NG_FP64, fp32=ng.NG_FP32, mixed=ng.NG_MIXED)[prec]
    solves = [sound(500), failing(200), sound(9000), failing(7001), sound(61)]
    print("failed members", prec, flush=True)
    res = []
    for coop in (-1, 0):
        b = ng.Batch(8, 64 << 20, precision=p)
        b.set_coop(coop)
        slots = [b.add(g, W.shape[2], 1, W, 1e9) for g, W in solves]
        b.run(200)
        first = [b.diagnostics(i) for i in slots]
        for n in (20, 30):
            b.run(n)
        last = [b.diagnostics(i) for i in slots]
        for k, (f, d) in enumerate(zip(first, last)):
            if k in (1, 3):
                assert f["status"] == ng.NG_EPHYS and f["flags"] & 4 and f["steps"] < 200
                same(d, f)
            else:
                assert d["status"] == 0 and d["steps"] == 250
        assert sorted(b.poll()) == sorted([slots[1], slots[3]])
        res.append((last, [b.conserved(i) for i in slots]))
        b.close()
    for d, e, U, V in zip(res[0][0], res[1][0], res[0][1], res[1][1]):
        same(d, e)
        assert np.array_equal(U, V)
