"""GPU: batches of 1D solves side by side in cooperative launches, bit for bit
against one launch per step: one and several workgroups per solve, cells in LDS
and in the state buffers, several kernels in one batch, solves that end early,
more solves than one launch holds, and a 2D solve beside them."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}


def members(prec, sizes, seed):
    """(gas, nx, ny, W, kwargs): ends, fluxes and closures in turn."""
    r = np.random.Generator(np.random.PCG64(seed))
    out = []
    for i, n in enumerate(sizes):
        gas = dict(wl.BASE_GAS, Q_T=float((2.0, 1.0, 1.3)[i % 3]), tau0=float(r.uniform(0.05, 0.3)))
        kw = {}
        if i % 4 == 1:
            kw = dict(bc=(1, 2, 0, 0))
        elif i % 4 == 2:
            gas, kw = wl.results_gas(0.5), dict(bc=(3, 2, 0, 0), source=(1e-2, 0.1))
        if i % 5 == 3:
            kw["riemann"] = 1
            if prec == "fp64":
                kw["scheme"] = 1
        x = (np.arange(n) + 0.5) / n
        W = wl.uniform_state(gas, n)
        W[0] += 1e-2 * np.sin(2 * np.pi * (1 + i % 5) * x)
        W[1] = 0.1 * np.cos(2 * np.pi * x)
        out.append((gas, n, 1, W, kw))
    return out


def run(ng, prec, solves, coop, steps, ends, max_steps):
    room = sum(ng.Batch.solve_bytes(n, ny, PREC[prec]) for _, n, ny, _, _ in solves)
    b = ng.Batch(len(solves) + 1, int(room * 1.1) + (64 << 20), precision=PREC[prec])
    b.set_coop(coop)
    slots = [b.add(g, n, ny, W, t_end=te, max_steps=ms, **kw)
             for (g, n, ny, W, kw), te, ms in zip(solves, ends, max_steps)]
    for k in steps:
        b.run(k)
    b.poll()
    res = [(b.conserved(s), b.diagnostics(s)) for s in slots]
    b.close()
    return res


def same(a, c):
    for (Ua, da), (Ub, db) in zip(a, c):
        for key in ("t", "dt_last", "dt_next", "steps", "status", "flags", "smax", "rho_min"):
            assert da[key] == db[key], key
        assert da["src_budget"][1] == pytest.approx(db["src_budget"][1], rel=1e-9, abs=1e-13)
        assert np.array_equal(Ua, Ub)


@pytest.mark.parametrize("prec", sorted(PREC))
@pytest.mark.parametrize("sizes", [
    (5, 61, 240, 241, 1003),                         # one workgroup each, ragged ends
    (4096, 70001, 200, 33333, 60, 1601, 58, 12345),  # several per solve
    (300001, 400003, 150001, 61),                    # beyond LDS in FP64 and mixed
], ids=["small", "uneven", "large"])
def test_fleet_equals_one_launch_per_step(prec, sizes):
    from paper_1805_03442_amd import ng
    solves = members(prec, sizes, len(sizes))
    if sizes[0] == 4096:        # and a 2D solve beside them
        gas = dict(wl.BASE_GAS, Q_T=2.0)
        solves.append((gas, 90, 70, wl.random_field_2d(gas, 90, wl.rng(3), kmax=6, rms=1e-2)[:, :70].copy(), {}))
    print(prec, sizes, flush=True)
    ends = [1e9] * len(solves)
    stop = [1 << 40] * len(solves)
    stop[1] = 9                  # one stops inside a launch
    ends[0] = 0.4 * 3.5 / sizes[0] / 1.3   # and one lands on its end time
    args = (ng, prec, solves)
    same(run(*args, -1, (1, 7, 12), ends, stop), run(*args, 0, (1, 7, 12), ends, stop))


def test_more_solves_than_one_launch_holds():
    from paper_1805_03442_amd import ng
    solves = members("fp32", [64 + 7 * (i % 40) for i in range(900)], 9)
    ends, stop = [1e9] * 900, [1 << 40] * 900
    same(run(ng, "fp32", solves, -1, (6,), ends, stop), run(ng, "fp32", solves, 0, (6,), ends, stop))
