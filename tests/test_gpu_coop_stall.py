"""GPU: cooperative launches whose waits run out.  With a spin limit of one poll
every launch of several workgroups gives up early; the calls that read then find
every step that was asked for, as with one launch per step: diagnostics, the
state alone, runs to a time, the finished solves of a batch, members that end,
fail or never waited.  The same beside the library's own long kernel on another
stream, which holds half of the CUs for longer than the default limit.  A limit
of 0 asks for the stall: each member of a batch then keeps a state of its own."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}
GAS = dict(wl.BASE_GAS, Q_T=2.0)


def start(nx, ny=1, gas=GAS):
    W = wl.uniform_state(gas, nx, ny)
    W[0] += 1e-2 * np.sin(2 * np.pi * 2 * (np.arange(nx) + 0.5) / nx)[None, :]
    W[1] = 0.02
    return W


def same(a, b):
    for key in ("t", "dt_last", "dt_next", "steps", "status", "flags", "smax", "rho_min", "p_min"):
        assert a[key] == b[key], key


@pytest.mark.parametrize("prec", sorted(PREC))
@pytest.mark.parametrize("kind", ["1d", "source", "2d"])
def test_lone_solve_takes_every_step(kind, prec):
    from paper_1805_03442_amd import ng
    nx, ny = (150, 131) if kind == "2d" else (9000, 1)
    gas, kw = GAS, {}
    if kind == "source":
        gas, kw = wl.results_gas(0.5), dict(bc=(3, 2, 0, 0), source=(1e-2, 0.1))
    W = start(nx, ny, gas)
    print("stalled lone solve", kind, prec, flush=True)
    for first in ("state", "diagnostics", "time"):
        s = ng.Solver(gas, nx, ny, W=W, precision=PREC[prec], **kw)
        r = ng.Solver(gas, nx, ny, W=W, precision=PREC[prec], **kw)
        r.set_coop(0)
        r.set_small_limit(0)
        s.set_coop(-1, 1)
        for n in (40, 2, 90):
            s.step(n)
            r.step(n)
        if first == "state":
            assert np.array_equal(s.conserved(), r.conserved())
        elif first == "time":
            t = r.diagnostics()["t"] * 1.3
            assert s.run_to_time(t) == r.run_to_time(t)
        same(s.diagnostics(), r.diagnostics())
        s.step(5)       # without the limits of run_to_time
        r.step(5)
        s.set_coop(-1, 1)
        t = r.diagnostics()["t"] * 1.1
        assert s.run_to_time(t, 7) == r.run_to_time(t, 7)
        same(s.diagnostics(), r.diagnostics())
        assert np.array_equal(s.conserved(), r.conserved())
        s.close()
        r.close()


def fleet(ng, prec, coop, spin):
    """Solves of one and of several workgroups; one stops at a step count, one
    at a time, one is rejected."""
    sink = dict(wl.BASE_GAS, Q0=0.0, I0=0.12 * 7001, I_rho=1.0, I_T=0.0)
    b = ng.Batch(8, 64 << 20, precision=PREC[prec])
    b.set_coop(coop, spin)
    members = [(GAS, 200, 1e9, 1 << 40), (GAS, 20000, 1e9, 1 << 40), (GAS, 9000, 1e9, 33),
               (GAS, 12000, 0.4 * 50 / 12000, 1 << 40), (sink, 7001, 1e9, 1 << 40)]
    slots = [b.add(g, n, 1, start(n, 1, g), te, max_steps=ms) for g, n, te, ms in members]
    return b, slots


@pytest.mark.parametrize("prec", sorted(PREC))
def test_batch_members_take_every_step(prec):
    from paper_1805_03442_amd import ng
    print("stalled batch", prec, flush=True)
    out = []
    for coop, spin in ((-1, 1), (0, -1)):
        b, slots = fleet(ng, prec, coop, spin)
        b.run(20)
        late = b.add(GAS, 800, 1, start(800), 1e9)      # joins behind a launch that stalled
        b.run(100)
        done = sorted(b.poll())
        b.run(30)
        ids = slots + [late]
        out.append((done, b.active(), [b.conserved(i) for i in ids], [b.diagnostics(i) for i in ids]))
        b.close()
    assert out[0][:2] == out[1][:2]
    for U, V, d, e in zip(out[0][2], out[1][2], out[0][3], out[1][3]):
        same(d, e)
        assert np.array_equal(U, V)


@pytest.mark.parametrize("prec", sorted(PREC))
def test_batch_members_stall_each_for_itself(prec):
    """A limit of 0: the members of several workgroups stop, each at a step whose
    state is that of one launch per step, and stay there; the member of one
    workgroup, which waits for nobody, goes on."""
    from paper_1805_03442_amd import ng
    b, slots = fleet(ng, prec, -1, 0)
    print("batch with no polls", prec, flush=True)
    b.run(50)
    first = [b.diagnostics(i) for i in slots]
    assert first[0]["status"] == 0 and first[0]["steps"] == 50
    assert [d["status"] for d in first[1:]] == [ng.NG_ESTALL] * 4
    b.set_coop(-1)
    b.run(50)
    assert b.diagnostics(slots[0])["steps"] == 100
    for d, i in zip(first[1:], slots[1:]):
        same(b.diagnostics(i), d)
    r, rs = fleet(ng, prec, 0, -1)
    taken = 0
    for want, i, j in sorted((d["steps"], i, j) for d, i, j in zip(first[1:], slots[1:], rs[1:])):
        if want > taken:
            r.run(want - taken)
        taken = want
        assert np.array_equal(b.conserved(i), r.conserved(j))
    b.close()
    r.close()


def test_beside_a_long_kernel():
    """128 small solves in one persistent launch of two seconds hold a CU each;
    grids that need all CUs then stall, and still take their steps."""
    import time

    import torch
    from paper_1805_03442_amd import ng
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    still = dict(wl.BASE_GAS, Q0=0.0, I0=0.0)
    b = ng.Batch(128, 256 << 20, precision=ng.NG_FP64, stream=one)
    for _ in range(128):
        b.add(still, 48, 40, start(48, 40, still), 1e9)
    b.run(200)
    b.poll()
    t = time.perf_counter()
    b.run(1000)
    b.poll()
    hold = int(2.0 * 1000 / (time.perf_counter() - t))
    for prec in ("fp64", "fp32"):
        print("beside a long kernel", prec, hold, "steps", flush=True)
        s = ng.Solver(GAS, 600, 600, W=start(600, 600), precision=PREC[prec], stream=two)
        s.step(5)
        assert s.diagnostics()["steps"] == 5
        b.run(hold)
        s.step(50)
        d = s.diagnostics()
        b.poll()
        r = ng.Solver(GAS, 600, 600, W=start(600, 600), precision=PREC[prec])
        r.set_coop(0)
        r.step(55)
        same(d, r.diagnostics())
        assert d["status"] == 0 and d["steps"] == 55
        assert np.array_equal(s.conserved(), r.conserved())
        s.close()
        r.close()
    b.close()
