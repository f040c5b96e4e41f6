"""GPU: the cooperative path of a batch in arenas of every size.  Whether a call
took it shows at a spin limit of 0, where a launch of several workgroups stalls
at its first wait and no other path does."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}
GAS = dict(wl.BASE_GAS, Q_T=2.0)


def start(nx, ny=1, m=2):
    W = wl.uniform_state(GAS, nx, ny)
    W[0] += 1e-2 * np.sin(2 * np.pi * m * (np.arange(nx) + 0.5) / nx)[None, :]
    W[1] = 0.02
    return W


def lone(ng, arena, prec, nx, ny, coop=-1, spin=-1):
    b = ng.Batch(4, int(arena), precision=PREC[prec])
    b.set_coop(coop, spin)
    return b, b.add(GAS, nx, ny, start(nx, ny), 1e9)


def cooperative(ng, arena, prec, nx, ny):
    b, i = lone(ng, arena, prec, nx, ny, spin=0)
    b.run(40)
    stalled = b.diagnostics(i)["status"] == ng.NG_ESTALL
    b.close()
    return stalled


def check_lone(ng, arena, prec, nx, ny):
    """Long and short calls in turn, against one launch per step."""
    assert cooperative(ng, arena, prec, nx, ny)
    out = []
    for coop in (-1, 0):
        b, i = lone(ng, arena, prec, nx, ny, coop)
        if coop == 0:
            b.set_small_limit(0)
        for n in (30, 1, 17, 2, 5):
            b.run(n)
        d = b.diagnostics(i)
        out.append((b.conserved(i), [d[k] for k in ("t", "dt_next", "steps", "status", "smax", "rho_min")]))
        b.close()
    assert out[0][1] == out[1][1] and out[0][1][2:4] == [55, 0]
    assert np.array_equal(out[0][0], out[1][0])


@pytest.mark.parametrize("prec,nx,ny,arena", [
    ("fp32", 1 << 16, 1, 8.6e6), ("fp64", 1 << 16, 1, 8.6e6), ("fp32", 1 << 18, 1, 16e6),
    ("mixed", 1 << 17, 1, 11e6), ("fp32", 300, 290, 6e6),
], ids=lambda v: str(v))
def test_lone_solve_on_the_workgroups_there_is_room_for(prec, nx, ny, arena):
    """Solves whose full shape has more workgroups than such an arena has room
    for in 1/64 of it."""
    from paper_1805_03442_amd import ng
    print("lone solve", prec, nx, ny, arena, flush=True)
    check_lone(ng, arena, prec, nx, ny)


@pytest.mark.parametrize("prec,nx,ny,arena", [
    ("fp32", 1 << 16, 1, 2.5e6), ("fp32", 20000, 1, 1.2e6), ("fp64", 1024, 1, 6e5),
    ("mixed", 1024, 1, 6e5), ("fp64", 4000, 1, 5e6), ("fp32", 150, 131, 3e6),
], ids=lambda v: str(v))
def test_lone_solve_in_a_small_arena(prec, nx, ny, arena):
    from paper_1805_03442_amd import ng
    print("lone solve in a small arena", prec, nx, ny, arena, flush=True)
    check_lone(ng, arena, prec, nx, ny)


@pytest.mark.parametrize("prec,nx,ny", [("fp32", 1 << 16, 1), ("fp64", 20011, 1), ("mixed", 9000, 1),
                                        ("fp32", 600, 600)], ids=lambda v: str(v))
def test_lone_solve_fills_the_arena(prec, nx, ny):
    """No space beside the solve: the exchange lies in its reduction records,
    which calls of one launch per step use in between."""
    from paper_1805_03442_amd import ng
    need = ng.Batch.solve_bytes(nx, ny, PREC[prec])
    lo, hi = need, need + (1 << 20)
    while hi - lo > 256:        # the least arena the solve fits in
        mid = (lo + hi) // 2
        try:
            b, i = lone(ng, mid, prec, nx, ny)
            b.close()
        except ng.NgError:
            i = None
        lo, hi = (mid, hi) if i is None else (lo, mid)
    print("lone solve fills the arena", prec, nx, ny, need, hi, flush=True)
    check_lone(ng, hi, prec, nx, ny)


@pytest.mark.parametrize("count", [1, 6, 30])
def test_an_arena_holds_its_solves(count):
    """Half a solve beyond the solves is room enough for the header, also when
    launches have run in between."""
    from paper_1805_03442_amd import ng
    n = 1 << 14 if count > 1 else 1 << 16
    need = ng.Batch.solve_bytes(n, 1, ng.NG_FP32)
    b = ng.Batch(16 if count < 16 else 64, count * need + need // 2, precision=ng.NG_FP32)
    W = start(n)
    slots = []
    for k in range(count):
        assert b.fits(n, 1)
        slots.append(b.add(GAS, n, 1, W, 1e9))
        assert slots[-1] is not None
        b.run(12)
    assert b.add(GAS, n, 1, W, 1e9) is None
    print("arena of", count, flush=True)
    r = ng.Solver(GAS, n, 1, W=W, precision=ng.NG_FP32)
    for k in reversed(range(count)):
        r.step(12)
        assert b.diagnostics(slots[k])["steps"] == 12 * (count - k)
        assert np.array_equal(b.conserved(slots[k]), r.conserved())
    r.close()
    b.close()


@pytest.mark.parametrize("prec", sorted(PREC))
def test_admissions_and_removals_as_without_the_path(prec):
    """A seeded run of admissions, removals and calls in an arena that is nearly
    full all the time: the same solves are admitted, to the same slots, and take
    the same steps, as with the path off."""
    from paper_1805_03442_amd import ng
    arena = 9 * ng.Batch.solve_bytes(12000, 1, PREC[prec])
    out = []
    for coop in (-1, 0):
        r = np.random.Generator(np.random.PCG64(77))
        b = ng.Batch(12, arena, precision=PREC[prec])
        b.set_coop(coop)
        log, live = [], []
        for k in range(60):
            what = r.random()
            if what < 0.5:
                n, m = int(r.integers(200, 24000)), int(r.integers(1, 5))
                fits = b.fits(n, 1)
                slot = b.add(GAS, n, 1, start(n, 1, m), 1e9)
                assert fits == (slot is not None)
                log.append(slot)
                if slot is not None:
                    live.append(slot)
            elif what < 0.65 and live:
                slot = live.pop(int(r.integers(len(live))))
                log.append(b.diagnostics(slot)["steps"])
                b.remove(slot)
            else:
                b.run(int(r.integers(1, 25)))
        log += [(i, b.diagnostics(i)["steps"], b.diagnostics(i)["t"], b.diagnostics(i)["status"]) for i in live]
        out.append((log, [b.conserved(i) for i in live]))
        b.close()
    assert out[0][0] == out[1][0] and len(out[0][1]) > 2
    for U, V in zip(out[0][1], out[1][1]):
        assert np.array_equal(U, V)


def test_several_solves_take_the_path_in_a_small_arena():
    from paper_1805_03442_amd import ng
    b = ng.Batch(4, 4 << 20, precision=ng.NG_FP32)
    b.set_coop(-1, 0)
    slots = [b.add(GAS, n, 1, start(n), 1e9) for n in (9000, 20000, 5000)]
    b.run(100)
    assert [b.diagnostics(i)["status"] for i in slots] == [ng.NG_ESTALL] * 3
    b.close()
