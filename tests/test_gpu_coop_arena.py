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
