"""GPU: the 2D cooperative path (ng_resident2d.hip), bit for bit against one
launch per step: grids of one and two strips, of one workgroup and the most,
ragged widths, every end kind and flux, launches of both parities, and a
rejected step."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}
ENDS = {
    "periodic": {},
    "walls": dict(bc=(1, 1, 2, 2)),
    "sector": dict(bc=(3, 1, 2, 2), source=(1e-2, 0.1, 0.5, 0.2), wedge=(0.0, 0.5, 0.5)),
}
# one workgroup (4x4, 60x12), one strip and a column more, an odd grid, one that
# fills every CU, more strips than rows
SHAPES = [(4, 4), (60, 12), (61, 13), (62, 48), (150, 131), (600, 599), (3001, 7)]


def pair(ng, gas, nx, ny, W, prec, **kw):
    a = ng.Solver(gas, nx, ny, W=W, precision=PREC[prec], **kw)
    b = ng.Solver(gas, nx, ny, W=W, precision=PREC[prec], **kw)
    b.set_coop(0)
    b.set_small_limit(0)
    return a, b


def same(a, b):
    da, db = a.diagnostics(), b.diagnostics()
    for key in ("t", "dt_last", "dt_next", "steps", "status", "flags", "smax", "rho_min", "p_min"):
        assert da[key] == db[key], key
    for q in (0, 3, 4):     # sums of the same numbers in another order
        assert da["total"][q] == pytest.approx(db["total"][q], rel=1e-12)
    assert np.array_equal(a.conserved(), b.conserved())
    return da


@pytest.mark.parametrize("flux", [0, 1], ids=["hllc", "hll"])
@pytest.mark.parametrize("ends", sorted(ENDS))
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("prec", sorted(PREC))
def test_shapes_equal_one_launch_per_step(prec, shape, ends, flux):
    from paper_1805_03442_amd import ng
    nx, ny = shape
    gas = wl.results_gas(0.5) if ends == "sector" else dict(wl.BASE_GAS, Q_T=2.0)
    r = np.random.Generator(np.random.PCG64(nx * ny))
    W = wl.uniform_state(gas, nx, ny)
    W[0] *= 1.0 + 0.02 * r.uniform(-1, 1, size=(ny, nx))
    W[1] = 0.05 * r.uniform(-1, 1, size=(ny, nx))
    W[2] = 0.05 * r.uniform(-1, 1, size=(ny, nx))
    print(prec, shape, ends, flux, flush=True)
    a, b = pair(ng, gas, nx, ny, W, prec, riemann=flux, h=1.0 / max(nx, ny), **ENDS[ends])
    for steps in (1, 6, 3):
        a.step(steps)
        b.step(steps)
        assert same(a, b)["status"] == 0
    t = a.diagnostics()["t"] * 1.35
    assert a.run_to_time(t) == b.run_to_time(t)
    assert same(a, b)["t"] == t
    a.close()
    b.close()


@pytest.mark.parametrize("shape", [(60, 12), (150, 131)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_rejected_step_keeps_the_last_state(shape):
    """A sink that takes the pressure below zero, first where the gas is
    densest: every workgroup rejects the same step."""
    from paper_1805_03442_amd import ng
    nx, ny = shape
    gas = dict(wl.BASE_GAS, Q0=0.0, I0=0.12 * nx, I_rho=1.0, I_T=0.0)
    W = wl.uniform_state(gas, nx, ny)
    W[0] += 0.1 * np.sin(2 * np.pi * (np.arange(nx) + 0.5) / nx)[None, :]
    a, b = pair(ng, gas, nx, ny, W, "fp64")
    a.step(300)
    b.step(300)
    d = same(a, b)
    assert d["status"] == ng.NG_EPHYS and 0 < d["steps"] < 300
    a.close()
    b.close()


def test_stalled_launch_ends(shape=(150, 131)):
    """No polls allowed: every workgroup leaves at its first wait, and the solve
    keeps a state of the per-step path."""
    from paper_1805_03442_amd import ng
    nx, ny = shape
    gas = dict(wl.BASE_GAS, Q_T=2.0)
    W = wl.random_field_2d(gas, 150, wl.rng(3), kmax=8, rms=1e-2)[:, :ny].copy()
    a, b = pair(ng, gas, nx, ny, W, "fp32")
    a.set_coop(-1, 0)
    a.step(50)
    d = a.diagnostics()
    assert d["status"] == ng.NG_ESTALL and d["steps"] < 50
    if d["steps"]:
        b.step(d["steps"])
    assert np.array_equal(a.conserved(), b.conserved())
    a.close()
    b.close()
