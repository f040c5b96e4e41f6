"""GPU: how many cells a lone 2D solve may have on the cooperative path.  The FP64
kernels without compiled closures leave it earlier, the FP32 HLL kernel somewhat; a
limit set by the caller holds for all.  Whether a call was cooperative shows at a
spin limit of 0, where it stalls at its first wait and no other path does."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}
BASE = dict(wl.BASE_GAS, Q_T=2.0)
KINDS = {   # gas, arguments, the last of SHAPES that is cooperative in FP64
    "periodic": (BASE, {}, 7),
    "section3_walls": (wl.results_gas(0.5), dict(bc=(1, 1, 2, 2)), 7),
    "walls": (BASE, dict(bc=(1, 1, 2, 2)), 1),
    "section3": (wl.results_gas(0.5), {}, 3),
    "general": (dict(BASE, Q_T=1.3), {}, 4),
    "general_walls": (dict(BASE, Q_T=1.3), dict(bc=(1, 1, 2, 2)), 4),
    "hll": (BASE, dict(riemann=1), 1),
    "general_hll": (dict(BASE, Q_T=1.3), dict(riemann=1), 4),
}
SHAPES = ((300, 300), (240, 512), (240, 513), (240, 700), (450, 450),    # 2048, 2052, 2800 rows
          (451, 450), (2048, 1792), (2048, 1793), (2100, 2000))


def run(ng, prec, shape, kind, max_cells, spin, steps=8):
    gas, kw, _ = KINDS[kind]
    nx, ny = shape
    W = wl.uniform_state(gas, nx, ny)
    W[0] += 1e-2 * np.sin(2 * np.pi * 2 * (np.arange(nx) + 0.5) / nx)[None, :]
    s = ng.Solver(gas, nx, ny, W=W, precision=PREC[prec], **kw)
    s.set_coop(max_cells, spin)
    s.step(steps)
    d = s.diagnostics()
    U = s.conserved() if spin != 0 else None
    s.close()
    return d, U


@pytest.mark.parametrize("kind", sorted(KINDS))
@pytest.mark.parametrize("prec", sorted(PREC))
def test_limits(prec, kind):
    from paper_1805_03442_amd import ng
    print("cooperative limit", prec, kind, flush=True)
    last = KINDS[kind][2] if prec == "fp64" else 6 if prec == "fp32" and kind.endswith("hll") else 7
    for shape, max_cells, taken in [(sh, -1, i <= last) for i, sh in enumerate(SHAPES)] + [((700, 600), 1 << 22, True)]:
        d, _ = run(ng, prec, shape, kind, max_cells, 0)
        assert (d["status"] == ng.NG_ESTALL) == taken, (shape, max_cells)
    a, U = run(ng, prec, (700, 600), kind, 1 << 22, -1)
    b, V = run(ng, prec, (700, 600), kind, 0, -1)
    assert a["status"] == b["status"] == 0 and a["t"] == b["t"] and a["dt_next"] == b["dt_next"]
    assert np.array_equal(U, V)
