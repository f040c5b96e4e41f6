"""GPU test of ng_step_static's launches: the priming pass whose last
workgroup folds the records, at one workgroup, at the numbers of workgroups it
is held to and beyond, and the step with its own fold (up to 256 workgroups) or
the folding kernel's, with one, two and four rows per work item, in both
dimensions, against the same step through the solver entry points, bit for bit.
Each grid is stepped three times in turn with a small one, so that each call
starts from the scratch another one left.
"""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(5, 1), (61, 1), (7, 9), (150, 150), (250, 250), (380, 400), (390, 420),
                                   (700, 300), (200003, 1)])
def test_static_step_in_turn(nx, ny):
    import torch
    from paper_1805_03442_amd import ng
    assert torch.cuda.is_available()
    gas = dict(wl.BASE_GAS, Q_T=2.0)
    r = np.random.Generator(np.random.PCG64(nx + ny))

    def start(nx, ny):
        W = np.empty((5, ny, nx))
        W[0] = gas["rho0"] * (1 + 0.05 * r.uniform(-1, 1, (ny, nx)))
        W[1:3] = 0.05 * r.normal(size=(2, ny, nx))
        W[3] = gas["R"] * gas["rho0"] * gas["T0"] * (1 + 0.05 * r.uniform(-1, 1, (ny, nx)))
        W[4] = gas["rho0"] * gas["Cv"] * gas["T0"]
        if ny == 1:
            W[2] = 0.0
        s = ng.Solver(gas, nx, ny, W=W, precision=ng.NG_FP64)
        U0 = s.conserved()
        s.step(1)
        U1, d = s.conserved(), s.diagnostics()
        s.close()
        return U0, U1, d

    grids = [((nx, ny), start(nx, ny)), ((64, 1), start(64, 1))]
    print(f"static step {nx}x{ny}", flush=True)
    for _ in range(3):
        for (mx, my), (U0, U1, d1) in grids:
            comps = [0, 1, 2, 3, 4] if my > 1 else [0, 1, 3, 4]
            src = torch.from_numpy(np.ascontiguousarray(U0[comps])).cuda()
            dst = torch.full_like(src, float("nan"))
            d = ng.step_static(gas, mx, my, src, dst)
            assert np.array_equal(dst.cpu().numpy().reshape(U1[comps].shape), U1[comps])
            assert d["dt_last"] == d1["dt_last"] and d["status"] == 0 and d["steps"] == 1


@pytest.mark.parametrize("nx,ny", [(100, 1), (700, 300)])
def test_static_step_rejects_bad_state(nx, ny):
    """A non-finite cell, and one without pressure, are rejected by the priming
    pass; the next call on a sound state is accepted."""
    import torch
    from paper_1805_03442_amd import ng
    assert torch.cuda.is_available()
    gas = dict(wl.BASE_GAS)
    nc = 5 if ny > 1 else 4
    good = torch.zeros(nc, nx * ny, dtype=torch.float64, device="cuda")
    good[0] = gas["rho0"]
    good[-1] = gas["rho0"] * gas["Cv"] * gas["T0"]
    good[-2] = good[-1] + gas["R"] * gas["rho0"] * gas["T0"] / (gas["gamma"] - 1.0)
    dst = torch.empty_like(good)
    for comp, value in ((1, float("nan")), (nc - 2, 0.0)):
        bad = good.clone()
        bad[comp, nx * ny - 1] = value
        print(f"static step of a bad state {nx}x{ny} {value}", flush=True)
        with pytest.raises(ng.NgError) as e:
            ng.step_static(gas, nx, ny, bad, dst)
        assert e.value.code == ng.NG_EPHYS
        assert ng.step_static(gas, nx, ny, good, dst)["steps"] == 1
