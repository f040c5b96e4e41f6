"""GPU: reading a state back (the conversion kernel, the pinned staging taken
half by half, the host threads that copy out of it) at sizes around one piece
of the least staging (64 KB) and of the most (16 MiB).

FP64 stores the conserved planes themselves, so they come back bit for bit;
the primitive planes are the same operations NumPy does on them, in the same
order up to the grouping of p, whose terms are a few times p: 16 units of
rounding.  FP32 rounds each deviation from the reference once (2^-24 of it),
mixed precision holds it in FP64."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [(5, 1), (2047, 1), (2048, 1), (2049, 1), (524287, 1), (524289, 1), (1300001, 1),
         (41, 40), (647, 648), (1500, 1201)]


@pytest.mark.parametrize("prec", ["fp64", "fp32", "mixed"])
@pytest.mark.parametrize("shape", SIZES, ids=lambda s: f"{s[0]}x{s[1]}")
def test_read_out(shape, prec):
    import torch
    from paper_1805_03442_amd import ng
    assert torch.cuda.is_available()
    nx, ny = shape
    gas = dict(wl.BASE_GAS)
    r = np.random.Generator(np.random.PCG64(nx))
    W = wl.uniform_state(gas, nx, ny)
    W[[0, 3, 4]] *= 1.0 + 1e-2 * r.uniform(-1, 1, (3, ny, nx))
    W[1] = 1e-2 * r.uniform(-1, 1, (ny, nx))
    if ny > 1:
        W[2] = 1e-2 * r.uniform(-1, 1, (ny, nx))
    rho, u, v, p, ev = W
    U = np.stack([rho, rho * u, rho * v, p / (gas["gamma"] - 1.0) + 0.5 * rho * (u * u + v * v) + ev, ev])
    print(f"read-out {nx}x{ny} {prec}", flush=True)
    s = ng.Solver(gas, nx, ny, U=U, precision=dict(fp64=ng.NG_FP64, fp32=ng.NG_FP32, mixed=ng.NG_MIXED)[prec])
    C, Q = s.conserved(), s.primitive()
    assert np.array_equal(C, s.conserved()) and np.array_equal(Q, s.primitive())
    s.close()
    if prec == "fp64":
        assert np.array_equal(C, U)
    # deviations are at most 5 % of values of order one
    eps = dict(fp64=2.0 ** -53, fp32=2.0 ** -24 * 0.1, mixed=2.0 ** -53)[prec]
    scale = np.abs(U).max(axis=(1, 2), keepdims=True) + np.abs(U[0]).max()
    assert (np.abs(C - U) <= 4 * eps * scale).all()
    W[1:3] = U[1:3] / U[0]
    scale = np.abs(W).max() + np.abs(U).max()
    assert (np.abs(Q - W) <= 16 * eps * scale).all()
