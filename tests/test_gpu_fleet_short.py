"""GPU: short calls of a batch of 1D solves take the persistent kernel and one
launch per step, long ones the cooperative launches; the states do not depend on
it.  Whether a call was cooperative shows at a spin limit of 0, where a launch of
several workgroups stalls at its first wait and no other path does."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

PREC = {"fp64": 0, "fp32": 1, "mixed": 2}
GAS = dict(wl.BASE_GAS, Q_T=2.0)


def batch(ng, prec, sizes, coop=-1, spin=-1):
    b = ng.Batch(len(sizes), 96 << 20, precision=PREC[prec])
    b.set_coop(coop, spin)
    slots = []
    for k, n in enumerate(sizes):
        W = wl.uniform_state(GAS, n)
        W[0] += 1e-2 * np.sin(2 * np.pi * (1 + k % 3) * (np.arange(n) + 0.5) / n)
        slots.append(b.add(GAS, n, 1, W, 1e9))
    return b, slots


# sizes, a call that is not worth a cooperative launch, one that is
CASES = [((1000, 1000), 3, 40), ((600,) * 8, 3, 40), ((1000, 20000), 3, 12), ((9000, 20000), 3, 12),
         ((700,) * 300, 4, 12)]


@pytest.mark.parametrize("prec", sorted(PREC))
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{len(c[0])}x{c[0][-1]}")
def test_short_calls_keep_their_paths(case, prec):
    from paper_1805_03442_amd import ng
    sizes, short, long = case
    print("short calls", prec, sizes[:2], len(sizes), flush=True)
    b, slots = batch(ng, prec, sizes, spin=0)
    for n in (short, 1, 2):
        b.run(n)
    assert all(b.diagnostics(i)["status"] == 0 for i in slots[:9])
    b.run(long)
    assert any(b.diagnostics(i)["status"] == ng.NG_ESTALL for i in slots[:9])
    b.close()
    out = []
    for coop in (-1, 0):
        b, slots = batch(ng, prec, sizes, coop)
        for n in (short, long, 1, 2, long + 60, short):
            b.run(n)
        d = [b.diagnostics(i) for i in slots]
        assert all(x["steps"] == 2 * (short + long) + 63 and x["status"] == 0 for x in d)
        out.append(([(x["t"], x["dt_next"], x["smax"]) for x in d], [b.conserved(i) for i in slots]))
        b.close()
    assert out[0][0] == out[1][0]
    for U, V in zip(out[0][1], out[1][1]):
        assert np.array_equal(U, V)
