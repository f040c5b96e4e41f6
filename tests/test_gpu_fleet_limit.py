"""GPU: where a batch of FP64 solves leaves the cooperative launches: 45000
segments of one kernel, whatever the other kernels have.  The states do not
depend on it.  Whether a call was cooperative shows at a spin limit of 0, where a
launch of several workgroups stalls at its first wait and no other path does."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

SIZE = 90000        # 1500 segments


@pytest.mark.parametrize("counts,taken", [((29,), True), ((31,), False), ((20, 20), True), ((2, 31), False)],
                         ids=lambda v: str(v))
def test_limit_is_per_kernel(counts, taken):
    from paper_1805_03442_amd import ng
    gases = [dict(wl.BASE_GAS, Q_T=2.0), dict(wl.BASE_GAS, Q_T=1.0)]
    total = sum(counts)
    print("segments", counts, flush=True)
    res = []
    for coop, spin in ((-1, 0), (-1, -1), (0, -1)):
        b = ng.Batch(total, total * ng.Batch.solve_bytes(SIZE, 1, ng.NG_FP64) + (64 << 20), precision=ng.NG_FP64)
        b.set_coop(coop, spin)
        slots = []
        for gas, n in zip(gases, counts):
            W = wl.uniform_state(gas, SIZE)
            W[0] += 1e-2 * np.sin(2 * np.pi * 5 * (np.arange(SIZE) + 0.5) / SIZE)
            slots += [b.add(gas, SIZE, 1, W, 1e9) for _ in range(n)]
        b.run(12)
        ends = (slots[0], slots[-1])
        d = [b.diagnostics(i) for i in ends]
        if spin == 0:
            assert [x["status"] for x in d] == [ng.NG_ESTALL if taken else 0] * 2
        else:
            res.append(([(x["t"], x["dt_next"], x["steps"], x["status"]) for x in d], [b.conserved(i) for i in ends]))
        b.close()
    assert res[0][0] == res[1][0] and res[0][0][0][2:] == (12, 0)
    for U, V in zip(res[0][1], res[1][1]):
        assert np.array_equal(U, V)
