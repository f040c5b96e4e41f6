"""GPU: stepping calls under stream capture.  ng_step refuses (it lifts the limits
of ng_run_to_time by what the host knows, which a replay does not), and the
capture and the solver go on; ng_batch_run is recorded, and every replay takes its
steps, with the program's own calls in between, as without a graph."""
import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

GAS = dict(wl.BASE_GAS, Q_T=2.0)


def start(nx, ny=1):
    W = wl.uniform_state(GAS, nx, ny)
    W[0] += 1e-2 * np.sin(2 * np.pi * 2 * (np.arange(nx) + 0.5) / nx)[None, :]
    return W


@pytest.mark.parametrize("shape", [(1024, 1), (150, 131)], ids=lambda s: f"{s[0]}x{s[1]}")
def test_step_is_refused(shape):
    import torch
    from paper_1805_03442_amd import ng
    nx, ny = shape
    st = torch.cuda.Stream()
    s = ng.Solver(GAS, nx, ny, W=start(nx, ny), precision=ng.NG_FP32, stream=st)
    r = ng.Solver(GAS, nx, ny, W=start(nx, ny), precision=ng.NG_FP32)
    s.step(4)
    t = 0.9 * s.diagnostics()["t"] * 2
    s.run_to_time(t)
    st.synchronize()
    x = torch.zeros(4, device="cuda")
    g = torch.cuda.CUDAGraph()
    print("captured step", shape, flush=True)
    with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
        x.add_(1.0)
        for n in (1, 4):
            with pytest.raises(ng.NgError) as e:
                s.step(n)
            assert e.value.code == ng.NG_EDEVICE
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert x.tolist() == [3.0] * 4
    s.step(5)       # past the end time of run_to_time
    r.step(4)
    r.run_to_time(t)
    r.step(5)
    a, b = s.diagnostics(), r.diagnostics()
    assert a["t"] == b["t"] > t and a["steps"] == b["steps"]
    assert np.array_equal(s.conserved(), r.conserved())
    s.close()
    r.close()


@pytest.mark.parametrize("sizes", [((1000, 1), (1001, 1)), ((9000, 1),), ((9000, 1), (20000, 1)),
                                   ((150, 131), (90, 70))], ids=lambda v: f"{len(v)}x{v[0][0]}")
@pytest.mark.parametrize("n", [2, 16])
def test_batch_run_is_recorded(sizes, n):
    import torch
    from paper_1805_03442_amd import ng
    st = torch.cuda.Stream()
    print("captured batch", sizes, n, flush=True)
    out = []
    for graph in (True, False):
        b = ng.Batch(4, 64 << 20, precision=ng.NG_FP32, stream=st)
        slots = [b.add(GAS, nx, ny, start(nx, ny), 1e9) for nx, ny in sizes]
        b.run(n)
        b.poll()
        if graph:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
                b.run(n)
        seen = []
        for k in range(4):
            if graph:
                with torch.cuda.stream(st):
                    g.replay()
            else:
                b.run(n)
            b.run(1 + k)
            seen.append([(b.diagnostics(i)["steps"], b.diagnostics(i)["t"]) for i in slots])
        assert seen[-1][0][0] == 5 * n + 10
        out.append((seen, [b.conserved(i) for i in slots]))
        b.close()
    assert out[0][0] == out[1][0]
    for U, V in zip(out[0][1], out[1][1]):
        assert np.array_equal(U, V)


def test_a_recorded_launch_keeps_its_room():
    """The exchange of a cooperative launch in a graph is not given to solves that
    are added later: a replay before the next call leaves them as they are."""
    import torch
    from paper_1805_03442_amd import ng
    n = 9000
    need = ng.Batch.solve_bytes(n, 1, ng.NG_FP64)
    st = torch.cuda.Stream()
    b = ng.Batch(9, 7 * need + need // 2, precision=ng.NG_FP64, stream=st)
    slots = [b.add(GAS, n, 1, start(n), 1e9)]
    b.run(20)
    b.poll()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st, capture_error_mode="thread_local"):
        b.run(20)
    while True:
        k = b.add(GAS, n, 1, start(n), 1e9)
        if k is None:
            break
        slots.append(k)
    assert len(slots) >= 3
    print("replay beside", len(slots), "solves", flush=True)
    before = [b.conserved(i) for i in slots[1:]]
    with torch.cuda.stream(st):
        for _ in range(3):
            g.replay()
    assert b.diagnostics(slots[0])["steps"] == 80
    assert all(np.array_equal(U, b.conserved(i)) for U, i in zip(before, slots[1:]))
    b.run(20)
    r = ng.Solver(GAS, n, 1, W=start(n), precision=ng.NG_FP64)
    r.step(20)
    assert all(np.array_equal(r.conserved(), b.conserved(i)) for i in slots[1:])
    r.step(80)
    assert np.array_equal(r.conserved(), b.conserved(slots[0]))
    r.close()
    b.close()
