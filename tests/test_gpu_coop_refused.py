"""GPU: solves in a process whose cooperative launches the runtime refuses (the
device's cooperative queue belongs to one process at a time, here to the test's
own) run on the other paths, with the same results."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1805_03442_amd import workloads as wl

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import numpy as np
from paper_1805_03442_amd import ng, workloads as wl
gas = dict(wl.BASE_GAS, Q_T=2.0)

def start(nx, ny):
    W = wl.uniform_state(gas, nx, ny)
    W[0] += 1e-2 * np.sin(2 * np.pi * (np.arange(nx) + 0.5) / nx)[None, :]
    return W

for nx, ny in ((3000, 1), (150, 131)):
    print("second process", nx, ny, flush=True)
    out = []
    for coop in (-1, 0):
        s = ng.Solver(gas, nx, ny, W=start(nx, ny), precision=ng.NG_FP64)
        s.set_coop(coop)
        if ny == 1:
            s.enable_timing(5)
            s.step(5)
            s.enable_timing(0)
        s.step(2)
        s.step(70)
        s.step(5)
        s.run_to_time(s.diagnostics()["t"] * 1.2)
        d = s.diagnostics()
        out.append((d["t"], d["steps"], d["status"], s.conserved()))
        s.close()
    assert out[0][:3] == out[1][:3] and out[0][2] == 0
    assert np.array_equal(out[0][3], out[1][3])
print("second process batch", flush=True)
out = []
for coop in (-1, 0):
    b = ng.Batch(5, 64 << 20, precision=ng.NG_FP32)
    b.set_coop(coop)
    slots = [b.add(gas, nx, ny, start(nx, ny), 1e9) for nx, ny in ((300, 1), (9000, 1), (2000, 1), (90, 70))]
    for n in (30, 4, 1, 30):
        b.run(n)
    out.append([(b.diagnostics(i)["t"], b.diagnostics(i)["steps"], b.conserved(i)) for i in slots])
    b.close()
for (t, n, U), (u, m, V) in zip(*out):
    assert t == u and n == m == 65 and np.array_equal(U, V)
print("second process ok", flush=True)
"""


def test_a_second_process_runs_on():
    from paper_1805_03442_amd import ng
    gas = dict(wl.BASE_GAS, Q_T=2.0)
    s = ng.Solver(gas, 1000, 1, W=wl.uniform_state(gas, 1000), precision=ng.NG_FP64)
    s.step(10)      # a cooperative launch: the queue is this process's
    assert s.diagnostics()["steps"] == 10
    print("first process runs cooperatively", flush=True)
    r = subprocess.run([sys.executable, "-u", "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100)
    print(r.stdout[-2000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0 and "second process ok" in r.stdout
    s.step(10)
    assert s.diagnostics()["steps"] == 20 and np.isfinite(s.conserved()).all()
    s.close()
