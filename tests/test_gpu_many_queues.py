"""The sweep of a box on its own in a process with eight hardware queues (their number
is fixed when HIP starts, so in a child process): one launch for a box that fills the GPU
by itself, one per group for one that does not, and the same results either way."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

CHILD = r"""
import os, sys
sys.path.insert(0, sys.argv[1])
import numpy as np, torch
from paper_1707_04232_amd import sdpd
from paper_1707_04232_amd.workload import lattice_state
# 16^3 = 4096 and 22^3 = 10648 cells
for side, layout in ((40, sdpd.SWEEP_PER_GROUP), (56, sdpd.SWEEP_ONE)):
    print("[case] eight queues, side", side, flush=True)
    q, p, eps, ids = lattice_state(side, jitter=0.2, Cv=10.0, T=1.0, seed=2)
    outs = []
    for mode in (sdpd.SWEEP_AUTO, sdpd.SWEEP_ONE, sdpd.SWEEP_PER_GROUP):
        S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
        with sdpd.Context(sdpd.SdpdParams(n=len(eps), box=float(side), dt=0.02, seed=5)) as c:
            c.set_sweep_mode(mode)
            assert mode != sdpd.SWEEP_AUTO or c.sweep_mode() == (mode, layout), c.sweep_mode()
            c.prepare(S)
            c.step(S, 0, 2, stats=False)
            c.sync()
        outs.append(S.to_numpy())
    for other in outs[1:]:
        for k in ("id", "q", "p", "eps", "rho", "f"):
            assert np.array_equal(outs[0][k], other[k]), (side, k)
print("ok", flush=True)
"""


def test_sweep_with_eight_queues():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    env = dict(os.environ, GPU_MAX_HW_QUEUES="8")
    print("[case] sweep with eight queues (child process)", flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD, root], env=env, cwd=root,
                       capture_output=True, text=True, timeout=110)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout[-2000:] + r.stderr[-2000:]
