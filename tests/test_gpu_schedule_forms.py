"""The pair schedule on both sides of the 6144 cells from which tasks run on lanes,
with some cells of more than 32 particles (tasks on a whole wave there) and empty
ones.  A wrong list, order or level shows in the sweep: against the oracle its
tolerance of the other parity tests holds (1e-10, identical counters)."""
import numpy as np
import pytest

import oracle as O
import parity_util as PU
from paper_1707_04232_amd.workload import uniform_state

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


# 18 x 18 x 18 = 5832 and 18 x 18 x 20 = 6480 cells of edge 2.5
@pytest.mark.parametrize("box", [(45.0, 45.0, 45.0), (45.0, 45.0, 50.0)])
def test_schedule_forms(box):
    from paper_1707_04232_amd import sdpd
    n = 20011
    say("schedule", box)
    q, p, eps, ids = uniform_state(n, box, seed=5)
    q = np.array(q).reshape(3, n)
    rng = np.random.default_rng(2)
    for k, cell in enumerate([(0, 0, 0), (17, 3, 9), (8, 8, 8), (9, 8, 8)]):   # 40 more each
        at = slice(40 * k, 40 * (k + 1))
        q[:, at] = 2.5 * (np.array(cell, dtype=float)[:, None] + rng.uniform(size=(3, 40)))
    q[:, 200:600] = rng.uniform(size=(3, 400)) * 2.5 * np.array([[2.0], [18.0], [18.0]])
    edges = [np.linspace(0.0, b, int(b / 2.5) + 1) for b in box]
    count = np.histogramdd(q.T, bins=edges)[0]
    assert 32 < count.max() <= 64 and count.min() == 0
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(n=n, box=box, dt=0.002, Cv=10.0, seed=11)) as ctx:
        ctx.prepare(S)
        stats = ctx.fd_metropolis(S, step=5)
        ctx.sync()
    P = O.OracleParams(n=n, box=box, dt=0.002, Cv=10.0, seed=11)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    PU.sweep_and_compare(P, R, 5, S.to_numpy(), stats, 1e-10, say)
