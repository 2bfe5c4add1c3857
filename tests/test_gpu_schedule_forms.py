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


# 4096 cells each: the schedule of one box runs in rounds, that of a launch shared by
# both (8192 cells) with tasks on lanes; with a part for each box both run in rounds
@pytest.mark.parametrize("parts", [1, 2])
def test_batch_schedule_equals_eager(parts):
    import torch
    from paper_1707_04232_amd import sdpd
    from paper_1707_04232_amd.workload import lattice_state
    say("batch schedule, parts", parts)
    outs = []
    for batch in (False, True):
        ctxs, states = [], []
        for b in range(2):
            q, p, eps, ids = lattice_state(40, jitter=0.2, Cv=10.0, T=1.0, seed=b)
            states.append(sdpd.DeviceState.from_numpy(q, p, eps, ids))
            ctxs.append(sdpd.Context(sdpd.SdpdParams(n=len(eps), box=40.0, seed=9, replica=b),
                                     stream=torch.cuda.Stream()))
            ctxs[-1].prepare(states[-1])
        torch.cuda.synchronize()
        if batch:
            B = sdpd.Batch(ctxs, states, layout=sdpd.BATCH_FUSED, parts=parts)
            B.run(0, 3)
            torch.cuda.synchronize()
            B.close()
        else:
            for c, S in zip(ctxs, states):
                c.step(S, 0, 3, stats=False)
        for c in ctxs:
            c.sync()
        outs.append([S.to_numpy() for S in states])
        for c in ctxs:
            c.close()
    for x, y in zip(*outs):
        for k in ("id", "q", "p", "eps", "rho", "f"):
            assert np.array_equal(x[k], y[k]), k
