"""Boxes of few particles in many cells: what a context takes of the device's memory, and
the sweep with one launch per group on both sides of the 2^13 cells up to which a box of
at most 2^14 particles forms the records of a whole sweep first."""
import numpy as np
import pytest

import oracle as O
import parity_util as PU
from paper_1707_04232_amd.workload import uniform_state

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def test_memory_of_a_dilute_box():
    """64^3 cells: per cell at most 400 B (counts, offsets and order of the 14 tasks of a
    cell: 14 x 20 B, and the cell's own words) beside 8 KB per particle and 64 MB."""
    import torch
    from paper_1707_04232_amd import sdpd
    say("memory of a dilute box")
    n, cells = 1000, 64 ** 3
    sdpd.Context(sdpd.SdpdParams(n=8, box=10.0)).close()   # the library's code is loaded
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    with sdpd.Context(sdpd.SdpdParams(n=n, box=160.0)) as ctx:
        assert np.prod(ctx.cell_info()[0]) == cells
        used = free0 - torch.cuda.mem_get_info()[0]
    assert used <= 400 * cells + 8192 * n + (64 << 20), used


# 20 x 20 x 20 = 8000 and 20 x 20 x 22 = 8800 cells of edge 2.5
@pytest.mark.parametrize("box", [(50.0, 50.0, 50.0), (50.0, 50.0, 55.0)])
def test_sweep_of_a_dilute_box(box):
    from paper_1707_04232_amd import sdpd
    n = 6007
    say("sweep of a dilute box", box)
    q, p, eps, ids = uniform_state(n, box, seed=5)
    kw = dict(n=n, box=box, dt=0.002, Cv=10.0, seed=11)
    outs, stats = [], []
    for mode in (sdpd.SWEEP_PER_GROUP, sdpd.SWEEP_ONE):
        S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
        with sdpd.Context(sdpd.SdpdParams(**kw)) as ctx:
            ctx.set_sweep_mode(mode)
            ctx.prepare(S)
            stats.append(ctx.fd_metropolis(S, step=5))
        outs.append(S.to_numpy())
    assert stats[0] == stats[1]
    for k in ("p", "eps"):
        assert np.array_equal(outs[0][k], outs[1][k]), k
    P = O.OracleParams(**kw)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    PU.sweep_and_compare(P, R, 5, outs[0], stats[0], 1e-10, say)
