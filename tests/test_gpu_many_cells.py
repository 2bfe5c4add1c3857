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


# 84^3 cells have 8104 blocks of 1024 task counts, 86^3 have 8697: above 8192 the sums of
# the blocks are scanned on their own.  A wrong offset shows in the sweep.
@pytest.mark.parametrize("side", [84, 86])
def test_schedule_of_many_cells(side):
    from paper_1707_04232_amd import sdpd
    n, box = 20011, (2.5 * side,) * 3
    say("schedule of many cells", side)
    q, p, eps, ids = uniform_state(n, box, seed=6)
    q = np.array(q).reshape(3, n)
    q[:, ::2] = np.array([[1.0], [40.0], [170.0]]) + 30.0 * (q[:, ::2] / box[0])   # dense
    kw = dict(n=n, box=box, dt=0.002, Cv=10.0, seed=11, ncell=(side,) * 3)
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(**kw)) as ctx:
        ctx.prepare(S)
        stats = ctx.fd_metropolis(S, step=5)
    kw.pop("ncell")
    P = O.OracleParams(**kw)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    PU.sweep_and_compare(P, R, 5, S.to_numpy(), stats, 1e-10, say)


def test_cells_beyond_the_first_scan():
    """204^3 cells: 8291 blocks of cell counts (and two levels above them)."""
    from paper_1707_04232_amd import sdpd
    side, n = 204, 50021
    say("cell list of many cells")
    q, p, eps, ids = uniform_state(n, (2.5 * side,) * 3, seed=8)
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(n=n, box=2.5 * side, ncell=(side,) * 3,
                                      fd=sdpd.FD_NONE)) as ctx:
        for _ in range(2):   # (the second build counts from what the first one left)
            ctx.build_cells(S)
        start = ctx.cell_start()
    x = np.minimum(np.floor(np.array(q).reshape(3, n) * (side / (2.5 * side))), side - 1)
    cell = (x[0] + side * (x[1] + side * x[2])).astype(np.int64)
    want = np.concatenate([[0], np.cumsum(np.bincount(cell, minlength=side ** 3))])
    assert np.array_equal(start, want)
