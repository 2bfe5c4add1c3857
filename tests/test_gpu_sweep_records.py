"""The forms of the fluctuation/dissipation sweep against one another and the
oracle: one launch (records formed in the ranges, two waves per SIMD), one
launch per group with the records of the whole sweep formed first (boxes of at
most 2^14 particles) and with the records formed in the launches (larger
boxes).  A pair's update does the same operations on the same values in all of
them, so they agree bit for bit; against the oracle the sweep's tolerance of
the other parity tests holds (1e-10, identical counters)."""
import numpy as np
import pytest

import oracle as O
import parity_util as PU
from paper_1707_04232_amd.workload import lattice_state

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


# around the 2^14 particles up to which the records have a launch of their own
@pytest.mark.parametrize("dims", [(25, 25, 26), (26, 26, 25)])
@pytest.mark.parametrize("scheme", ["ems", "ams_cubic", "ssa", "mixed"])
def test_sweep_forms_agree(dims, scheme):
    from paper_1707_04232_amd import sdpd
    say("sweep forms", dims, scheme)
    kw = {"ems": dict(Cv=1.5), "ams_cubic": dict(Cv=10.0, fd=1, kernel=1, zeta=0.4),
          "ssa": dict(Cv=40.0, fd=2), "mixed": dict(Cv=10.0, prec=1)}[scheme]
    q, p, eps, ids = lattice_state(dims, jitter=0.2, Cv=kw["Cv"], T=1.0, seed=3)
    box = tuple(float(d) for d in dims)
    outs, stats = [], []
    for mode in (sdpd.SWEEP_ONE, sdpd.SWEEP_PER_GROUP):
        S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
        with sdpd.Context(sdpd.SdpdParams(n=len(eps), box=box, dt=0.05, seed=11, **kw)) as ctx:
            ctx.set_sweep_mode(mode)
            ctx.prepare(S)
            stats.append(ctx.fd_metropolis(S, step=5))
        outs.append(S.to_numpy())
    assert stats[0] == stats[1]
    for k in ("p", "eps"):
        assert np.array_equal(outs[0][k], outs[1][k]), k
    if scheme == "mixed":
        return   # its tolerance against the oracle: the mixed-precision tests
    okw = dict(kw)
    P = O.OracleParams(n=len(eps), box=box, dt=0.05, seed=11, Cv=okw.pop("Cv"),
                       fd_mode=okw.pop("fd", 0), **okw)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    PU.sweep_and_compare(P, R, 5, outs[0], stats[0], 1e-10, say)
