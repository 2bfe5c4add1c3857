"""Dense regions of mostly empty boxes: particles whose partners fill both parts of their
lists (a droplet) or more (a cluster around a corner of eight cells, 56 in each, with
more partners than any list holds), with few cells (a workgroup per cell in the density
pass) and with many (2^15 and more of a dilute box).

FP64 against the oracle as in the other parity tests (1e-12 of the largest value).  FP32:
rho within 2e-5; a separation carries some 1e-6 of error (three times per axis the
rounding of a coordinate of up to a cell edge of 4), so the force is off by at most 2e-6
sum |m^2 (Pi_i + Pi_j) F| and, through its terms' own rounding and the error of rho in
Pi, 2.2e-5 sum |m^2 (Pi_i + Pi_j) F r|: a missing or doubled partner is a hundred times
that."""
import numpy as np
import pytest

import oracle as O
import parity_util as PU
from paper_1707_04232_amd.workload import uniform_state

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)


def droplet(box, side=10, h=3.6):
    """side^3 jittered particles at unit spacing, some 190 partners inside."""
    n = side ** 3
    q, p, eps, ids = uniform_state(n, (box,) * 3, seed=3)
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij")).reshape(3, n)
    jitter = 0.2 * (np.array(q).reshape(3, n) / box - 0.5)
    q = (g + jitter + np.array([[box / 2], [box - 5.0], [box / 2]])) % box   # across a face
    return q, np.array(p).reshape(3, n), eps, ids, dict(h=h)


def cluster(box, h=2.5):
    """Eight octants of 56 particles around a cell corner, and 300 more in the box."""
    n = 8 * 56 + 300
    q, p, eps, ids = uniform_state(n, (box,) * 3, seed=4)
    q = np.array(q).reshape(3, n)
    edge = box / (2 * int(box / h / 2))
    sign = np.array([[(o >> a) & 1 for a in range(3)] for o in range(8)]).T * 2 - 1
    inner = 0.05 + 1.2 * (q[:, :448] / box)
    q[:, :448] = (edge * np.array([[2], [0], [3]]) + np.repeat(sign, 56, axis=1) * inner) % box
    return q, np.array(p).reshape(3, n), eps, ids, dict(h=h)


# 36^3 and 32^3 = 2^15 cells; 12^3 (two workgroups a cell fewer) and 8^3
CASES = {"droplet_few_cells": lambda: droplet(44.0), "droplet_many_cells": lambda: droplet(130.0),
         "cluster_few_cells": lambda: cluster(20.0), "cluster_many_cells": lambda: cluster(80.0)}
BOX = {"droplet_few_cells": 44.0, "droplet_many_cells": 130.0, "cluster_few_cells": 20.0,
       "cluster_many_cells": 80.0}


def separations(q, box):
    d = q[:, :, None] - q[:, None, :]
    return d - box * np.rint(d / box)


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
def test_density_forces_and_masks(name, kernel, prec):
    from paper_1707_04232_amd import sdpd
    say("dense region", name, kernel, prec)
    (q, p, eps, ids, kw), box = CASES[name](), BOX[name]
    n, h = len(eps), kw["h"]
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(n=n, box=box, kernel=kernel, prec=prec, fd=sdpd.FD_AMS,
                                      dt=1e-5, **kw)) as ctx:
        cells = int(np.prod(ctx.cell_info()[0]))
        ctx.prepare(S)
        ctx.sync()
        G = S.to_numpy()
        try:   # (the masks: the pairs that a sweep proposes)
            proposed = ctx.fd_metropolis(S, step=0)["proposed"]
        except sdpd.SdpdError as e:
            assert e.rc == sdpd.ECAPACITY
            proposed = None
    assert (cells >= 1 << 15) == ("many" in name)
    P = O.OracleParams(n=n, box=(box,) * 3, kernel=kernel, **kw)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    assert np.array_equal(G["id"], R.id)
    r = np.sqrt((separations(R.q, box) ** 2).sum(axis=0))
    pairs = (r < h) & ~np.eye(n, dtype=bool)
    most = int(pairs.sum(axis=1).max()) + 1
    assert most > (320 if "cluster" in name else 128), most
    if proposed is not None and not prec:
        assert proposed == pairs.sum() // 2
    assert np.abs(G["rho"] - R.rho).max() <= (2e-5 if prec else 1e-12) * R.rho.max()
    if not prec:
        assert np.abs(G["f"] - R.f).max() <= 1e-12 * np.abs(R.f).max()
        return
    x = r / h
    if kernel == 0:
        F = 315.0 / (4 * np.pi * h ** 5) * (1 - x) ** 2
    else:
        F = 48.0 / (np.pi * h ** 5) * np.where(x <= 0.5, 2 - 3 * x,
                                               (1 - x) ** 2 / np.maximum(x, 0.5))
    Pi = (P.Cv / (3 * P.kB)) * P.kB * R.eps / (P.m * P.Cv) / R.rho
    sc = np.where(pairs, P.m ** 2 * (Pi[:, None] + Pi[None, :]) * F, 0.0)
    bound = 2e-6 * sc.sum(axis=1) + 2.2e-5 * (sc * r).sum(axis=1)
    worst = (np.abs(G["f"] - R.f) / np.maximum(bound, 1e-300)).max()
    say(f"error over its bound {worst:.3f}, most partners {most}")
    assert worst <= 1.0


def droplet_in_vapour():
    """36^3 cells with 0.6 particles on average, 16 in those of a droplet across a corner
    of the box: empty and thin cells beside dense ones, on all sides."""
    side, box = 12, 90.0
    n = side ** 3 + 28001
    q, p, eps, ids = uniform_state(n, (box,) * 3, seed=9)
    q, k = np.array(q).reshape(3, n), side ** 3
    g = np.stack(np.meshgrid(*[np.arange(side)] * 3, indexing="ij")).reshape(3, k)
    q[:, ::-1][:, :k] = (g - 5.3 + 0.3 * (q[:, :k] / box)) % box
    return q, p, eps, ids, box


@pytest.mark.parametrize("kernel", [0, 1])
def test_sweep_of_a_droplet_in_vapour(kernel):
    from paper_1707_04232_amd import sdpd
    say("sweep of a droplet in vapour", kernel)
    q, p, eps, ids, box = droplet_in_vapour()
    kw = dict(n=len(eps), dt=0.002, Cv=10.0, seed=11, kernel=kernel)
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(box=box, **kw)) as ctx:
        ctx.prepare(S)
        f = S.to_numpy()["f"]
        stats = ctx.fd_metropolis(S, step=5)
    P = O.OracleParams(box=(box,) * 3, **kw)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    assert np.abs(S.to_numpy()["rho"] - R.rho).max() <= 1e-12 * R.rho.max()
    assert np.abs(f - R.f).max() <= 1e-12 * np.abs(R.f).max()
    PU.sweep_and_compare(P, R, 5, S.to_numpy(), stats, 1e-10, say)


def test_mixed_droplet_in_vapour():
    """FP32: rho as above; the forces within 2e-4 of the largest possible term of a pair,
    as in the other mixed-precision tests; after a step those of a box stepped eagerly and
    in a batch agree bit for bit."""
    import torch
    from paper_1707_04232_amd import sdpd
    say("mixed droplet in vapour")
    q, p, eps, ids, box = droplet_in_vapour()
    n = len(eps)
    P = O.OracleParams(n=n, box=(box,) * 3, Cv=10.0)
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(P, R)
    outs = []
    for batch in (False, True):
        S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
        ctx = sdpd.Context(sdpd.SdpdParams(n=n, box=box, Cv=10.0, prec=1, dt=0.002, seed=3),
                           stream=torch.cuda.Stream())
        torch.cuda.synchronize()
        ctx.prepare(S)
        ctx.sync()
        G = S.to_numpy()
        assert np.array_equal(G["id"], R.id)
        assert np.abs(G["rho"] - R.rho).max() <= 2e-5 * R.rho.max()
        Pi = (P.Cv / (3 * P.kB)) * P.kB * R.eps / (P.m * P.Cv) / R.rho
        term = P.m ** 2 * 2 * Pi.max() * 315.0 / (4 * np.pi * P.h ** 4) * 4.0 / 27.0
        assert np.abs(G["f"] - R.f).max() <= 2e-4 * term
        if batch:
            B = sdpd.Batch([ctx], [S], layout=sdpd.BATCH_FUSED)
            B.run(0, 2)
            torch.cuda.synchronize()
            B.close()
        else:
            ctx.step(S, 0, 2, stats=False)
        ctx.sync()
        outs.append(S.to_numpy())
        ctx.close()
    for k in ("id", "q", "p", "eps", "rho", "f"):
        assert np.array_equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("kernel", [0, 1])
@pytest.mark.parametrize("name", ["droplet_few_cells", "cluster_few_cells"])
def test_gradient(name, kernel):
    """Directional derivative against central differences of the oracle's forward, with
    the bar of the other gradient tests (1e-6)."""
    import torch
    from paper_1707_04232_amd import sdpd
    say("gradient of a dense region", name, kernel)
    (q, p, eps, ids, kw), box = CASES[name](), BOX[name]
    n, K = len(eps), 3
    kw = dict(kw, Cv=10.0, dt=1e-3, kernel=kernel)
    rng = np.random.default_rng(5)
    a, b = rng.normal(size=(3, n)), rng.normal(size=(3, n))

    def J(x):
        P = O.OracleParams(n=n, box=(box,) * 3, fd_mode=O.FD_NONE, **kw)
        S = O.State.from_arrays(x, p, eps, ids)
        O.prepare(P, S)
        assert O.step(P, S, 0, K)[0] == 0
        return float((a[:, S.id] * S.q).sum() + (b[:, S.id] * S.p).sum())

    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(n=n, box=box, fd=sdpd.FD_NONE, **kw)) as ctx:
        ctx.prepare(S)
        ctx.adjoint_forward(S, K, 2)
        g = ctx.adjoint_backward(torch.as_tensor(a, device="cuda"),
                                 torch.as_tensor(b, device="cuda"))
        ctx.sync()
    d = rng.normal(size=(3, n))
    delta = 1e-6
    fd = (J(q + delta * d) - J(q - delta * d)) / (2 * delta)
    ad = float((g[0].cpu().numpy() * d).sum())
    say(f"adjoint {ad:.10e} central differences {fd:.10e}")
    assert abs(ad - fd) <= 1e-6 * max(abs(fd), 1e-3)


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_of_dilute_boxes(prec):
    """The multi-box forms of the passes of dilute boxes: bit for bit the eager steps."""
    import torch
    from paper_1707_04232_amd import sdpd
    say("batch of dilute boxes", prec)
    outs = []
    for batch in (False, True):
        ctxs, states = [], []
        for b, name in enumerate(["droplet_many_cells", "cluster_many_cells"]):
            (q, p, eps, ids, kw), box = CASES[name](), BOX[name]
            for kernel in (0, 1):
                states.append(sdpd.DeviceState.from_numpy(q, p, eps, ids))
                ctxs.append(sdpd.Context(sdpd.SdpdParams(
                    n=len(eps), box=box, kernel=kernel, prec=prec, fd=sdpd.FD_NONE, dt=1e-4,
                    replica=b, **kw), stream=torch.cuda.Stream()))
                torch.cuda.synchronize()
                ctxs[-1].prepare(states[-1])
        torch.cuda.synchronize()
        if batch:
            B = sdpd.Batch(ctxs, states, layout=sdpd.BATCH_FUSED)
            B.run(0, 2)
            torch.cuda.synchronize()
            B.run(2, 2)
            torch.cuda.synchronize()
            B.close()
        else:
            for c, S in zip(ctxs, states):
                c.step(S, 0, 4, stats=False)
        for c in ctxs:
            c.sync()
        outs.append([S.to_numpy() for S in states])
        for c in ctxs:
            c.close()
    for x, y in zip(*outs):
        for k in ("id", "q", "p", "eps", "rho", "f"):
            assert np.array_equal(x[k], y[k]), k
