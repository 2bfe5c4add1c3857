"""Gradient where a third of the particles have more partners than the lists of the
density pass hold (they are looked up among their candidates), and of a context whose
buffers serve several passes.  Directional derivatives against central differences of
the oracle's forward with the bar of the other gradient tests (1e-6); passes that
take over the buffers of a longer or an equal one repeat bit for bit."""
import numpy as np
import pytest

import oracle as O
from paper_1707_04232_amd.workload import uniform_state

pytestmark = pytest.mark.gpu


def cluster(n=900, box=20.0):
    q, p, eps, ids = uniform_state(n, (box,) * 3, seed=7)
    rng = np.random.default_rng(3)
    d = rng.normal(size=(3, n // 3))
    d *= 1.6 * rng.uniform(size=n // 3) ** (1 / 3) / np.linalg.norm(d, axis=0)
    q = np.array(q).reshape(3, n)
    q[:, ::3] = (d + np.array([[10.0], [20.0], [5.0]])) % box
    return q, np.array(p).reshape(3, n), eps, np.arange(n)


@pytest.mark.parametrize("kernel", [0, 1])
def test_gradient_beyond_the_lists(kernel):
    import torch
    from paper_1707_04232_amd import sdpd
    print("[case] gradient of a cluster, kernel", kernel, flush=True)
    q, p, eps, ids = cluster()
    n, box, K, kw = len(eps), 20.0, 3, dict(Cv=10.0, dt=1e-3, kernel=kernel)
    rng = np.random.default_rng(5)
    a, b = rng.normal(size=(3, n)), rng.normal(size=(3, n))

    def J(x):
        P = O.OracleParams(n=n, box=(box,) * 3, fd_mode=O.FD_NONE, **kw)
        S = O.State.from_arrays(x, p, eps, ids)
        O.prepare(P, S)
        assert O.step(P, S, 0, K)[0] == 0
        return float((a[:, S.id] * S.q).sum() + (b[:, S.id] * S.p).sum())

    def gradient(ctx, k):
        S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
        ctx.prepare(S)
        ctx.adjoint_forward(S, k, 2)
        g = ctx.adjoint_backward(torch.as_tensor(a, device="cuda"),
                                 torch.as_tensor(b, device="cuda"))
        ctx.sync()
        return [x.cpu().numpy() for x in g[:3]] + [g[3]]

    with sdpd.Context(sdpd.SdpdParams(n=n, box=box, fd=sdpd.FD_NONE, **kw)) as ctx:
        first = gradient(ctx, K)
        gradient(ctx, K + 1)                      # more buffers than the first pass
        again = [gradient(ctx, K) for _ in range(2)]
    for g in again:
        for x, y in zip(first, g):
            assert np.array_equal(x, y)
    d = rng.normal(size=(3, n))
    delta = 1e-6
    fd = (J(q + delta * d) - J(q - delta * d)) / (2 * delta)
    ad = float((first[0] * d).sum())
    print(f"adjoint {ad:.10e} central differences {fd:.10e}", flush=True)
    assert abs(ad - fd) <= 1e-6 * max(abs(fd), 1e-3)
