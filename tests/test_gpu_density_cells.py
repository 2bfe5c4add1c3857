"""Density, masks, lists and forces at the edges of the cell-wise passes: few cells
(a workgroup per cell), many (a wave per cell), many nearly empty ones (a lane per
particle), empty cells, cells of more than 32 particles (two mask words) and nearly
full ones, and particles with more partners than their lists hold.  The forces are
sums over the lists, so a wrong entry shows in them.  FP64 against the oracle as in the
other parity tests (1e-12 of the largest value); mixed precision rho within 2e-5 (FP32
separations, see the tests there)."""
import numpy as np
import pytest

import oracle as O
from paper_1707_04232_amd.workload import uniform_state

pytestmark = pytest.mark.gpu

# (particles, box): cells of edge 2.5 = h, 1024 and 1152 of them (the former is
# the largest box with a workgroup per cell), dilute or with 36 particles a cell
BOXES = {
    "dilute_1024_cells": (3001, (20.0, 20.0, 40.0)),
    "dilute_1152_cells": (3001, (20.0, 20.0, 45.0)),
    "dense_64_cells": (2450, (10.0, 10.0, 10.0)),
    "dense_1152_cells": (41003, (20.0, 20.0, 45.0)),
    # 34^3 cells: a lane per particle
    "sparse_39304_cells": (20011, (85.0, 85.0, 85.0)),
    "few_particles": (5, (10.0, 15.0, 10.0)),
    # a third of the particles within 1.6 of a cell corner: more partners than the
    # lists of the density pass, sized for the mean density, hold
    "cluster": (900, (20.0, 20.0, 20.0)),
}


@pytest.mark.parametrize("name", list(BOXES))
@pytest.mark.parametrize("form", ["lucy", "cubic", "mixed"])
def test_cell_edges(name, form):
    from paper_1707_04232_amd import sdpd
    n, box = BOXES[name]
    print("[case]", name, form, flush=True)
    q, p, eps, ids = uniform_state(n, box, seed=7)
    if name == "cluster":
        rng = np.random.default_rng(3)
        d = rng.normal(size=(3, 300))
        d *= 1.6 * rng.uniform(size=300) ** (1 / 3) / np.linalg.norm(d, axis=0)
        q = np.array(q).reshape(3, n)
        q[:, ::3] = (d + np.array([[10.0], [20.0], [5.0]])) % 20.0
    edges = [np.linspace(0.0, b, int(round(b / 2.5)) + 1) for b in box]
    full = int(np.histogramdd(np.asarray(q).reshape(3, n).T, bins=edges)[0].max())
    assert full <= 64 and (full > 48 or not name.startswith("dense"))
    kernel = 1 if form == "cubic" else 0
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(n=n, box=box, kernel=kernel,
                                      prec=1 if form == "mixed" else 0)) as ctx:
        ctx.prepare(S)
        ctx.sync()
    R = O.State.from_arrays(q, p, eps, ids)
    O.prepare(O.OracleParams(n=n, box=box, kernel=kernel), R)
    G = S.to_numpy()
    assert np.array_equal(G["id"], R.id)
    assert np.abs(G["rho"] - R.rho).max() <= (2e-5 if form == "mixed" else 1e-12) * R.rho.max()
    if form != "mixed":
        assert np.abs(G["f"] - R.f).max() <= 1e-12 * max(np.abs(R.f).max(), 1e-300)


@pytest.mark.parametrize("edge", [25.0, 2000.0])
def test_wide_cells_keep_pairs_at_the_cutoff(edge):
    """Cells far wider than h (the caller's choice of the grid): pairs a relative 1e-9
    to 1e-4 inside the cutoff, in all directions and across cells and the boundary, are
    all proposed by a sweep, and pairs as far outside are not."""
    from paper_1707_04232_amd import sdpd
    print("[case] wide cells", edge, flush=True)
    h, L, m = 2.5, 4 * edge, 120
    rng = np.random.default_rng(11)
    a = rng.uniform(0.0, L, size=(3, m))
    a[:, ::4] = edge * rng.integers(0, 4, size=(3, m // 4)) + rng.uniform(-1.0, 1.0, (3, m // 4))
    d = rng.normal(size=(3, m))
    d /= np.linalg.norm(d, axis=0)
    off = 10.0 ** rng.uniform(-9, -4, m) * np.where(np.arange(m) % 3 == 0, 1.0, -1.0)
    q = np.concatenate([a % L, (a + h * (1.0 + off) * d) % L], axis=1)
    n = 2 * m
    dist = [q[k][:, None] - q[k][None, :] for k in range(3)]
    r2 = sum((x - L * np.rint(x / L)) ** 2 for x in dist)
    inside = int(np.count_nonzero(np.triu(r2 < h * h, 1)))
    assert inside >= m // 2
    p, eps, ids = np.zeros((3, n)), np.ones(n), np.arange(n, dtype=np.uint32)
    S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
    with sdpd.Context(sdpd.SdpdParams(n=n, box=L, h=h, ncell=(4, 4, 4), dt=1e-6)) as ctx:
        ctx.prepare(S)
        stats = ctx.fd_metropolis(S, step=0)
    assert stats["proposed"] == inside
