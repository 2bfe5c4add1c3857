"""Device memory of a context, and a context made where the device has no room for what
only saves time."""
import numpy as np
import pytest

from paper_1707_04232_amd.workload import lattice_state

pytestmark = pytest.mark.gpu


def used_by(make):
    import torch
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    ctx = make()
    return ctx, free - torch.cuda.mem_get_info()[0]


def warm():
    from paper_1707_04232_amd import sdpd
    sdpd.Context(sdpd.SdpdParams(n=8, box=10.0)).close()   # the library's code is loaded


def test_memory_per_particle():
    """2^20 particles: with the sweep in one launch 512 B of pair entries, 108 of list
    positions, 112 of masks, 768 of partner lists and about 150 of state copies and
    indices per particle, and the sweep's record slices (3072 workgroups of up to 20 KB
    of entries, 16 times as many bytes): below 2.2 KB; without a sweep, with lists for
    full cells (1152 B), below 1.5 KB.
    Launches per group take 2 KB more when they are asked for."""
    from paper_1707_04232_amd import sdpd
    print("[case] memory per particle", flush=True)
    warm()
    n, box = 1 << 20, (128.0, 128.0, 64.0)
    ctx, used = used_by(lambda: sdpd.Context(sdpd.SdpdParams(n=n, box=box)))
    assert ctx.sweep_mode()[1] == sdpd.SWEEP_ONE
    assert used <= 2200 * n, used / n
    _, more = used_by(lambda: ctx.set_sweep_mode(sdpd.SWEEP_PER_GROUP))
    assert 0 < more <= 2100 * n, more / n
    ctx.close()
    ctx, used = used_by(lambda: sdpd.Context(sdpd.SdpdParams(n=n, box=box, fd=sdpd.FD_NONE)))
    assert used <= 1500 * n, used / n
    ctx.close()


def fill_device(room):
    """Blocks that leave about `room` bytes of the device (as the allocator has them: it
    hands out more than it reports free)."""
    import torch
    blocks = []
    for size in (4 << 30, 24 << 20):
        try:
            while True:
                blocks.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            pass
    while room > 0:
        room -= blocks.pop().numel()
        assert blocks and blocks[-1].numel() == 24 << 20
    torch.cuda.empty_cache()
    return blocks


# what may be missing per particle: the lists and, for the small box, half of its records
@pytest.mark.parametrize("side,prec,spare", [(24, 0, 2560), (64, 0, 512), (64, 1, 512)])
def test_context_without_room_for_lists(side, prec, spare):
    """Steps of a context made beside a filler that leaves it too little for its lists:
    the same pairs, draws and masks; the sums over partners in another order."""
    import torch
    from paper_1707_04232_amd import sdpd
    print("[case] little memory", side, prec, flush=True)
    q, p, eps, ids = lattice_state(side, jitter=0.2, Cv=10.0, T=1.0, seed=4)
    n = len(eps)
    prm = sdpd.SdpdParams(n=n, box=float(side), dt=0.002, seed=3, prec=prec)
    warm()
    outs, stats = [], []
    ctx, used = used_by(lambda: sdpd.Context(prm))
    for little in (False, True):
        if little:
            fill = fill_device(used - spare * n // 2 - (24 << 20))
            ctx, less = used_by(lambda: sdpd.Context(prm))
            del fill
            torch.cuda.empty_cache()
            assert less <= used - spare * n // 2, (less, used)
        S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
        ctx.prepare(S)
        stats.append(ctx.step(S, 0, 1))
        ctx.sync()
        ctx.close()
        outs.append(S.to_numpy())
    a, b = outs
    assert np.array_equal(a["id"], b["id"]) and np.array_equal(a["rho"], b["rho"])
    assert stats[0][0]["proposed"] == stats[1][0]["proposed"]
    if prec:   # (one order of the sums in both forms)
        assert np.array_equal(a["f"], b["f"]) and np.array_equal(a["p"], b["p"])
    else:
        assert np.abs(a["f"] - b["f"]).max() <= 1e-12 * np.abs(a["f"]).max()
