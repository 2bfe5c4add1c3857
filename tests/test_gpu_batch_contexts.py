"""Contexts that belong to a batch, stepped on their own between its replays and after
it is gone: bit for bit what contexts give that never were in one.  Boxes on both sides
of the 2^14 particles up to which a sweep on its own forms all its records first, and of
the some 450 cells from which it is one launch, and a box tuned by its user."""
import numpy as np
import pytest

from paper_1707_04232_amd.workload import lattice_state

pytestmark = pytest.mark.gpu

SIDES = (10, 20, 25, 26)     # 64, 512, 1000 and 1000 cells
TUNED = 1                    # this one with ranges of its user's


@pytest.mark.parametrize("layout", ["fused", "flow", "graphs"])
@pytest.mark.parametrize("mode", ["auto", "per_group"])
def test_contexts_of_a_batch_step_on_their_own(layout, mode):
    import torch
    from paper_1707_04232_amd import sdpd
    print("[case] contexts of a batch", layout, mode, flush=True)
    want = {"fused": sdpd.BATCH_FUSED, "flow": sdpd.BATCH_FUSED_FLOW,
            "graphs": sdpd.BATCH_GRAPHS}[layout]

    def boxes():
        out = []
        for b, side in enumerate(SIDES):
            q, p, eps, ids = lattice_state(side, jitter=0.2, Cv=10.0, T=1.0, seed=b)
            S = sdpd.DeviceState.from_numpy(q, p, eps, ids)
            c = sdpd.Context(sdpd.SdpdParams(n=len(eps), box=float(side), dt=0.02, seed=7,
                                             replica=b), stream=torch.cuda.Stream())
            if b == TUNED:
                c.tune(fd_tasks=(2, 3, 5, 7), lds_particles=(-1,) * 4, lds_pairs=(-1,) * 4)
            if mode == "per_group":
                c.set_sweep_mode(sdpd.SWEEP_PER_GROUP)
            torch.cuda.synchronize()
            c.prepare(S)
            out.append((c, S))
        torch.cuda.synchronize()
        return out

    ref, bat = boxes(), boxes()
    tunings = [c.get_tuning() for c, _ in bat]
    in_use = [c.sweep_mode() for c, _ in bat]
    step = 0

    def same(what):
        for side, (cb, Sb), (cr, Sr) in zip(SIDES, bat, ref):
            cb.sync()
            cr.sync()
            x, y = Sb.to_numpy(), Sr.to_numpy()
            for k in ("id", "q", "p", "eps", "rho", "f"):
                assert np.array_equal(x[k], y[k]), f"{what}: {k} of the box of side {side}"

    def alone(what):
        nonlocal step
        for c, S in bat + ref:
            c.step(S, step, 1, stats=False)
        for (cb, Sb), (cr, Sr) in zip(bat, ref):
            assert cb.fd_metropolis(Sb, step + 100) == cr.fd_metropolis(Sr, step + 100), what
        step += 1
        same(what)

    B = sdpd.Batch([c for c, _ in bat], [S for _, S in bat], layout=want)
    alone("before the first replay")
    for rep in range(2):
        B.run(step, 2)
        for c, S in ref:
            c.step(S, step, 2, stats=False)
        step += 2
        same(f"replay {rep}")
        alone(f"after replay {rep}")
    B.close()
    alone("after the batch")
    assert [c.get_tuning() for c, _ in bat] == tunings
    assert [c.sweep_mode() for c, _ in bat] == in_use
    for c, _ in ref + bat:
        c.close()
