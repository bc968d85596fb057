"""Batches over several large landscapes: the wide window that one of them has
earned alone is taken, and given up after a call in which more than a quarter of
the fires left it. Seen from the simulations in flight: a lattice over half of
the LDS has one whole-lattice workgroup per compute unit, the wide window three."""
import numpy as np
import pytest

from gpu_util import SEED, say
from paper_1701_03549_amd import synth

pytestmark = pytest.mark.gpu


def _in_flight(times):
    t = times.cpu().numpy()
    ends = np.concatenate([np.stack([t[:, 0], np.ones(len(t), np.int64)], 1),
                           np.stack([t[:, 1], -np.ones(len(t), np.int64)], 1)])
    ends = ends[np.lexsort((ends[:, 1], ends[:, 0]))]  # a finish before a take at the same tick
    return int(np.cumsum(ends[:, 1]).max())


@pytest.mark.parametrize("host", [True, False])
@pytest.mark.parametrize("leaving", [8, 2])
def test_wide_window_over_several_landscapes(host, leaving):
    """One fire in `leaving` crosses its lattice, the others stay small."""
    import torch
    from paper_1701_03549_amd import fire
    W, H, n = 1000, 930, 1600
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ctx = fire.FireGPU(0)
    try:
        ls = synth.make_landscape(W, H, 103)
        c = synth.ignition_site(ls)
        lid = ctx.load_landscape(ls)
        sims = fire.make_sims(n, lid, -1, c)
        sims["max_steps"][np.arange(n) % leaving != 0] = 60
        beta = np.array([[-0.2, 0.0, 0.0, 0.0, 0.0]])
        say(f"several large landscapes, host {host}, one in {leaving} leaving: one landscape alone")
        ctx.run(beta, sims[:800], SEED)  # its small window is repeated
        ctx.sync()
        assert ctx.get_schedule(W * H, 1, n)["window"] > 600  # the wide window is next
        sims["landscape_id"][n // 2:] = ctx.load_landscape(ls)
        d_sims = torch.from_numpy(sims.view(np.uint8).copy()).cuda()
        d_beta = torch.from_numpy(beta).cuda()
        times = torch.zeros((n, 2), dtype=torch.int64, device="cuda")
        ctx.set_sim_timing(times)
        outs, flight = [], []
        for k in range(3):
            say(f"several large landscapes, host {host}, one in {leaving} leaving: both, run {k}")
            if host:
                out, _ = ctx.run(beta, sims, SEED)
            else:
                out = torch.empty((n, 24), dtype=torch.uint8, device="cuda")
                ctx.run_dev(d_beta, d_sims, n, SEED, out)
            ctx.sync()
            outs.append(out)
            flight.append(_in_flight(times))
        ctx.set_sim_timing(None)
        assert flight[0] > cus
        if leaving == 2:
            assert flight[1] <= cus and flight[2] <= cus
            assert ctx.get_schedule(W * H, 1, n)["window"] == 0
        else:
            assert flight[1] > cus and flight[2] > cus
        ctx.set_schedule(512, 1024, 0, 1, window=0)
        want, _ = ctx.run(beta, sims, SEED)
        ctx.sync()
        for out in outs:
            assert torch.equal(out, want)
    finally:
        ctx.close()
