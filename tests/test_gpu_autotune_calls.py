"""The autotuner's functions as a program calls them: a schedule timed on device
descriptors, and a class tuned on the batch that it is given."""
import inspect

import numpy as np
import pytest

from gpu_util import BETA_STAR, SEED, say
from paper_1701_03549_amd import synth


def test_arguments():
    from paper_1701_03549_amd import autotune
    assert list(inspect.signature(autotune.time_schedule).parameters) == \
        ["g", "sched", "d_beta", "d_sims", "n", "seed", "out", "reps"]
    assert list(inspect.signature(autotune.tune).parameters)[:6] == ["g", "lid", "sims", "betas", "seed", "log"]


@pytest.mark.gpu
def test_time_schedule_runs_the_batch():
    import torch
    from paper_1701_03549_amd import autotune, fire
    say("autotuner: one schedule on device descriptors")
    g = fire.FireGPU(0)
    try:
        ls = synth.make_landscape(64, 64, 101)
        lid = g.load_landscape(ls)
        sims = fire.make_sims(40, lid, -1, synth.ignition_site(ls))
        d_sims = torch.from_numpy(sims.view(np.uint8).copy()).cuda()
        d_beta = torch.tensor([BETA_STAR], dtype=torch.float64).cuda()
        out = torch.zeros((40, 24), dtype=torch.uint8, device="cuda")
        sched = dict(threads=64, queue_cap=256, table_mode=1, wg_per_cu=2)
        for s in (None, sched):
            assert autotune.time_schedule(g, s, d_beta, d_sims, 40, SEED, out, reps=2) > 0.0
        want, _ = g.run(np.array([BETA_STAR]), sims, SEED)
        g.sync()
        assert torch.equal(out, want)
    finally:
        g.close()
