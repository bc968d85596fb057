"""Replicate batches on lattices whose bitset takes more than half of the LDS:
the wide window that follows the first repeats and the whole-lattice runs that
follow it give the same results, through both entry points; and replicate
batches over several landscapes in one call equal one call per landscape."""
import numpy as np
import pytest

from gpu_util import SEED, say
from paper_1701_03549_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("turn_off", [False, True])
@pytest.mark.parametrize("host", [True, False])
@pytest.mark.parametrize("intercept", [-0.2, 6.0])
def test_wide_window_equals_whole_lattice(turn_off, host, intercept):
    import torch
    from paper_1701_03549_amd import fire
    W, H, n = 1000, 930, 800
    ctx = fire.FireGPU(0)
    try:
        ls = synth.make_landscape(W, H, 103)
        c = synth.ignition_site(ls)
        lid = ctx.load_landscape(ls)
        if turn_off:
            ctx.set_burn_steps(lid, np.full(256, 2, dtype=np.uint8))
        sims = fire.make_sims(n, lid, -1, c)
        sims["max_steps"][::3] = 290  # fires that stay within the wide window
        beta = np.array([[intercept, 0.0, 0.0, 0.0, 0.0]])
        d_sims = torch.from_numpy(sims.view(np.uint8).copy()).cuda()
        d_beta = torch.from_numpy(beta).cuda()

        def once():
            if host:
                out, _ = ctx.run(beta, sims, SEED)
            else:
                out = torch.empty((n, 24), dtype=torch.uint8, device="cuda")
                ctx.run_dev(d_beta, d_sims, n, SEED, out)
            ctx.sync()
            return out

        outs, windows = [], []
        for k in range(3):
            say(f"wide window, host {host}, turn-off {turn_off}, intercept {intercept}, run {k}")
            windows.append(ctx.get_schedule(W * H, 1, n)["window"])
            outs.append(once())
        # the small window, then the wide one, which most of these fires leave
        assert 0 < windows[0] < windows[1] and windows[2] == 0
        ctx.set_schedule(512, 1024, 1, 1, window=0)
        want = once()
        for o in outs:
            assert torch.equal(o, want)
        assert fire.results_to_numpy(want)["burnt"].max() > W * H // 8
    finally:
        ctx.close()


@pytest.mark.parametrize("each", [1, 2, 40])
def test_replicates_on_several_landscapes(each):
    import torch
    from paper_1701_03549_amd import fire
    ctx = fire.FireGPU(0)
    try:
        beta = np.array([[-0.3, -0.3, 0.2, 0.8, 1.0]])
        parts, alone = [], []
        for k, (w, h) in enumerate([(70, 40), (130, 97), (64, 200)]):
            ls = synth.make_landscape(w, h, 30 + k)
            lid = ctx.load_landscape(ls)
            parts.append(fire.make_sims(each, lid, -1, synth.ignition_site(ls)))
            # (coins follow each descriptor's sim_index, not its place)
        say(f"replicates on three landscapes, {each} each")
        for s in parts:
            alone.append(ctx.run(beta, s, SEED)[0])
        mixed = np.stack(parts, axis=1).reshape(-1)  # interleaved
        got, _ = ctx.run(beta, mixed, SEED)
        ctx.sync()
        for k in range(3):
            assert torch.equal(got[k::3], alone[k])
    finally:
        ctx.close()
