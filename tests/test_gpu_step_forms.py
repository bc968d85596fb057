"""The simulation step's forms (two lanes a cell, a lane a cell, queue entries
with spilling) and the bitset's edges, against the oracle: lattice widths at
and around word boundaries, fires from corners and edges, fronts that pass
each form's limit for the workgroup sizes, queues of 64 entries that spill,
tables and per-trial thresholds, whole lattice and window."""
import numpy as np
import pytest

import oracle
from gpu_util import SEED, compare_with_oracle, say
from paper_1701_03549_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def g():
    from paper_1701_03549_amd import fire
    ctx = fire.FireGPU(0)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("W,H", [(32, 40), (33, 35), (63, 64), (64, 64), (96, 33), (160, 130)])
@pytest.mark.parametrize("threads", [64, 128, 256, 512])
def test_step_forms_match_oracle(g, W, H, threads):
    """beta 2.5 makes nearly every coin succeed (fronts of whole squares, the
    most duplicates), beta 0 every second one."""
    from paper_1701_03549_amd import fire
    ls = synth.random_small_landscape(W, H, 7 * W + H, p_blocked=0.05)
    ls["veg"][[0, 0, H - 1, H - 1, H // 2], [0, W - 1, 0, W - 1, min(31, W - 1)]] = 2
    igns = [(0, 0), (W - 1, 0), (0, H - 1), (W - 1, H - 1), (min(31, W - 1), H // 2)]
    betas = [(2.5, 0.0, 0.0, 0.3, 0.0), (0.0, 0.2, 0.1, 0.4, 0.1)]
    lid = g.load_landscape(ls)
    sims = fire.make_sims(10, lid, -1, np.array(igns * 2), param_index=np.repeat([0, 1], 5))
    sims["max_steps"][4] = 5
    for table in (1, 0):
        for cap, win in ((64, 0), (1024, 0), (128, 64)):
            say(f"step forms {W}x{H} threads {threads} table {table} queue {cap} window {win}")
            g.set_schedule(threads=threads, queue_cap=cap, table_mode=table, wg_per_cu=2, window=win)
            res, maps = g.run(betas, sims, SEED, want_maps=True)
            g.sync()
            T = [g.thresholds(lid, b).cpu().numpy().view(np.uint32) for b in betas]
            compare_with_oracle(ls, T, fire.results_to_numpy(res), maps.cpu().numpy().view(np.uint32), sims, SEED)
    g.set_schedule(reset=True)
    g.free_landscape(lid)
