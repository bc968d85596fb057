"""Small fronts on lattices whose burn bitset lies in global memory: fires from
corners, edges and word boundaries of lattices whose width is at and around a
multiple of 32, against the oracle, with tables and per-trial thresholds and
with turn-off times."""
import numpy as np
import pytest

import oracle
from gpu_util import SEED, compare_with_oracle, say
from paper_1701_03549_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [351, 352, 353])
@pytest.mark.parametrize("turn_off", [False, True])
def test_small_fronts_match_oracle(W, turn_off):
    """4096 rows of 11 or 12 words: over the 40,960 words of the LDS. beta 2.5
    ignites whole squares; a few dozen cells a step for at most 12 steps."""
    from paper_1701_03549_amd import fire
    H = 4096
    ls = synth.random_small_landscape(W, H, W, p_blocked=0.05)
    igns = [(0, 0), (W - 1, 0), (0, H - 1), (W - 1, H - 1), (31, 700), (32, 701), (W - 1, 2000), (319, H - 1)]
    for x, y in igns:
        ls["veg"][y, x] = 2
    betas = [(2.5, 0.0, 0.0, 0.3, 0.0), (0.0, 0.2, 0.1, 0.4, 0.1)]
    g = fire.FireGPU(0)
    try:
        lid = g.load_landscape(ls)
        steps = None
        if turn_off:
            steps = np.full(256, 3, dtype=np.uint8)
            steps[2] = 1
            g.set_burn_steps(lid, steps)
        n = len(igns)
        sims = fire.make_sims(2 * n, lid, -1, np.array(igns * 2), param_index=np.repeat([0, 1], n))
        sims["max_steps"] = 6 if turn_off else 12
        T = [g.thresholds(lid, b).cpu().numpy().view(np.uint32) for b in betas]
        for threads, table in ((64, 1), (256, 0), (1024, 1), (1024, 0)):
            say(f"global bitset {W}x{H} turn-off {turn_off} threads {threads} table {table}")
            g.set_schedule(threads=threads, queue_cap=256, table_mode=table, wg_per_cu=1)
            res, maps = g.run(betas, sims, SEED, want_maps=True)
            g.sync()
            compare_with_oracle(ls, T, fire.results_to_numpy(res), maps.cpu().numpy().view(np.uint32), sims, SEED,
                                burn_steps=steps)
    finally:
        g.close()
