"""A few fires of one parameter vector on a lattice of 2^22 cells and more, from
host descriptors: small fires take no Eq. 1 table (32 B of every cell), large
ones, and smaller lattices, do; results are those of table runs."""
import numpy as np
import pytest

from gpu_util import SEED, say
from paper_1701_03549_amd import synth

pytestmark = pytest.mark.gpu

SMALL, OPEN = (-3.0, -0.5, 2.0, 1.0, 2.0), (0.0, 0.0, 0.0, 0.5, 0.5)


@pytest.mark.parametrize("W,H,beta,n,table", [(2048, 2048, SMALL, 1, False), (2048, 2048, SMALL, 2, False),
                                              (2049, 2055, SMALL, 8, False), (2049, 2055, SMALL, 9, True),
                                              (2048, 2048, OPEN, 2, True), (2048, 2047, SMALL, 2, True)])
def test_tables_of_few_fires(W, H, beta, n, table):
    import torch
    from paper_1701_03549_amd import fire
    say(f"{n} fires on {W}x{H}, beta {beta}")
    ls = synth.make_landscape(W, H, 102)
    ctx = fire.FireGPU(0)
    try:
        lid = ctx.load_landscape(ls)
        sims = fire.make_sims(n, lid, -1, synth.ignition_site(ls), max_steps=40)
        ctx.sync()
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        got, gmaps = ctx.run([beta], sims, SEED, want_maps=True)
        ctx.sync()
        used = free - torch.cuda.mem_get_info()[0]
        queues = n * 2 * W * H * 4  # two queues a simulation in flight; a table is 32 B a cell
        assert (used > queues + 16 * W * H) == table
        assert (ctx.get_schedule(W * H, 1, n)["table_mode"] == 1)  # what other batches of the class use
        ctx.set_schedule(256, 1024, 1, 1)
        want, wmaps = ctx.run([beta], sims, SEED, want_maps=True)
        ctx.sync()
        assert torch.equal(got, want) and torch.equal(gmaps, wmaps)
        if beta is OPEN:
            assert fire.results_to_numpy(want)["burnt"].max() > 1000
    finally:
        ctx.close()
