"""Scores written into memory that also holds the network's inputs: a program
that no longer needs its rows may put the scores of one call there."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 33, 65536])
@pytest.mark.parametrize("at", ["first", "last"])
def test_scores_over_the_inputs(rows, at):
    """65536 rows are more workgroups than are resident at once, so the later
    ones read their rows after the first ones' scores are written."""
    import torch
    from paper_1701_03549_amd import nn
    say(f"scores over the inputs: {rows} rows, {at}")
    net = nn.Surrogate(max_batch=rows, lattice=(256, 256), seed=3)
    try:
        x = torch.randn(rows, 7, generator=torch.Generator().manual_seed(rows)).cuda()
        want = net.predict(x).clone()
        flat = x.view(-1)
        out = flat[:rows] if at == "first" else flat[6 * rows:]
        assert torch.equal(net.predict(x, out=out), want)
    finally:
        net.close()
