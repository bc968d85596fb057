"""Edges of the surrogate's fused kernels: batches at and around a workgroup's
rows, and the weights' transposed copy after Adam steps."""
import numpy as np
import pytest

from oracle import surrogate_ref as S

pytestmark = pytest.mark.gpu


def _rows(n, seed, side=256):
    rng = np.random.default_rng(seed)
    x = np.empty((n, 7), dtype=np.float32)
    x[:, :5] = np.clip(rng.normal(0.0, 5.0, size=(n, 5)), -30, 30)
    x[:, 5:] = rng.integers(0, side, size=(n, 2))
    return x, rng.uniform(0.0, 1.0, size=n).astype(np.float32)


@pytest.mark.parametrize("B", [1, 31, 32, 33, 65, 512])
def test_forward_rows_at_workgroup_edges(B):
    """Each row's prediction is the one it has in a batch of 512, and the
    binary64 reference's with the same bf16 rounding points."""
    import torch
    from paper_1701_03549_amd import nn
    net = nn.Surrogate(max_batch=512, lattice=(256, 256), seed=3)
    x, _ = _rows(512, 5)
    whole = net.predict(torch.from_numpy(x).cuda()).cpu().numpy()
    t = net.predict(torch.from_numpy(x[:B]).cuda()).cpu().numpy()
    assert np.array_equal(t, whole[:B])
    p = net.get_params().cpu().numpy().astype(np.float64)
    ref = S.forward(p, x[:B], 256, 256, bf16=True)["t"]
    # rows of 256 products of bf16 values: a flip of a hidden activation's
    # last bf16 place moves the sum by at most a few 2^-9 of its terms
    assert np.allclose(t, ref, rtol=1e-2, atol=1e-3)
    net.close()


def test_adam_keeps_the_weight_copies_together():
    """After Adam steps the forward pass (transposed copy) and the gradients
    (both copies) are those of a network that is given the same parameters."""
    import torch
    from paper_1701_03549_amd import nn
    B = 96
    net = nn.Surrogate(max_batch=B, lattice=(256, 256), seed=4)
    x, y = (torch.from_numpy(a).cuda() for a in _rows(B, 6))
    m = (torch.rand((B, 128, 128), generator=torch.Generator().manual_seed(1)) < 0.2).to(torch.uint8).cuda()
    for _ in range(3):
        net.train_step(x, y, m)
    other = nn.Surrogate(max_batch=B, lattice=(256, 256), seed=9)
    other.set_params(net.get_params())
    assert torch.equal(net.predict(x), other.predict(x))
    for a, b in zip(net.gradients(x, y, m), other.gradients(x, y, m)):
        assert torch.equal(a, b)
    net.close()
    other.close()
