"""fire_gemm_bf16 where its staging changes (contractions of 256 and 1024, 256
output tiles) and at the largest grids a launch takes."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(64, 64, 255), (64, 64, 256), (65, 63, 257), (1024, 1024, 256), (1025, 1024, 256),
                                   (1025, 1024, 1023), (1025, 1024, 1024), (130, 70, 1055)])
@pytest.mark.parametrize("layout", ["nn", "nt", "tn", "odd"])
def test_stages_against_binary64(M, N, K, layout):
    """Products of bf16 are exact in fp32; K sums in fp32 are off by at most K
    roundings of 2^-24 of the sum of magnitudes."""
    import torch
    from paper_1701_03549_amd import nn
    say(f"gemm stages {M}x{N}x{K} {layout}")
    gen = torch.Generator().manual_seed(M + N + K)
    off = 1 if layout == "odd" else 0
    A = torch.randn(M * K + 1, generator=gen).to(torch.bfloat16).cuda()[off:off + M * K]
    B = torch.randn(K * N + 1, generator=gen).to(torch.bfloat16).cuda()[off:off + K * N]
    a = A.view(K, M).t() if layout == "tn" else A.view(M, K)
    b = B.view(N, K).t() if layout == "nt" else B.view(K, N)
    C = torch.empty(M, N, device="cuda")
    nn.gemm_bf16(A, B, M, N, K, a.stride(0), a.stride(1), b.stride(0), b.stride(1), C, N)
    a64, b64 = a.double().contiguous(), b.double().contiguous()
    assert ((C.double() - a64 @ b64).abs() <= K * 2.0 ** -24 * (a64.abs() @ b64.abs())).all()


def test_two_rows_of_tiles_of_the_widest_grid():
    """65 rows of 2^29 + 70 columns: 2^24 + 2 tiles, more than one row of a grid
    holds."""
    import torch
    from paper_1701_03549_amd import nn
    M, N = 65, 2 ** 29 + 70
    if torch.cuda.mem_get_info()[0] < 4 * M * N + 2 * N + 2 ** 33:
        pytest.skip("needs 142 GB of device memory")
    say(f"gemm {M}x{N}x1")
    A = torch.arange(1, M + 1, device="cuda").to(torch.bfloat16)  # whole numbers up to 65: exact
    B = torch.empty(N, dtype=torch.bfloat16, device="cuda").fill_(3.0)
    B[-70:] = 5.0
    C = torch.empty((M, N), dtype=torch.float32, device="cuda")
    C[:, -100:] = 0.0
    C[:, :100] = 0.0
    nn.gemm_bf16(A, B, M, N, 1, 1, 1, N, 1, C, N)
    for cols, rows in ((slice(0, 100), 3.0), (slice(N - 100, N - 70), 3.0), (slice(N - 70, N), 5.0)):
        assert torch.equal(C[:, cols], (A.float() * rows)[:, None].expand(M, cols.stop - cols.start))
    del C, B
    torch.cuda.empty_cache()
