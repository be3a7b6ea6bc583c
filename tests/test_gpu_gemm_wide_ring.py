"""bf16 GEMM with 256x256 tiles: the ring holds four half stages, so a product's first stages, its steady ones (two at a time) and its last ones take different
paths; K of one to nine stages, whole and with a last stage filled in part, rows and columns that end inside a half."""
import pytest
import torch

from test_gpu_gemm_tiles import dh  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("K", [56, 64, 128, 184, 192, 256, 264, 320, 384, 392, 448, 512, 520, 576])
def test_stages(dh, ta, tb, K):  # noqa: F811
    M, N = 2888, 3016  # 144 tiles; the last row of tiles ends in its first half, the last column in its second
    print("case", M, N, K, ta, tb, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(K)
    A = torch.randn((K, M) if ta else (M, K), generator=gen, device="cuda").bfloat16()
    B = torch.randn((N, K) if tb else (K, N), generator=gen, device="cuda").bfloat16()
    ref = torch.mm(A.double().t().contiguous() if ta else A.double(), B.double().t().contiguous() if tb else B.double())
    out = torch.full((M * N + 64,), 3.0, device="cuda", dtype=torch.bfloat16)
    dh.dh_gemm(dh.DH_BF16, ta, tb, M, N, K, A, B, out, False)
    assert float((out[: M * N].double().view(M, N) - ref).norm() / ref.norm()) <= 2.0 ** -9  # half a unit in the last place
    acc = torch.full((M * N + 64,), 3.0, device="cuda")
    dh.dh_gemm(dh.DH_BF16, ta, tb, M, N, K, A, B, acc, True)
    assert float((acc[: M * N].double().view(M, N) - 3.0 - ref).norm() / ref.norm()) <= 2e-6  # exact products, sums of 2^-24 an addition
    assert torch.all(out[M * N:] == 3.0) and torch.all(acc[M * N:] == 3.0)
