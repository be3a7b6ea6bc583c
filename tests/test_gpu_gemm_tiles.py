"""bf16 GEMM: every tile shape at its edges, K ranges summed in the block or through the workspace."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dh():
    from paper_2411_15871_amd import dhelix
    assert torch.cuda.is_available()
    return dhelix


# Sizes that take 64x64, 64x128, 96x128 (one and two blocks a unit), 128x128, 192x128, 256x128 and 256x256 tiles: last rows, columns
# and stages of K filled in part, one stage of K, K ranges that end between stages of the ring.  bf16 results: half a unit in
# the last place per element, 2^-9 in all; float32 ones: sums of up to 8192 exact products, each addition 2^-24, in blocks of random sign.
@pytest.mark.parametrize("ws", [False, True])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (72, 136, 72), (264, 520, 1000), (1000, 1536, 1544), (1096, 2056, 520), (1504, 2056, 2056), (2056, 768, 4096),
                                   (4000, 1416, 1032), (1512, 3208, 2056), (4104, 520, 4040), (4096, 1800, 584), (4088, 4104, 200), (8192, 1288, 264)])
def test_gemm_bf16_tile_shapes(dh, M, N, K, ta, tb, ws):
    print("case", M, N, K, ta, tb, ws, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A = torch.randn((K, M) if ta else (M, K), generator=gen, device="cuda").bfloat16()
    B = torch.randn((N, K) if tb else (K, N), generator=gen, device="cuda").bfloat16()
    ref = torch.mm(A.double().t().contiguous() if ta else A.double(), B.double().t().contiguous() if tb else B.double())
    need = dh.dh_gemm_workspace_bytes(dh.DH_BF16, ta, tb, M, N, K) if ws else 0
    buf = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    out = torch.full((M * N + 64,), 3.0, device="cuda", dtype=torch.bfloat16)
    dh.dh_gemm(dh.DH_BF16, ta, tb, M, N, K, A, B, out, False, buf if need else None, need)
    assert float((out[: M * N].double().view(M, N) - ref).norm() / ref.norm()) <= 2.0 ** -9
    acc = torch.full((M * N + 64,), 3.0, device="cuda")
    dh.dh_gemm(dh.DH_BF16, ta, tb, M, N, K, A, B, acc, True, buf if need else None, need)
    assert float((acc[: M * N].double().view(M, N) - 3.0 - ref).norm() / ref.norm()) <= 2e-6
    assert torch.all(out[M * N:] == 3.0) and torch.all(acc[M * N:] == 3.0)

