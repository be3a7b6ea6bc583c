"""bf16 GEMM: every tile shape at its edges, K ranges summed in the block or through the workspace, and a linear's two gradient
products in one launch against the two apart."""
import pytest
import torch

from paper_2411_15871_amd import harness as H

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


LLAMA = dict(arch="llama", n_ranks=2, bf16=True)
PAIRS = [dict(LLAMA, batch=1, seq=40, hidden=264, nq=2, nkv=1, d=64, ffn=136),                # SwiGLU on its own
         dict(LLAMA, batch=3, seq=333, hidden=1024, nq=4, nkv=4, d=64, ffn=1408),             # SwiGLU in the data gradient's epilogue
         dict(LLAMA, batch=1, seq=2000, hidden=1024, nq=8, nkv=8, d=64, ffn=1408, rope_pairing=1),
         dict(LLAMA, batch=1, seq=2049, hidden=2048, nq=4, nkv=1, d=128, ffn=896),
         dict(arch="gpt", batch=2, seq=264, hidden=520, nq=4, nkv=4, d=128, ffn=1000, n_ranks=4, bf16=True),
         dict(arch="moe", batch=1, seq=500, hidden=1024, nq=4, nkv=2, d=128, ffn=800, n_ranks=1, bf16=True, n_experts=8, n_local=2),
         dict(arch="moe", batch=1, seq=1, hidden=256, nq=2, nkv=2, d=64, ffn=264, n_ranks=1, bf16=True, n_experts=8, n_local=4),  # experts without rows
         dict(arch="llama_cp", batch=1, seq=384, hidden=768, nq=4, nkv=1, d=128, ffn=1024, n_ranks=2, bf16=True, cp_ranks=2, cp_rank=1),
         dict(LLAMA, bf16=False, batch=1, seq=37, hidden=72, nq=4, nkv=2, d=16, ffn=104),
         dict(LLAMA, bf16=False, batch=1, seq=128, hidden=256, nq=4, nkv=4, d=64, ffn=688)]


# A backward pass issues a linear's data and weight gradient as one launch where the plan has them next to each other: the same
# bits as with every weight gradient moved to the end of the pass, where each is a launch of its own.
@pytest.mark.parametrize("cfg", PAIRS, ids=lambda c: "-".join(str(c[k]) for k in ("arch", "batch", "seq", "hidden", "ffn")))
def test_paired_gradients_match_separate_launches(dh, cfg):
    print("case", cfg, flush=True)
    run = H.LayerRun(cfg)
    try:
        a, b = run.strand(0), run.strand(1)
        run.fwd(b)
        run.bwd(b)
        torch.cuda.synchronize()
        want = [b.dx.clone()] + [g.clone() for g in run.g.values()]
        names = dh.op_names(H.ARCH[cfg["arch"]], 1)
        gf = dh.dh_layer_op_graph(run.layer, 0)
        late = [i for i, n in enumerate(names) if n.endswith("WGRAD")]
        order = [i for i in range(len(names)) if i not in late] + late
        plan = dh.make_plan(list(range(gf.n_ops)), order, [(0, gf.n_ops, 0, len(order))])
        sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        for t in [b.dx] + list(run.g.values()):
            t.zero_()
        torch.cuda.synchronize()
        run.si_step(a, b, plan, sa, sb)
        torch.cuda.synchronize()
        for got, ref in zip([b.dx] + list(run.g.values()), want):
            assert torch.equal(got, ref)
    finally:
        run.close()
