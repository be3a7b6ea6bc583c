"""A linear's two gradient products in one launch: every tile shape the rule takes, dense and grouped, by itself and beside another strand, against the
two apart (the same bits), and an SI step that takes such launches against one that issues every weight gradient by itself.  Which shape a launch
takes is asked of the library, so that none is left out when the rule's figures change."""
import ctypes as C

import pytest
import torch

from paper_2411_15871_amd import dhelix as dh
from paper_2411_15871_amd import harness as H

# internal to the library, not part of the C interface
SHAPE, PAIR, GROUPED = "_Z18dh_gemm_pair_shapeiiiib", "_Z24dh_launch_gemm_pair_bf16iiiPKDF16bS0_S0_PDF16bPfS0_bPvmP12ihipStream_t", \
    "_Z32dh_launch_gemm_grouped_pair_bf16iPKiiiiPKDF16bS2_S2_PDF16bPfbP12ihipStream_t"
# tile shape -> (groups, T, k, n, beside): the data gradient is T x k over n, the weight gradient k x n over T, of all groups together
CASES = {
    1: [(0, 199, 4088, 816, False), (0, 129, 3912, 976, True), (8, 40, 1448, 144, False), (8, 33, 1320, 160, True)],        # 128x128, two blocks a unit
    2: [(0, 282, 3976, 1240, False), (0, 652, 2616, 1720, True), (4, 1086, 984, 1320, False), (8, 4460, 200, 2664, True), (0, 1500, 2048, 2048, True)],  # 256x128
    3: [(0, 34, 136, 128, False), (0, 35, 128, 144, True), (4, 33, 128, 128, False), (8, 32, 136, 128, True)],              # 64x64
    4: [(0, 69, 3808, 808, False), (0, 125, 3936, 784, True), (4, 270, 1056, 680, False), (4, 786, 1368, 328, True)],        # 128x128, one block a unit
    5: [(0, 131, 3960, 1248, False), (0, 137, 3344, 1432, True), (4, 397, 1120, 1128, False), (2, 353, 1824, 1400, True)],   # 192x128
    6: [(0, 32, 3496, 744, False), (0, 66, 3032, 600, True), (2, 36, 2480, 504, False), (1, 67, 2376, 712, True)],           # 96x128, one block a unit
    7: [(0, 233, 3952, 840, False), (0, 268, 3536, 544, True), (2, 135, 2744, 784, False), (2, 134, 3400, 336, True)],       # 96x128, two
    8: [(0, 69, 1952, 456, False), (0, 70, 1704, 464, True), (8, 34, 840, 216, False), (8, 33, 792, 224, True)],             # 64x128
}
ALL = [(cfg,) + c for cfg, cs in CASES.items() for c in cs]


def function(name, *argtypes):
    f = getattr(dh.lib, name)
    f.restype, f.argtypes = C.c_int, list(argtypes)
    return f


def pair_shape(groups, T, k, n, beside):
    return function(SHAPE, *[C.c_int] * 4, C.c_bool)(groups, T, k, n, beside)


def test_cases_take_every_shape():
    assert sorted(CASES) == list(range(1, 9))
    for cfg, groups, T, k, n, beside in ALL:
        assert pair_shape(groups, T, k, n, beside) == cfg, (cfg, groups, T, k, n, beside)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,groups,T,k,n,beside", ALL)
def test_pair_has_the_bits_of_two_launches(cfg, groups, T, k, n, beside):
    print("case", cfg, groups, T, k, n, beside, flush=True)
    assert pair_shape(groups, T, k, n, beside) == cfg  # on this device, too
    gen = torch.Generator(device="cuda").manual_seed(T + k)
    bf = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    G = max(1, groups)
    dY, W, X = bf(T, n), bf(G, k, n), bf(T, k)
    p, stream = (lambda t: t.data_ptr()), torch.cuda.current_stream().cuda_stream
    guard = lambda *s, dtype: torch.full((torch.Size(s).numel() + 64,), 3.0, device="cuda", dtype=dtype)
    for gu in [None] + ([bf(T, 2 * k)] if groups == 0 and dh.dh_gemm_swiglu_bwd_fits(T, k, n) else []):
        wide = k if gu is None else 2 * k
        (dX, dX2), (dW, dW2) = [guard(T, wide, dtype=torch.bfloat16) for _ in range(2)], [guard(G, k, n, dtype=torch.float32) for _ in range(2)]
        if groups == 0:
            need = max(dh.dh_gemm_workspace_bytes(dh.DH_BF16, 0, 1, T, k, n), dh.dh_gemm_workspace_bytes(dh.DH_BF16, 1, 0, k, n, T), 16)
            ws = torch.empty(need, dtype=torch.uint8, device="cuda")
            f = function(PAIR, *[C.c_int] * 3, *[C.c_void_p] * 6, C.c_bool, C.c_void_p, C.c_size_t, C.c_void_p)
            assert f(T, k, n, p(dY), p(W), p(X), p(dX), p(dW), None if gu is None else p(gu), beside, p(ws), need, stream) == 0
            if gu is None:
                dh.dh_gemm(dh.DH_BF16, 0, 1, T, k, n, dY, W, dX2, False, ws, need)
            else:
                dh.dh_gemm_swiglu_bwd(T, k, n, dY, W, gu, dX2)
            dh.dh_gemm(dh.DH_BF16, 1, 0, k, n, T, X, dY, dW2, True, ws, need)
        else:  # unequal groups, one of them empty
            cuts = torch.randint(0, T + 1, (G - 1,), generator=torch.Generator().manual_seed(T)).tolist()
            cuts = sorted(cuts[:-1] + [cuts[0] if G > 2 else T] if G > 1 else []) + [T]
            rows = torch.tensor([b - a for a, b in zip([0] + cuts, cuts)], dtype=torch.int32, device="cuda")
            f = function(GROUPED, C.c_int, C.c_void_p, *[C.c_int] * 3, *[C.c_void_p] * 5, C.c_bool, C.c_void_p)
            assert f(G, p(rows), T, k, n, p(dY), p(W), p(X), p(dX), p(dW), beside, stream) == 0
            dh.dh_gemm_grouped(dh.DH_BF16, 1, G, rows, T, n, k, dY, W, dX2)
            dh.dh_gemm_grouped(dh.DH_BF16, 2, G, rows, T, k, n, X, dY, dW2)
        torch.cuda.synchronize()
        assert torch.equal(dX, dX2) and torch.equal(dW, dW2)
        assert torch.all(dX[T * wide:] == 3.0) and torch.all(dW[G * k * n:] == 3.0)
        assert float((dW[: G * k * n].double() - 3.0).norm()) > 0


# the linears of each layer as (groups, T, k, n), in a step in the default order beside another strand
STEPS = [dict(arch="moe", batch=1, seq=1500, hidden=2048, nq=16, nkv=4, d=128, ffn=800, n_ranks=1, bf16=True, n_experts=8, n_local=2),
         dict(arch="gpt", batch=1, seq=1676, hidden=1664, nq=4, nkv=4, d=128, ffn=2416, n_ranks=4, bf16=True),
         dict(arch="llama", batch=3, seq=333, hidden=1024, nq=4, nkv=4, d=64, ffn=1408, n_ranks=2, bf16=True),
         dict(arch="llama_cp", batch=1, seq=384, hidden=768, nq=4, nkv=1, d=128, ffn=1024, n_ranks=2, bf16=True, cp_ranks=2, cp_rank=1),
         dict(arch="llama", batch=1, seq=128, hidden=256, nq=4, nkv=4, d=64, ffn=688, n_ranks=2, bf16=False)]


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", STEPS, ids=lambda c: "%s-%d-%s" % (c["arch"], c["hidden"], "bf16" if c["bf16"] else "f32"))
def test_step_with_pairs_beside_a_strand(cfg):
    print("case", cfg, flush=True)
    moe, gpt = cfg["arch"] == "moe", cfg["arch"] == "gpt"
    T, Hd, F, nq, nkv, d = cfg["batch"] * cfg["seq"], cfg["hidden"], cfg["ffn"], cfg["nq"], cfg["nkv"], cfg["d"]
    G, Tf, Fin = (cfg["n_local"], 2 * T, 2 * F) if moe else (0, T, F if gpt else 2 * F)
    linears = [(G, Tf, F, Hd), (G, Tf, Hd, Fin), (0, T, nq * d, Hd), (0, T, Hd, (nq + 2 * nkv) * d)]
    if cfg["bf16"]:
        assert any(pair_shape(*l, True) for l in linears)
    run = H.LayerRun(cfg)
    try:
        a, b = run.strand(0), run.strand(1)
        run.fwd(b)
        torch.cuda.synchronize()
        names = dh.op_names(H.ARCH[cfg["arch"]], 1)
        nf, nb = dh.dh_layer_op_graph(run.layer, 0).n_ops, len(names)
        late = [i for i, n in enumerate(names) if n.endswith("WGRAD")]
        sa, sb, sc = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        got = []
        for order in (list(range(nb)), [i for i in range(nb) if i not in late] + late):
            for t in [b.dx] + list(run.g.values()):
                t.zero_()
            torch.cuda.synchronize()
            run.si_step(a, b, dh.make_plan(list(range(nf)), order, [(0, nf, 0, nb)]), sa, sb, sc)
            torch.cuda.synchronize()
            got.append([t.clone() for t in [a.out, b.dx] + list(run.g.values())])
        for x, y in zip(*got):
            assert torch.equal(x, y)
    finally:
        run.close()
