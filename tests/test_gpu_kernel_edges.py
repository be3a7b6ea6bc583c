"""GPU parity of single operators at the edges of their kernels' tiles, steps and dispatch rules, against plain float64
products on the host or float32 ones on the device."""
import numpy as np
import pytest
import torch

from oracle import layer_ref as R
from paper_2411_15871_amd import inputs as gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dh():
    from paper_2411_15871_amd import dhelix
    assert torch.cuda.is_available()
    return dhelix


def rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


# float32 GEMM: 16x16 tiles (few blocks) and 32x32 tiles, K ranges that leave waves without work, rows that allow 16-byte
# loads and rows that do not
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(16, 16, 16), (17, 33, 31), (128, 256, 1376), (520, 516, 36), (513, 1031, 70), (1024, 512, 33)])
def test_gemm_f32_tiles(dh, ta, tb, M, N, K):
    A, B = gen.normal(80, (K, M) if ta else (M, K)), gen.normal(81, (N, K) if tb else (K, N))
    bias = gen.normal(82, (N,))
    Ad, Bd, bd = (torch.from_numpy(v).cuda() for v in (A, B, bias))
    ref = (A.T if ta else A).astype(np.float64) @ (B.T if tb else B).astype(np.float64)
    C = torch.full((M * N + 64,), 3.0, device="cuda")
    dh.dh_gemm_bias(dh.DH_F32, ta, tb, M, N, K, Ad, Bd, bd, C, False)
    assert rel(C[: M * N].cpu().numpy().reshape(M, N), ref + bias) <= 1e-6
    C.fill_(3.0)
    dh.dh_gemm(dh.DH_F32, ta, tb, M, N, K, Ad, Bd, C, True)
    assert rel(C[: M * N].cpu().numpy().reshape(M, N), ref + 3.0) <= 1e-6
    assert torch.all(C[M * N:] == 3.0)


# float32 attention: every instantiation of the head width, ragged last tiles, grouped heads, a query offset that is no
# multiple of a tile
@pytest.mark.parametrize("batch,seq,q_off,nq,nkv,d", [(1, 1, 0, 1, 1, 16), (2, 17, 0, 4, 2, 32), (1, 130, 0, 3, 1, 64), (1, 200, 0, 4, 4, 128),
                                                      (1, 70, 0, 2, 1, 256), (2, 37, 21, 4, 2, 40), (1, 48, 160, 8, 1, 128)])
def test_attention_f32_tiles(dh, batch, seq, q_off, nq, nkv, d):
    T, S = batch * seq, q_off + seq
    full = [gen.normal(83 + i, (batch * S, n * d)) for i, n in enumerate((nq, nkv, nkv))]
    dof = gen.normal(86, (batch * S, nq * d))
    own = np.concatenate([np.arange(b * S + q_off, (b + 1) * S) for b in range(batch)])
    dof[np.setdiff1d(np.arange(batch * S), own)] = 0.0   # only the last seq positions are queries
    q64, k64, v64 = (a.astype(np.float64).reshape(batch * S, n, d) for a, n in zip(full, (nq, nkv, nkv)))
    o_ref, lse_ref = R.attention_fwd(q64, k64, v64, batch, S)
    dq, dk, dv = R.attention_bwd(dof.astype(np.float64).reshape(batch * S, nq, d), q64, k64, v64, batch, S)
    qkv = torch.from_numpy(np.concatenate(full, axis=1)[own].copy()).cuda()
    kv = torch.from_numpy(np.concatenate(full[1:], axis=1).copy()).cuda()
    do = torch.from_numpy(dof[own].copy()).cuda()
    o, lse, delta = torch.empty(T, nq * d, device="cuda"), torch.empty(nq, T, device="cuda"), torch.empty(nq, T, device="cuda")
    dqkv, dkv = torch.zeros_like(qkv), torch.zeros_like(kv)
    dh.dh_attn_ctx_fwd(dh.DH_F32, batch, seq, q_off, nq, nkv, d, qkv, kv, o, lse)
    dh.dh_attn_ctx_bwd(dh.DH_F32, batch, seq, q_off, nq, nkv, d, qkv, kv, o, do, lse, dqkv, dkv, delta)
    assert rel(o.cpu().numpy(), o_ref.reshape(batch * S, -1)[own]) <= 2e-6
    assert np.max(np.abs(lse.cpu().numpy() - lse_ref[:, own])) <= 1e-5
    floor = np.linalg.norm(dv) if S == 1 else 0.0        # dq = dk = 0 exactly when a row sees one key
    for got, ref in ((dqkv.cpu().numpy()[:, : nq * d], dq.reshape(batch * S, -1)[own]), (dkv.cpu().numpy()[:, : nkv * d], dk.reshape(batch * S, -1)),
                     (dkv.cpu().numpy()[:, nkv * d:], dv.reshape(batch * S, -1))):
        assert np.linalg.norm(got - ref) <= 5e-6 * max(np.linalg.norm(ref), floor)


# float32 attention with an infinity or a NaN in one row of one operand: what may not see that row keeps its values (sums of
# at most q_off + seq terms in another order), what sees it does not stay finite
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("what", ["q", "k", "v", "do"])
@pytest.mark.parametrize("batch,seq,q_off,nq,nkv,d,row", [(2, 37, 0, 4, 2, 24, 15), (1, 64, 0, 2, 2, 64, 0), (1, 150, 0, 2, 1, 128, 149), (1, 40, 0, 2, 1, 256, 20),
                                                          (1, 37, 21, 4, 2, 64, 30), (1, 40, 160, 2, 1, 128, 5)])
def test_attention_f32_nonfinite_rows(dh, batch, seq, q_off, nq, nkv, d, row, what, bad):
    print("case", batch, seq, q_off, nq, nkv, d, row, what, bad, flush=True)
    T, S, b = batch * seq, q_off + seq, batch - 1

    def run(dirty):
        qkv, kv, do = gen.normal(90, (T, (nq + 2 * nkv) * d)), gen.normal(91, (batch * S, 2 * nkv * d)), gen.normal(92, (T, nq * d))
        if dirty:  # element 1 of head 0 of the row (k, v) or of the query at position q_off + row (q, do)
            a, r, c = {"q": (qkv, b * seq + row, 1), "k": (kv, b * S + q_off + row, 1), "v": (kv, b * S + q_off + row, nkv * d + 1),
                       "do": (do, b * seq + row, 1)}[what]
            a[r, c] = bad
        qkv, kv, do = (torch.from_numpy(x).cuda() for x in (qkv, kv, do))
        o, lse, delta = torch.empty(T, nq * d, device="cuda"), torch.empty(nq, T, device="cuda"), torch.empty(nq, T, device="cuda")
        dqkv, dkv = torch.zeros_like(qkv), torch.zeros_like(kv)
        dh.dh_attn_ctx_fwd(dh.DH_F32, batch, seq, q_off, nq, nkv, d, qkv, kv, o, lse)
        dh.dh_attn_ctx_bwd(dh.DH_F32, batch, seq, q_off, nq, nkv, d, qkv, kv, o, do, lse, dqkv, dkv, delta)
        heads = lambda t, n, m: t.cpu().numpy().reshape(batch, m, n, d)
        return {"o": heads(o, nq, seq), "dq": heads(dqkv[:, : nq * d].contiguous(), nq, seq),
                "dk": heads(dkv[:, : nkv * d].contiguous(), nkv, S), "dv": heads(dkv[:, nkv * d:].contiguous(), nkv, S)}

    clean, got = run(False), run(True)
    i = np.arange(seq)
    spoilt = {"o": {"q": i == row, "k": i >= row, "v": i >= row, "do": i < 0}[what],    # queries of head 0 that see it
              "dq": {"q": i == row, "k": i >= row, "v": i >= row, "do": i == row}[what]}
    j = np.arange(S)                                                                     # keys of the group of head 0
    spoilt["dk"] = {"q": j <= q_off + row, "k": j >= 0, "v": j >= 0, "do": j <= q_off + row}[what]
    spoilt["dv"] = {"q": j <= q_off + row, "k": j >= 0, "v": j < 0, "do": j <= q_off + row}[what]
    n_h = {"o": 1 if what in ("q", "do") else nq // nkv, "dq": 1 if what in ("q", "do") else nq // nkv, "dk": 1, "dv": 1}
    for name, ref in clean.items():
        keep = np.ones(ref.shape, bool)
        hs = np.arange(n_h[name])
        keep[b, np.flatnonzero(spoilt[name])[:, None], hs[None, :]] = False
        scale = np.abs(ref).max()
        assert np.all(np.isfinite(got[name][keep])), name
        # a query's or key's terms in another order: S (and nq / nkv times as many for dk, dv) roundings of 2^-24 of the partial sums
        assert np.max(np.abs(got[name] - ref)[keep], initial=0.0) <= 2.0 ** -24 * S * (nq // nkv) * scale, name
        for r in np.flatnonzero(spoilt[name]) if np.isnan(bad) or what in ("v", "do") else ():  # an infinite score may be minus infinity
            assert not np.all(np.isfinite(got[name][b, r, 0])), (name, r)


# float32 attention where every score a query sees is minus infinity: the softmax of such a row has no value, and says so; a row
# that also sees a finite score has the softmax of those, wherever the tiles lie
@pytest.mark.parametrize("seq,first,d", [(20, 1, 32), (150, 64, 64), (300, 150, 128), (40, 17, 256)])
def test_attention_f32_no_finite_score(dh, seq, first, d):
    qkv = np.abs(gen.normal(93, (seq, 3 * d))) + 0.1
    qkv[:first, d: 2 * d] = -np.inf                    # the first keys: scores of minus infinity
    qkv = torch.from_numpy(qkv.astype(np.float32)).cuda()
    o, lse = torch.empty(seq, d, device="cuda"), torch.empty(1, seq, device="cuda")
    dh.dh_attn_fwd(dh.DH_F32, 1, seq, 1, 1, d, qkv, o, lse)
    assert torch.all(torch.isnan(o[:first])) and torch.all(torch.isnan(lse[0, :first]))
    ref, ref_lse = R.attention_fwd(*(qkv[first:, i * d: (i + 1) * d].cpu().double().numpy()[:, None] for i in range(3)), 1, seq - first)
    assert rel(o[first:].cpu().numpy(), ref[:, 0]) <= 2e-6
    assert np.max(np.abs(lse[0, first:].cpu().numpy() - ref_lse[0])) <= 1e-5


# float32 attention with more sequences than a grid's third dimension holds: every sequence is one token that sees itself
@pytest.mark.parametrize("batch", [65535, 65537, 140001])
def test_attention_f32_many_sequences(dh, batch):
    nq, nkv, d = 2, 1, 16
    g = torch.Generator(device="cuda").manual_seed(5)
    qkv = torch.randn(batch, (nq + 2 * nkv) * d, generator=g, device="cuda")
    do = torch.randn(batch, nq * d, generator=g, device="cuda")
    o, lse, delta = torch.zeros(batch, nq * d, device="cuda"), torch.zeros(nq, batch, device="cuda"), torch.zeros(nq, batch, device="cuda")
    dqkv = torch.full_like(qkv, 7.0)
    dh.dh_attn_fwd(dh.DH_F32, batch, 1, nq, nkv, d, qkv, o, lse)
    dh.dh_attn_bwd(dh.DH_F32, batch, 1, nq, nkv, d, qkv, o, do, lse, dqkv, delta)
    q, k, v = qkv[:, : nq * d].view(batch, nq, d), qkv[:, nq * d: (nq + 1) * d], qkv[:, (nq + 1) * d:]
    # one key: o = v, dv = the sum of the group's dO; dq and dk are zero up to the rounding of dP - delta
    assert torch.equal(o.view(batch, nq, d), v[:, None].expand(batch, nq, d))
    s = (q.double() * k.double()[:, None]).sum(-1) / d ** 0.5
    assert float((lse.t().double() - s).abs().max()) <= 1e-5
    assert float((dqkv[:, (nq + 1) * d:] - do.view(batch, nq, d).sum(1)).abs().max()) <= 1e-5
    assert float(dqkv[:, : (nq + 1) * d].abs().max()) <= 1e-3


# float32 GEMM with more tiles of rows, and of columns, than a grid's second dimension holds
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(65535 * 32 + 5, 8, 8), (8, 65535 * 32 + 4, 8), (65535 * 16 + 40, 7, 5)])
def test_gemm_f32_long_sides(dh, ta, tb, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(6)
    A, B = torch.randn((K, M) if ta else (M, K), generator=g, device="cuda"), torch.randn((N, K) if tb else (K, N), generator=g, device="cuda")
    C = torch.full((M, N), 3.0, device="cuda")
    dh.dh_gemm(dh.DH_F32, ta, tb, M, N, K, A, B, C, False)
    a, b = (A.t() if ta else A).double(), (B.t() if tb else B).double()
    err = torch.zeros(M, N, dtype=torch.float64, device="cuda") - C
    for k in range(K):
        err += a[:, k: k + 1] * b[k: k + 1]
    assert float(err.abs().max()) <= 1e-4   # 8 products of normal numbers in 32 bits


# float32 GEMM with a result or a bias that is 4-byte aligned only: stored (and read) one element at a time
@pytest.mark.parametrize("M,N,K", [(40, 36, 20), (520, 516, 36)])
def test_gemm_f32_misaligned_result(dh, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(7)
    A, B = torch.randn(M, K, generator=g, device="cuda"), torch.randn(K, N, generator=g, device="cuda")
    buf, bias = torch.full((M * N + 8,), 3.0, device="cuda"), torch.randn(N + 1, generator=g, device="cuda")[1:]
    ref = torch.empty(M, N, device="cuda")
    dh.dh_gemm_bias(dh.DH_F32, 0, 0, M, N, K, A, B, bias.clone(), ref, False)
    dh.dh_gemm_bias(dh.DH_F32, 0, 0, M, N, K, A, B, bias, buf[1:], False)
    assert torch.equal(buf[1: M * N + 1].view(M, N), ref)
    assert float(buf[0]) == 3.0 and torch.all(buf[M * N + 1:] == 3.0)


# bf16 GEMM with 256x256 tiles: K below, at and beyond its two-stage pipeline and off the K step, ragged rows and columns
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(2824, 3080, 8), (2817, 3080, 64), (2560, 3336, 72), (2560, 3328, 128), (3080, 2568, 200), (2832, 2824, 264),
                                   (2568, 3088, 328)])
def test_gemm_bf16_wide_tiles(dh, ta, tb, M, N, K):
    if ta:
        M = (M + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device="cuda", dtype=torch.bfloat16)
    B = torch.randn((N, K) if tb else (K, N), generator=g, device="cuda", dtype=torch.bfloat16)
    bias = torch.randn(N, generator=g, device="cuda", dtype=torch.bfloat16)
    ref = (A.float().t().contiguous() if ta else A.float()) @ (B.float().t().contiguous() if tb else B.float())
    C = torch.full((M * N + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    dh.dh_gemm_bias(dh.DH_BF16, ta, tb, M, N, K, A, B, bias, C, False)
    want = ref + bias.float()
    assert float((C[: M * N].view(M, N).float() - want).norm() / want.norm()) <= 4e-3
    assert torch.all(C[M * N:] == 7.0)
    Cf = torch.full((M * N + 64,), 1.0, device="cuda")
    dh.dh_gemm(dh.DH_BF16, ta, tb, M, N, K, A, B, Cf, True)
    assert float((Cf[: M * N].view(M, N) - 1.0 - ref).norm() / ref.norm()) <= 2e-5
    assert torch.all(Cf[M * N:] == 1.0)


# bf16 GEMM over its tile shapes: 64x64 alone and with K ranges summed in the block (also ranges that end inside a stage), 128x128
# one and two blocks to a unit, 256x128, K split through the workspace, 256x256; K below the ring's depth and off its step
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0)])
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (64, 64, 64), (130, 200, 520), (65, 72, 1000), (72, 136, 1576), (1000, 520, 1064), (2056, 264, 328),
                                   (656, 384, 7680), (1030, 2304, 1000), (264, 4096, 3560), (3081, 3080, 136), (4096, 2072, 1032), (2050, 3080, 1992),
                                   (4090, 4088, 200), (4096, 3848, 456)])
def test_gemm_bf16_tile_shapes(dh, ta, tb, M, N, K):
    test_gemm_bf16_wide_tiles(dh, ta, tb, M, N, K)
    if ta:
        M = (M + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(M + K)
    A = torch.randn((K, M) if ta else (M, K), generator=g, device="cuda", dtype=torch.bfloat16)
    B = torch.randn((N, K) if tb else (K, N), generator=g, device="cuda", dtype=torch.bfloat16)
    ref = (A.float().t().contiguous() if ta else A.float()) @ (B.float().t().contiguous() if tb else B.float())
    C = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
    wsb = dh.dh_gemm_workspace_bytes(dh.DH_BF16, ta, tb, M, N, K)
    ws = torch.empty(max(wsb, 16), dtype=torch.uint8, device="cuda")
    dh.dh_gemm(dh.DH_BF16, ta, tb, M, N, K, A, B, C, False, ws, wsb)
    assert float((C.float() - ref).norm() / ref.norm()) <= 4e-3


# SwiGLU in the epilogues of every tile shape, token counts and feature widths that fill no tile
@pytest.mark.parametrize("T,F,H", [(1, 128, 64), (200, 384, 1096), (700, 1152, 1000), (2049, 1792, 1024), (4000, 3584, 1536), (130, 136, 200), (2047, 1800, 1024)])
def test_gemm_swiglu_ragged(dh, T, F, H):
    g = torch.Generator(device="cuda").manual_seed(T + F)
    bf = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    x, w1, dy, wd = bf(T, H), bf(H, 2 * F) * 0.05, bf(T, H), bf(F, H) * 0.05
    wsb = max(dh.dh_gemm_workspace_bytes(dh.DH_BF16, 0, 0, T, 2 * F, H), dh.dh_gemm_workspace_bytes(dh.DH_BF16, 0, 1, T, F, H))
    ws = torch.empty(max(wsb, 16), dtype=torch.uint8, device="cuda")
    gu, a, da, dgu = (torch.zeros(T, n, dtype=torch.bfloat16, device="cuda") for n in (2 * F, F, F, 2 * F))
    dh.dh_gemm(dh.DH_BF16, 0, 0, T, 2 * F, H, x, w1, gu, False, ws, wsb)
    dh.dh_swiglu_fwd(dh.DH_BF16, T, F, gu, a)
    dh.dh_gemm(dh.DH_BF16, 0, 1, T, F, H, dy, wd, da, False, ws, wsb)
    dh.dh_swiglu_bwd(dh.DH_BF16, T, F, gu, da, dgu)
    if dh.dh_gemm_swiglu_fwd_fits(T, F, H):
        gu1, a1 = (torch.full((T * n + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for n in (2 * F, F))
        dh.dh_gemm_swiglu_fwd(T, F, H, x, w1, gu1, a1)
        assert torch.equal(gu1[:-64].view_as(gu), gu) and torch.equal(a1[:-64].view_as(a), a)
        assert torch.all(gu1[-64:] == 7.0) and torch.all(a1[-64:] == 7.0)
    if dh.dh_gemm_swiglu_bwd_fits(T, F, H):
        dgu1 = torch.full((T * 2 * F + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
        dh.dh_gemm_swiglu_bwd(T, F, H, dy, wd, gu, dgu1)
        assert torch.equal(dgu1[:-64].view_as(dgu), dgu) and torch.all(dgu1[-64:] == 7.0)


# Norms and residual adds that take in the reduction in front of them (stand-ins that may use the whole chip) against the
# separate operators (stand-ins on a block budget): one to sixteen partials, one to eight vectors a thread, row remainders
@pytest.mark.parametrize("arch,ranks,seq,hidden", [("llama", 1, 33, 72), ("llama", 3, 513, 2056), ("llama", 8, 1030, 4104), ("llama", 16, 70, 8200),
                                                   ("gpt", 1, 33, 72), ("gpt", 2, 1026, 2056), ("gpt", 9, 63, 4104), ("gpt", 8, 64, 8200)])
@pytest.mark.parametrize("bf16", [True, False])
def test_reduction_with_its_consumer(dh, arch, ranks, seq, hidden, bf16):
    from paper_2411_15871_amd import harness as H
    run = H.LayerRun(dict(arch=arch, batch=1, seq=seq, hidden=hidden, nq=2, nkv=1, d=64, ffn=72, n_ranks=ranks, bf16=bf16))
    try:
        got = []
        for blocks in (0, 5):
            dh.dh_layer_set_comm_blocks(run.layer, blocks)
            s = run.strand(0)
            s.saved.zero_()
            run.zero_grads()
            run.fwd(s)
            run.bwd(s)
            torch.cuda.synchronize()
            got.append([s.out.clone(), s.saved.clone(), s.dx.clone()] + [v.clone() for v in run.g.values()])
        for a, b in zip(*got):
            assert torch.equal(a, b)
    finally:
        run.close()


# bf16 attention backward: grouped heads (dQ kernel with two tile slots, rows split into chunks when few heads leave the chip
# idle, a last chunk of one tile, a last tile of one key) and one head per key/value head (one launch for dQ and dK/dV)
@pytest.mark.parametrize("seq,nq,nkv,d", [(64, 2, 1, 128), (65, 2, 1, 128), (129, 3, 3, 128), (1025, 2, 1, 128), (1600, 1, 1, 128),
                                          (1537, 2, 1, 64)])
def test_attention_bwd_tile_edges(dh, seq, nq, nkv, d):
    n = (nq + 2 * nkv) * d
    qkv, do = gen.normal(90, (seq, n), 1.0, 0.0, True), gen.normal(91, (seq, nq * d), 1.0, 0.0, True)
    qd, dod = (torch.from_numpy(v.astype(np.float32)).bfloat16().cuda() for v in (qkv, do))
    o, lse = torch.empty(seq, nq * d, dtype=torch.bfloat16, device="cuda"), torch.empty(nq, seq, device="cuda")
    dh.dh_attn_fwd(dh.DH_BF16, 1, seq, nq, nkv, d, qd, o, lse)
    size = dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, 1, seq, nq, nkv, d)
    ws = torch.empty(max(size, 16), dtype=torch.uint8, device="cuda")
    dqkv, delta = torch.zeros(seq, n, dtype=torch.bfloat16, device="cuda"), torch.empty(nq, seq, device="cuda")
    dh.dh_attn_bwd(dh.DH_BF16, 1, seq, nq, nkv, d, qd, o, dod, lse, dqkv, delta, ws, size)
    q, k, v = (qkv[:, a * d: b * d].astype(np.float64).reshape(seq, -1, d) for a, b in ((0, nq), (nq, nq + nkv), (nq + nkv, nq + 2 * nkv)))
    ref = R.attention_bwd(do.astype(np.float64).reshape(seq, nq, d), q, k, v, 1, seq)
    got = dqkv.float().cpu().numpy()
    # bf16 probabilities and score gradients (2^-9 each) and a bf16 result: below 1e-2 in the norm, as for the other sizes
    for part, want in zip((got[:, : nq * d], got[:, nq * d: (nq + nkv) * d], got[:, (nq + nkv) * d:]), ref):
        assert rel(part, want.reshape(seq, -1)) <= 2e-2
