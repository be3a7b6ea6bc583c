"""bf16 attention backward with grouped heads: a key block walks the query tiles of all heads of its group, cut into chunks that end
inside one head or at the border of two, whole chunks first and what is left of the blocks behind them."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dh():
    from paper_2411_15871_amd import dhelix
    assert torch.cuda.is_available()
    return dhelix


def reference(q, k, v, do, q_off):
    """Causal attention of one head group in float64: q, do [heads, queries, d], k, v [keys, d]; query i sits at position q_off + i."""
    d = q.shape[-1]
    s = torch.matmul(q, k.t()) / d ** 0.5
    pos = torch.arange(k.shape[0], device=q.device)
    s.masked_fill_(pos[None, None, :] > (q_off + torch.arange(q.shape[1], device=q.device))[None, :, None], float("-inf"))
    p = torch.softmax(s, -1)
    dp = torch.matmul(do, v.t())
    ds = p * (dp - (p * dp).sum(-1, keepdim=True)) / d ** 0.5
    dv = sum(torch.matmul(p[h].t().contiguous(), do[h]) for h in range(q.shape[0]))
    dk = sum(torch.matmul(ds[h].t().contiguous(), q[h]) for h in range(q.shape[0]))
    return torch.matmul(ds, k), dk, dv


# one block of one tile, blocks of a single chunk (no partial results), many chunks a block, a ragged last tile in every head, groups of 2 to
# 16 heads, several sequences, queries behind a key buffer, more than 64 blocks (two to a lane of the unit search), both head widths; chunks of two
# tiles; equal heads behind a key buffer: rows cut and columns whole, both cut
@pytest.mark.parametrize("batch,seq,q_off,nq,nkv,d", [(1, 40, 0, 2, 1, 128), (2, 130, 0, 8, 2, 128), (1, 300, 0, 16, 1, 128), (3, 257, 0, 4, 1, 64),
                                                      (1, 1500, 0, 16, 4, 128), (2, 1000, 0, 32, 4, 64), (1, 700, 1152, 4, 1, 128), (2, 333, 256, 6, 3, 64),
                                                      (1, 8300, 0, 2, 1, 64), (1, 2000, 0, 3, 3, 128), (1, 224, 0, 4, 2, 128), (1, 145, 0, 32, 8, 64),
                                                      (1, 189, 7808, 4, 4, 128), (4, 187, 2048, 1, 1, 64), (1, 1231, 3840, 2, 2, 128)])
def test_grouped_attention_backward(dh, batch, seq, q_off, nq, nkv, d):
    print("case", batch, seq, q_off, nq, nkv, d, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seq + nq)
    T, S, grp = batch * seq, q_off + seq, nq // nkv

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda").bfloat16()

    qkv, kv, do = normal(T, (nq + 2 * nkv) * d), normal(batch * S, 2 * nkv * d), normal(T, nq * d)
    o, lse, delta = torch.empty_like(do), torch.empty(nq, T, device="cuda"), torch.empty(nq, T, device="cuda")
    n = dh.dh_attn_ctx_fwd_workspace_bytes(dh.DH_BF16, batch, seq, q_off, nq, nkv, d)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    dh.dh_attn_ctx_fwd(dh.DH_BF16, batch, seq, q_off, nq, nkv, d, qkv, kv, o, lse, ws, n)
    n = dh.dh_attn_ctx_bwd_workspace_bytes(dh.DH_BF16, batch, seq, q_off, nq, nkv, d)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    got = []
    for _ in range(2):
        dqkv, dkv = torch.full_like(qkv, 3.0), torch.full_like(kv, 3.0)
        dh.dh_attn_ctx_bwd(dh.DH_BF16, batch, seq, q_off, nq, nkv, d, qkv, kv, o, do, lse, dqkv, dkv, delta, ws, n)
        got.append((dqkv, dkv))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])  # fixed order of every sum
    # bf16 probabilities and score gradients (2^-9 each) and a bf16 result: below 1e-2 in the norm
    for b in range(batch):
        rows, keys = slice(b * seq, (b + 1) * seq), slice(b * S, (b + 1) * S)
        q = qkv[rows, : nq * d].double().view(seq, nq, d).transpose(0, 1).contiguous()
        g = do[rows].double().view(seq, nq, d).transpose(0, 1).contiguous()
        k, v = (kv[keys].double().view(S, 2, nkv, d)[:, i] for i in (0, 1))
        for h in range(nkv):
            own = slice(h * grp, (h + 1) * grp)
            want = reference(q[own], k[:, h].contiguous(), v[:, h].contiguous(), g[own], q_off)
            dq = dqkv[rows, : nq * d].double().view(seq, nq, d).transpose(0, 1)[own]
            dk, dv = (dkv[keys].double().view(S, 2, nkv, d)[:, i, h] for i in (0, 1))
            for x, y in zip((dq, dk, dv), want):
                assert float((x - y).norm()) <= 1e-2 * float(y.norm())
