"""bf16 attention forward, D = 128: the pipelined loop (units of ten and more key tiles) forms a tile's scores an iteration ahead.  Even and odd tile
counts, whole and ragged last tiles, waves that stop a tile before the others, reference maxima that move late; long rows cut into chunks of ten tiles and more,
whose units begin behind the first key, end below the diagonal and leave float32 partial results."""
import math

import pytest
import torch

from test_gpu_attn_chunks import dh  # noqa: F401

pytestmark = pytest.mark.gpu
D = 128


def reference(q, k, v, q_off):
    """[heads, queries, D] of one key/value head in float64: output and log sums."""
    s = q @ k.t() / math.sqrt(D)
    s = s.masked_fill(torch.arange(k.shape[0], device=k.device)[None, :] > q_off + torch.arange(q.shape[1], device=k.device)[:, None], -math.inf)
    return torch.softmax(s, -1) @ v, torch.logsumexp(s, -1)


def inputs(batch, seq, q_off, nq, nkv, growth):
    gen, keys, T = torch.Generator(device="cuda").manual_seed(seq), q_off + seq, batch * seq
    qkv = torch.randn(T, (nq + 2 * nkv) * D, generator=gen, device="cuda")
    kv = torch.randn(batch * keys, 2 * nkv * D, generator=gen, device="cuda")
    # later keys longer along a direction all queries share: a row's reference maximum moves again and again
    ramp = growth * torch.linspace(0, 1, keys, device="cuda").repeat(batch)[:, None] * torch.ones(D, device="cuda") / D ** 0.5
    qkv[:, :nq * D] += 2.0 if growth else 0.0
    kv[:, :nkv * D] += ramp.repeat(1, nkv)
    qkv, kv = qkv.bfloat16(), kv.bfloat16()
    if q_off == 0:
        qkv[:, nq * D:] = kv
    return qkv, kv


def forward(dh, batch, seq, q_off, nq, nkv, qkv, kv, workspace):  # noqa: F811
    """Output, log sums and the bytes of workspace that were there to use."""
    T = batch * seq
    o, lse = torch.full((T, nq * D), 7.0, device="cuda").bfloat16(), torch.zeros(nq, T, device="cuda")
    if q_off == 0:
        n = dh.dh_attn_fwd_workspace_bytes(dh.DH_BF16, batch, seq, nq, nkv, D) if workspace else 0
        ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
        dh.dh_attn_fwd(dh.DH_BF16, batch, seq, nq, nkv, D, qkv, o, lse, ws if n else None, n)
    else:
        n = dh.dh_attn_ctx_fwd_workspace_bytes(dh.DH_BF16, batch, seq, q_off, nq, nkv, D) if workspace else 0
        ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
        dh.dh_attn_ctx_fwd(dh.DH_BF16, batch, seq, q_off, nq, nkv, D, qkv, kv, o, lse, ws if n else None, n)
    torch.cuda.synchronize()
    return o, lse, n


def check(batch, seq, q_off, nq, nkv, qkv, kv, o, lse):
    keys = q_off + seq
    q = qkv[:, :nq * D].double().view(batch, seq, nq, D).permute(0, 2, 1, 3)
    k = kv[:, :nkv * D].double().view(batch, keys, nkv, D).permute(0, 2, 1, 3)
    v = kv[:, nkv * D:].double().view(batch, keys, nkv, D).permute(0, 2, 1, 3)
    got = o.double().view(batch, seq, nq, D).permute(0, 2, 1, 3)
    for b in range(batch):
        for h in range(nkv):
            own = slice(h * (nq // nkv), (h + 1) * (nq // nkv))
            want, want_lse = reference(q[b, own], k[b, h], v[b, h], q_off)
            # probabilities and outputs are bf16 (2^-9 each); a score's float32 sum of 128 products is off by at most 128 * 2^-24 of its terms (300)
            assert float((got[b, own] - want).norm()) <= 1e-2 * float(want.norm())
            rows = lse[own, b * seq:(b + 1) * seq].double()
            assert float((rows - want_lse).abs().max()) <= 3e-3
            assert float(((got[b, own] - want).norm(dim=-1) / want.norm(dim=-1)).max()) <= 2e-2


@pytest.mark.parametrize("growth", [0.0, 40.0])
@pytest.mark.parametrize("workspace", [False, True])
@pytest.mark.parametrize("batch,seq,q_off,nq,nkv", [
    (1, 577, 0, 2, 2), (1, 608, 0, 1, 1), (2, 640, 0, 2, 1), (1, 641, 0, 3, 1), (1, 672, 0, 1, 1), (1, 703, 0, 2, 2), (1, 704, 0, 1, 1), (3, 705, 0, 2, 1),
    (1, 768, 0, 1, 1), (1, 1290, 0, 4, 1), (1, 1, 640, 2, 1), (2, 100, 640, 4, 2), (1, 333, 1152, 2, 2), (1, 256, 2048, 4, 1)])
def test_pipelined_forward(dh, batch, seq, q_off, nq, nkv, workspace, growth):  # noqa: F811
    print("case", batch, seq, q_off, nq, nkv, workspace, growth, flush=True)
    qkv, kv = inputs(batch, seq, q_off, nq, nkv, growth)
    o, lse, _ = forward(dh, batch, seq, q_off, nq, nkv, qkv, kv, workspace)
    check(batch, seq, q_off, nq, nkv, qkv, kv, o, lse)


def chunk_of(batch, seq, q_off, nq, n):
    """Tiles a chunk of a launch whose workspace holds n bytes: the even length that makes its number of units (128 rows of D + 2 floats each)."""
    units, tiles = n // (batch * nq * 128 * (D + 2) * 4), [-(-min((i + 1) * 128, q_off + seq) // 64) for i in range(q_off // 128, -(-(q_off + seq) // 128))]
    fits = [c for c in range(2, max(tiles), 2) if sum(-(-t // c) for t in tiles) == units]
    assert len(fits) == 1
    return fits[0]


@pytest.mark.parametrize("growth", [0.0, 40.0])
@pytest.mark.parametrize("batch,seq,q_off,nq,nkv,chunk", [
    (1, 4096, 0, 4, 1, 10), (1, 4033, 0, 4, 1, 10), (1, 3905, 0, 4, 2, 10), (2, 4001, 0, 2, 1, 10), (1, 5057, 0, 4, 1, 16), (1, 2048, 2048, 8, 8, 14),
    (1, 2017, 2048, 8, 2, 14), (1, 1000, 7808, 4, 1, 10)])
def test_cut_rows(dh, batch, seq, q_off, nq, nkv, chunk, growth):  # noqa: F811
    print("case", batch, seq, q_off, nq, nkv, growth, flush=True)
    qkv, kv = inputs(batch, seq, q_off, nq, nkv, growth)
    o, lse, n = forward(dh, batch, seq, q_off, nq, nkv, qkv, kv, True)
    assert chunk_of(batch, seq, q_off, nq, n) == chunk  # ten tiles and more: the pipelined loop takes them
    check(batch, seq, q_off, nq, nkv, qkv, kv, o, lse)
    whole, whole_lse, _ = forward(dh, batch, seq, q_off, nq, nkv, qkv, kv, False)
    # probabilities against another reference maximum and the result are rounded to bf16 once each; float32 sums of up to 8808 terms
    assert float((o.double() - whole.double()).norm()) <= 2.0 ** -7 * float(whole.double().norm())
    assert float((lse - whole_lse).abs().max()) <= 8808 * 2.0 ** -24
