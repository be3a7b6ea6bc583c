"""bf16 attention backward, D = 128: the dK/dV loop publishes a tile ahead.  Units of one to five tiles (the ring has
three slots), whole and ragged last tiles, waves that see nothing of a head's first tile, heads that follow one another inside a unit."""
import pytest
import torch

from test_gpu_attn_chunks import dh, reference  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nkv", [(1, 1), (3, 1), (2, 2)])
@pytest.mark.parametrize("seq", [1, 63, 64, 65, 128, 129, 191, 192, 193, 256, 257, 320])
def test_unit_lengths(dh, seq, nq, nkv):  # noqa: F811
    print("case", seq, nq, nkv, flush=True)
    d, gen = 128, torch.Generator(device="cuda").manual_seed(seq)
    qkv = torch.randn(seq, (nq + 2 * nkv) * d, generator=gen, device="cuda").bfloat16()
    do = (torch.randn(seq, nq * d, generator=gen, device="cuda") + 1.0).bfloat16()  # a mean of its own: delta as large as dP
    o, lse, delta = torch.empty_like(do), torch.empty(nq, seq, device="cuda"), torch.empty(nq, seq, device="cuda")
    n = dh.dh_attn_fwd_workspace_bytes(dh.DH_BF16, 1, seq, nq, nkv, d)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    dh.dh_attn_fwd(dh.DH_BF16, 1, seq, nq, nkv, d, qkv, o, lse, ws, n)
    n = dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, 1, seq, nq, nkv, d)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    dqkv = torch.full_like(qkv, 3.0)
    dh.dh_attn_bwd(dh.DH_BF16, 1, seq, nq, nkv, d, qkv, o, do, lse, dqkv, delta, ws, n)
    torch.cuda.synchronize()
    heads = lambda t, n: t.double().view(seq, n, d).transpose(0, 1).contiguous()  # noqa: E731
    q, k, v = (heads(t, n) for t, n in zip(qkv.split([nq * d, nkv * d, nkv * d], 1), (nq, nkv, nkv)))
    dq, dk, dv = (heads(t, n) for t, n in zip(dqkv.split([nq * d, nkv * d, nkv * d], 1), (nq, nkv, nkv)))
    g, grp = heads(do, nq), nq // nkv
    for h in range(nkv):
        own = slice(h * grp, (h + 1) * grp)
        want = reference(q[own], k[h], v[h], g[own], 0)
        # bf16 probabilities, score gradients and results (2^-9 each) and delta from a bf16 output: a query that sees one key has a score gradient of
        # exactly zero, where delta's 2^-9 of dP remains, so the score gradients' share is measured against the scale of dV
        for x, y in zip((dq[own], dk[h], dv[h]), want):
            assert float((x - y).norm()) <= 1e-2 * float(max(y.norm(), want[2].norm() / d ** 0.5))
