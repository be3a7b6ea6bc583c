"""bf16 attention backward: a score gradient P (dP - delta) takes the whole sum dP first and delta from it, in the dQ and the dK/dV loops and at both head
widths alike.  With K = 0 and zero log sums P is 1; dP is 2^22 + 1/2 (1/8 from each of the first four 16-wide steps, the large term in the last) and
delta 2^22, both exact, so every score gradient is exactly 1/2.  A sum that starts from delta loses the eighths."""
import pytest
import torch

from test_gpu_attn_chunks import dh  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("seq,nq,nkv", [(1, 1, 1), (64, 2, 1), (65, 1, 1), (200, 4, 2), (256, 3, 1), (333, 2, 2)])
def test_delta_is_subtracted_from_the_whole_sum(dh, seq, nq, nkv, d):  # noqa: F811
    print("case", seq, nq, nkv, d, flush=True)
    ones = torch.ones(seq, 1, device="cuda")
    do, v, o = (torch.zeros(seq, d, device="cuda") for _ in range(3))
    first = [0, 16, 32, 40] if d == 64 else [0, 16, 32, 48]  # the last step's columns hold the large term alone
    do[:, first], v[:, first] = 1.0, 0.125
    do[:, d - 1], v[:, d - 1], o[:, d - 1] = 2.0 ** 11, 2.0 ** 11, 2.0 ** 11
    do, o = do.repeat(1, nq).bfloat16(), o.repeat(1, nq).bfloat16()
    qkv = torch.cat([ones.expand(seq, nq * d), torch.zeros(seq, nkv * d, device="cuda"), v.repeat(1, nkv)], 1).bfloat16().contiguous()
    lse, delta, dqkv = torch.zeros(nq, seq, device="cuda"), torch.empty(nq, seq, device="cuda"), torch.full_like(qkv, 3.0)
    n = dh.dh_attn_bwd_workspace_bytes(dh.DH_BF16, 1, seq, nq, nkv, d)
    ws = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda")
    dh.dh_attn_bwd(dh.DH_BF16, 1, seq, nq, nkv, d, qkv, o, do, lse, dqkv, delta, ws, n)
    torch.cuda.synchronize()
    dk = dqkv[:, nq * d:(nq + nkv) * d].float()
    # key j: the sum of 1/2 * q (= 1) over the group's heads and the queries from j on, exact in float32, scaled and rounded to bf16 once
    want = 0.5 * (nq // nkv) * (seq - torch.arange(seq, device="cuda", dtype=torch.float32))[:, None] * (1.0 / d ** 0.5)
    assert float((dk / want - 1).abs().max()) <= 2.0 ** -8
    assert not dqkv[:, :nq * d].any()  # K is zero
