"""RoPE with several heads a thread against one head at a time: the same bits, for head counts that fill no group of four, both pairings and types, on both
sides of the thread count from which a thread takes four heads; what lies behind the rotated heads of a row stays."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("adjacent", [False, True])
@pytest.mark.parametrize("T,heads,d", [(2341, 7, 128), (2340, 7, 128), (16384, 1, 128), (5500, 6, 64), (9, 5, 16), (3300, 5, 256)])
def test_heads_at_once_match_heads_apart(bf16, adjacent, T, heads, d):
    from paper_2411_15871_amd import dhelix as dh
    dt, pair = (dh.DH_BF16 if bf16 else dh.DH_F32), (dh.DH_ROPE_ADJACENT if adjacent else dh.DH_ROPE_HALVES)
    seq = T // 3 + 1
    g = torch.Generator(device="cuda").manual_seed(T + heads)
    x = torch.randn(T, heads + 2, d, device="cuda", generator=g).to(torch.bfloat16 if bf16 else torch.float32)
    for inverse in (0, 1):
        both, apart = x.clone(), x.clone()
        dh.dh_rope_pairs(dt, pair, T, seq, 11, heads, d, (heads + 2) * d, 10000.0, inverse, both)
        n = max(1, (1 << 16) // d)                      # rows at a time, a head at a time: far below the limit
        for h in range(heads):
            col = x[:, h].contiguous()
            for s in range(0, T, seq):                  # each sequence starts at the same position
                for r in range(s, min(T, s + seq), n):
                    k = min(n, T - r, s + seq - r)
                    dh.dh_rope_pairs(dt, pair, k, seq, 11 + r - s, 1, d, d, 10000.0, inverse, col[r:r + k])
            apart[:, h] = col
        torch.cuda.synchronize()
        assert torch.equal(both, apart)
        assert torch.equal(both[:, heads:], x[:, heads:])
