"""The router's gradient from one token to more elements than a launch has threads, against the softmax's derivative in float64: every element is
written, those of experts not kept with zero."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# one element short of, at and past the grid's own limit (2^20 blocks of 256 threads); 2^32 elements, 16 GiB
@pytest.mark.parametrize("T,E", [(1, 2), (1500, 16), (257, 255), ((1 << 20) - 1, 256), (1 << 20, 256), ((1 << 20) + 3, 256), (1 << 24, 256)])
def test_router_gradient_of_every_size(T, E):
    from paper_2411_15871_amd import dhelix as dh
    print("case", T, E, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + E)
    first = torch.randint(0, E, (T,), generator=g, device="cuda")
    idx = torch.stack([first, (first + torch.randint(1, E, (T,), generator=g, device="cuda")) % E], dim=1).int().contiguous()
    p0 = torch.rand(T, generator=g, device="cuda")
    prob = torch.stack([p0, 1 - p0], dim=1).contiguous()
    dprob = torch.randn(T, 2, generator=g, device="cuda")
    out = torch.full((T, E), float("nan"), device="cuda")
    dh.dh_moe_route_bwd(T, E, dprob, idx, prob, out)
    torch.cuda.synchronize()
    step = 1 << 20
    for t0 in range(0, T, step):
        p, dp, i = (v[t0: t0 + step] for v in (prob.double(), dprob.double(), idx.long()))
        kept = p * (dp - (p * dp).sum(1, keepdim=True))
        want = torch.zeros(len(p), E, device="cuda", dtype=torch.float32).scatter_(1, i, kept.float())
        # p * (g - s) of values below 8 in float32: a few roundings of 2^-24 each
        assert torch.all((out[t0: t0 + step] - want).abs() <= 4e-6)  # a NaN left over fails it
