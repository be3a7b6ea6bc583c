"""Column sums at the edges of the one-launch kernel: remainders of its 256 row lanes, 8 rows in flight and 32 columns, and both sides of the
limits of rows and elements beyond which partial rows are written first."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("T,N", [(1, 32), (255, 40), (256, 8), (257, 24), (2047, 72), (2048, 4096), (2048, 4104), (2049, 72)])
def test_colsum_edges(bf16, T, N):
    from paper_2411_15871_amd import dhelix as dh
    gen = torch.Generator(device="cuda").manual_seed(T * 7 + N)
    x = torch.randn(T, N, device="cuda", generator=gen).to(torch.bfloat16 if bf16 else torch.float32)
    out = torch.full((N + 8,), 0.5, device="cuda")
    wsb = dh.dh_colsum_ws_bytes(T, N)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    dh.dh_colsum(dh.DH_BF16 if bf16 else dh.DH_F32, T, N, x, out, ws, wsb)
    torch.cuda.synchronize()
    got, xs = out.double().cpu().numpy(), x.double().cpu().numpy()
    assert np.all(got[N:] == 0.5)
    # float32 sums: at most T/256 + 4 + 16 + 1 additions one after the other in the one-launch kernel, T/32 + 32 with partial rows, each within 2^-24 of
    # a partial sum that the sum of magnitudes bounds
    bound = (T / 32 + 40) * 2.0 ** -24 * (np.abs(xs).sum(axis=0) + 0.5)
    assert np.all(np.abs(got[:N] - 0.5 - xs.sum(axis=0)) <= bound)
