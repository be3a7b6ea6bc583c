"""Grouped products whose remainder rows go to a second launch: few of them (64x64 tiles) and many (128x128 tiles), with remainders of one row, of a tile
and a row, of a large tile less one row, and none."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n", [([2049, 2048], 4096), ([2113, 1983], 4096), ([2303, 1793], 4096), ([1025, 1279, 1024, 1024], 4096), ([4160], 4096)])
def test_grouped_remainders(rows, n):
    from paper_2411_15871_amd import dhelix as dh
    print("case", rows, n, flush=True)
    k, G, tot = 4096, len(rows), sum(rows)
    g = torch.Generator(device="cuda").manual_seed(tot)
    bf = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    x, W, Wt = bf(tot, k), bf(G, k, n), bf(G, n, k)
    rd = torch.tensor(rows, dtype=torch.int32, device="cuda")
    c, d = (torch.full((tot + 1, n), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    dh.dh_gemm_grouped(dh.DH_BF16, 0, G, rd, tot, k, n, x, W, c)
    dh.dh_gemm_grouped(dh.DH_BF16, 1, G, rd, tot, n, k, x, Wt, d)
    torch.cuda.synchronize()
    assert torch.all(c[tot] == 7.0) and torch.all(d[tot] == 7.0)
    r0 = 0
    for i, r in enumerate(rows):
        xs = x[r0: r0 + r].float()
        for got, w in ((c, W[i].float()), (d, Wt[i].float().t().contiguous())):
            ref = xs @ w
            err = (got[r0: r0 + r].float() - ref).norm(dim=1) / ref.norm(dim=1)
            assert float(err.max()) <= 4e-3  # per row: a rounding of 2^-9 an element
        r0 += r


# A remainder's rows have the bits they have as part of a group that ends with a whole large tile: neither the launch nor its tile shape
# (64x64 where remainders are few, else 128x128) shows in them.
@pytest.mark.parametrize("rows", [[2049, 2048], [2113, 1983], [1025, 1279, 1024, 1024]])
def test_remainder_rows_have_the_bits_of_whole_tiles(rows):
    from paper_2411_15871_amd import dhelix as dh
    print("case", rows, flush=True)
    n, k, G = 4096, 4096, len(rows)
    whole = [-(-r // 256) * 256 for r in rows]
    g = torch.Generator(device="cuda").manual_seed(sum(rows))
    bf = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    xs, W = [bf(w, k) for w in whole], bf(G, k, n)
    outs = []
    for counts in (rows, whole):
        x, tot = torch.cat([v[:r] for v, r in zip(xs, counts)]).contiguous(), sum(counts)
        c = torch.full((tot, n), 7.0, dtype=torch.bfloat16, device="cuda")
        dh.dh_gemm_grouped(dh.DH_BF16, 0, G, torch.tensor(counts, dtype=torch.int32, device="cuda"), tot, k, n, x, W, c)
        outs.append(torch.split(c, counts))
    torch.cuda.synchronize()
    for few, all_, r in zip(*outs, rows):
        assert torch.equal(few, all_[:r])
