"""Norm backward of short rows, which groups of a block's threads take side by side: widths around 512 and 1024, row counts at the block sizes (1, 2, 4, 8 rows)
and ones that leave some groups without a row, against float64; the same rows where the norm adds the ranks' partial buffers itself, in layers."""
import pytest
import torch

from paper_2411_15871_amd import dhelix as dh
from paper_2411_15871_amd import harness
from test_gpu_layer import Worst, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("layer", [True, False])
@pytest.mark.parametrize("rows", [3, 513, 1025, 1030, 4096, 4101])
@pytest.mark.parametrize("H", [8, 504, 512, 520, 1024, 1032])
def test_short_rows(H, rows, layer, bf16):
    print("case", H, rows, layer, bf16, flush=True)
    dt, code = (torch.bfloat16, dh.DH_BF16) if bf16 else (torch.float32, dh.DH_F32)
    gen = torch.Generator(device="cuda").manual_seed(H + rows)
    x, dy, res = (torch.randn(rows, H, generator=gen, device="cuda").to(dt) for _ in range(3))
    gamma = (1 + 0.1 * torch.randn(H, generator=gen, device="cuda")).to(dt)
    xd, dyd, gd = x.double(), dy.double(), gamma.double()
    mu = xd.mean(1, keepdim=True) if layer else torch.zeros(rows, 1, device="cuda", dtype=torch.float64)
    rstd = ((xd - mu).pow(2).mean(1, keepdim=True) + 1e-5).rsqrt()
    dx, dgamma, dbeta = torch.full_like(x, 5.0), torch.ones(H, device="cuda"), torch.ones(H, device="cuda")
    n = (dh.lib.dh_layernorm_bwd_ws_bytes if layer else dh.lib.dh_rmsnorm_bwd_ws_bytes)(rows, H)
    ws, st = torch.empty(max(n, 16), dtype=torch.uint8, device="cuda"), torch.cuda.current_stream().cuda_stream
    m32, r32 = mu.float().flatten().contiguous(), rstd.float().flatten().contiguous()
    p = [t.data_ptr() for t in (dy, x, gamma)]
    if layer:
        rc = dh.lib.dh_layernorm_bwd(code, rows, H, *p, m32.data_ptr(), r32.data_ptr(), res.data_ptr(), dx.data_ptr(), dgamma.data_ptr(), dbeta.data_ptr(),
                                     ws.data_ptr(), n, st)
    else:
        rc = dh.lib.dh_rmsnorm_bwd(code, rows, H, *p, r32.data_ptr(), res.data_ptr(), dx.data_ptr(), dgamma.data_ptr(), ws.data_ptr(), n, st)
    assert rc == 0
    torch.cuda.synchronize()
    xh, gh = (xd - mu) * rstd, gd * dyd
    want = rstd * (gh - xh * (gh * xh).mean(1, keepdim=True) - (gh.mean(1, keepdim=True) if layer else 0)) + res.double()
    # the result is stored once (2^-9 or 2^-24), sums of H and of `rows` float32 terms are off by less than 1e-5 of their terms
    assert float((dx.double() - want).norm()) <= (4e-3 if bf16 else 1e-5) * float(want.norm())
    assert float((dgamma.double() - 1 - (dyd * xh).sum(0)).abs().max()) <= 1e-5 * float((dyd * xh).abs().sum(0).max() + 1)
    if layer:
        assert float((dbeta.double() - 1 - dyd.sum(0)).abs().max()) <= 1e-5 * float(dyd.abs().sum(0).max() + 1)


# the rows of a norm: tokens, or a rank's share of them; four groups of threads a block, two, one, each with row counts that leave groups without a row
@pytest.mark.parametrize("bf16", [True, False])
@pytest.mark.parametrize("arch,tokens,ranks", [("llama", 1025, 2), ("llama", 1030, 8), ("gpt", 2058, 2)])
@pytest.mark.parametrize("hidden", [504, 520, 1024, 1032])
def test_partial_buffers(hidden, arch, tokens, ranks, bf16):
    print("case", hidden, arch, tokens, ranks, bf16, flush=True)
    got = []
    for blocks in (0, 64):  # the norm adds the buffers; a stand-in adds them ahead of it
        run = harness.LayerRun(dict(arch=arch, batch=1, seq=tokens, hidden=hidden, nq=1, nkv=1, d=64, ffn=64, n_ranks=ranks, bf16=bf16, comm_blocks=blocks))
        try:
            s = run.strand(0)
            run.fwd(s)
            run.bwd(s)
            torch.cuda.synchronize()
            names = ["dg1", "dg2"] + (["db1", "db2"] if arch == "gpt" else [])
            got.append([s.dx.clone()] + [run.g[n].clone() for n in names])
            if blocks == 0:
                _, dx, grads = oracle_run(run, s)
                tol, worst = (2e-2 if bf16 else 1e-5), Worst("norms", 2e-2 if bf16 else 1e-5)  # the bounds of the layer's oracle tests
                worst.check("dx", harness.to_np(s.dx), dx)
                for n in names:
                    err = abs(harness.to_np(run.g[n]) - grads[n]).max() / abs(grads[n]).max()
                    assert err <= tol, (n, err)
        finally:
            run.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
