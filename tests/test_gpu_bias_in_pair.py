"""Bias gradients that ride in the launch of a linear's two gradient products: the bits of dh_colsum.  Widths that end inside a block of 32 columns, row counts
around the 256 row lanes and at the limit of one launch, small layers (carried) and ones whose tiles fill the units (not carried)."""
import pytest
import torch

from paper_2411_15871_amd import dhelix as dh
from paper_2411_15871_amd import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,hidden,ffn", [(1, 64, 72), (63, 72, 64), (255, 40, 200), (256, 64, 64), (257, 520, 1000), (528, 520, 1000), (2047, 104, 136),
                                          (2048, 64, 256), (2049, 64, 256), (1024, 2048, 2056)])
def test_bias_gradient_bits(T, hidden, ffn):
    print("case", T, hidden, ffn, flush=True)
    run = H.LayerRun(dict(arch="gpt", batch=1, seq=T, hidden=hidden, nq=1, nkv=1, d=64, ffn=ffn, n_ranks=1, bf16=True))
    try:
        s = run.strand(0)
        run.fwd(s)
        run.bwd(s)
        torch.cuda.synchronize()
        n = dh.lib.dh_colsum_ws_bytes(T, hidden)
        ws, want = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda"), torch.zeros(hidden, device="cuda")
        assert dh.lib.dh_colsum(dh.DH_BF16, T, hidden, s.dout.data_ptr(), want.data_ptr(), ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        assert torch.equal(run.g["dbfc2"], want)
        for name, t in run.g.items():
            assert torch.isfinite(t).all(), name
        # rows are summed once: a second pass doubles every bias gradient
        first = {k: run.g[k].clone() for k in ("dbfc1", "dbfc2", "dbo", "dbqkv")}
        run.bwd(s)
        torch.cuda.synchronize()
        for k, v in first.items():
            assert torch.equal(run.g[k], v + v), k
    finally:
        run.close()
