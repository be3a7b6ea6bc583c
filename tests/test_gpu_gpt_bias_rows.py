"""Bias gradients of GPT layers whose sequence shard is summed in blocks of 8 rows while the whole sequence takes 32: the column-sum workspace holds
either (2048 to 4094 tokens over two ranks), against column sums of the same gradients in float64."""
import pytest
import torch

from paper_2411_15871_amd import harness as H

pytestmark = pytest.mark.gpu

SHAPES = [(2046, 2, 64, 64), (2048, 2, 256, 64), (4094, 2, 64, 72), (4096, 2, 64, 64), (3072, 3, 128, 64)]  # tokens, ranks, hidden, ffn


@pytest.mark.parametrize("T,ranks,hidden,ffn", SHAPES)
@pytest.mark.parametrize("bf16", [True, False])
def test_bias_gradients_of_the_shard(T, ranks, hidden, ffn, bf16):
    print("case", T, ranks, hidden, ffn, bf16, flush=True)
    run = H.LayerRun(dict(arch="gpt", batch=1, seq=T, hidden=hidden, nq=1, nkv=1, d=64, ffn=ffn, n_ranks=ranks, bf16=bf16))
    try:
        s = run.strand(0)
        run.fwd(s)
        run.bwd(s)
        torch.cuda.synchronize()
        want = s.dout.double().sum(0)   # the down projection's bias is added after the reduction: its gradient is the sum of dout's rows
        got = run.g["dbfc2"].double()
        # float32 sums of up to 2048 values: an addition is off by 2^-24 of the running sum at most
        assert torch.all((got - want).abs() <= 2048 * 2.0 ** -24 * s.dout.double().abs().sum(0))
        assert torch.isfinite(run.g["dbo"]).all() and float(run.g["dbo"].norm()) > 0
    finally:
        run.close()
