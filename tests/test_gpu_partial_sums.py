"""Residual adds that take in a reduction, either side of the size from which a thread reads the partial buffers one after the other (2048 blocks of
256 threads, 8 elements each), with few and many ranks: the bits of the reduction and the add apart."""
import pytest
import torch

from paper_2411_15871_amd import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch,ranks,rows", [("llama", r, t) for r in (2, 4, 5, 8, 9, 12) for t in (1023, 1024)] + [("gpt", 4, 1023), ("gpt", 4, 1024)])
@pytest.mark.parametrize("bf16", [True, False])
def test_sums_ahead_and_one_by_one(arch, ranks, rows, bf16):
    from paper_2411_15871_amd import dhelix as dh
    print("case", arch, ranks, rows, bf16, flush=True)
    hidden = 4096  # rows * 4096 / 2048: two blocks a row
    run = H.LayerRun(dict(arch=arch, batch=1, seq=rows * (ranks if arch == "gpt" else 1), hidden=hidden, nq=1, nkv=1, d=64, ffn=64, n_ranks=ranks, bf16=bf16))
    try:
        got, s = [], run.strand(0)
        for blocks in (0, 64):
            dh.dh_layer_set_comm_blocks(run.layer, blocks)
            run.fwd(s)
            torch.cuda.synchronize()
            got.append(s.out.clone())
        assert torch.equal(*got)
    finally:
        run.close()
