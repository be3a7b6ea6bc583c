"""Float32: SwiGLU in the epilogues of the gate/up projection and of the down projection's data gradient, against the separate operators: the same bits.  Widths
that end inside a tile, K of one wave to all sixteen, one product's waves side by side or in turn, more blocks than one launch takes (the forward
activation stays apart then); the data gradient alone and paired with the weight gradient."""
import pytest
import torch

from paper_2411_15871_amd import dhelix as dh
from paper_2411_15871_amd import harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("arch", ["llama", "llama_cp"])
@pytest.mark.parametrize("T,hidden,ffn", [(1, 16, 8), (17, 32, 24), (128, 256, 688), (100, 272, 40), (130, 512, 520), (33, 1024, 104), (512, 64, 1000), (1040, 64, 528)])
def test_same_bits_as_separate(T, hidden, ffn, arch):
    print("case", T, hidden, ffn, arch, flush=True)
    cp = dict(cp_ranks=1, cp_rank=0) if arch == "llama_cp" else {}
    run = H.LayerRun(dict(arch=arch, batch=1, seq=T, hidden=hidden, nq=1, nkv=1, d=16, ffn=ffn, n_ranks=1, bf16=False, **cp))
    try:
        got = {}
        for mask in (3, 0):
            assert dh.dh_layer_set_fused_activation(run.layer, mask) == (mask if T * ffn <= 512 * 32 * 32 else mask & 2)
            s = run.strand(0)
            run.zero_grads()
            run.fwd(s)
            run.bwd(s)
            torch.cuda.synchronize()
            got[mask] = [s.out.clone(), s.dx.clone()] + [run.g[k].clone() for k in sorted(run.g)]
        for a, b in zip(got[3], got[0]):
            assert torch.equal(a, b)
            assert torch.isfinite(a).all() and float(a.abs().max()) > 0
    finally:
        run.close()
