"""float32: a linear's data and weight gradient in one launch give the bits of the two launches, for each pair of tile sizes (16x16 tiles where
32x32 ones are few), shares of K of the two products that differ, sizes that fill no tile, biases, and experts of unequal size or none.
The reference is a backward pass with every weight gradient moved to its end, where each is a launch of its own."""
import pytest
import torch

from paper_2411_15871_amd import harness as H

pytestmark = pytest.mark.gpu

F32 = dict(n_ranks=1, bf16=False)
CASES = [dict(F32, arch="llama", batch=1, seq=5, hidden=520, nq=1, nkv=1, d=16, ffn=24),             # 16 waves for one product, 1 for the other
         dict(F32, arch="llama", batch=1, seq=33, hidden=1032, nq=2, nkv=1, d=64, ffn=520),          # small data gradient, large weight gradient
         dict(F32, arch="llama", batch=2, seq=520, hidden=264, nq=2, nkv=2, d=64, ffn=72),           # the other way round
         dict(F32, arch="llama", batch=1, seq=640, hidden=544, nq=4, nkv=2, d=64, ffn=608),          # both large
         dict(arch="gpt", batch=2, seq=64, hidden=136, nq=2, nkv=2, d=32, ffn=264, n_ranks=4, bf16=False),
         dict(F32, arch="moe", batch=1, seq=301, hidden=264, nq=2, nkv=2, d=64, ffn=136, n_experts=8, n_local=2),
         dict(F32, arch="moe", batch=1, seq=1, hidden=64, nq=2, nkv=2, d=16, ffn=72, n_experts=8, n_local=4)]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: "-".join(str(c[k]) for k in ("arch", "batch", "seq", "hidden", "ffn")))
def test_paired_f32_gradients(cfg):
    from paper_2411_15871_amd import dhelix as dh
    print("case", cfg, flush=True)
    run = H.LayerRun(cfg)
    try:
        a, b = run.strand(0), run.strand(1)
        run.fwd(b)
        run.bwd(b)
        torch.cuda.synchronize()
        want = [b.dx.clone()] + [g.clone() for g in run.g.values()]
        names = dh.op_names(H.ARCH[cfg["arch"]], 1)
        late = [i for i, n in enumerate(names) if n.endswith("WGRAD")]
        order = [i for i in range(len(names)) if i not in late] + late
        nf = dh.dh_layer_op_graph(run.layer, 0).n_ops
        plan = dh.make_plan(list(range(nf)), order, [(0, nf, 0, len(order))])
        sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        for t in [b.dx] + list(run.g.values()):
            t.zero_()
        torch.cuda.synchronize()
        run.si_step(a, b, plan, sa, sb)
        torch.cuda.synchronize()
        for got, ref in zip([b.dx] + list(run.g.values()), want):
            assert torch.isfinite(ref).all() and torch.equal(got, ref)
    finally:
        run.close()
