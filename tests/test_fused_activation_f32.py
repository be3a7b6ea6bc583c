"""Float32 layers report, and leave to a plan, exactly the activations that one launch does not take along: the forward one up to 512 blocks of the gate/up
projection, the backward one at any size.  Host only, no GPU needed."""
import pytest

from paper_2411_15871_amd import dhelix as dh


@pytest.mark.parametrize("arch", [dh.DH_ARCH_LLAMA, dh.DH_ARCH_LLAMA_CP, dh.DH_ARCH_GPT])
@pytest.mark.parametrize("T,ffn,fits", [(1, 8, True), (128, 688, True), (1024, 512, True), (1025, 512, False), (1024, 520, False), (1040, 528, False), (8192, 1024, False)])
def test_only_one_launch_is_called_fused(T, ffn, fits, arch):
    cp = dict(cp_ranks=1, cp_rank=0) if arch == dh.DH_ARCH_LLAMA_CP else {}
    layer = dh.dh_layer_create(arch=arch, dtype=dh.DH_F32, batch=1, seq=T, hidden=64, n_q_heads=1, n_kv_heads=1, head_dim=16, ffn=ffn, eps=1e-5, rope_base=1e4,
                               n_ranks=1, **cp)
    try:
        for mask in (3, 2, 1, 0):
            want = 0 if arch == dh.DH_ARCH_GPT else mask & (3 if fits else 2)
            assert dh.dh_layer_set_fused_activation(layer, mask) == want
    finally:
        dh.dh_layer_destroy(layer)
