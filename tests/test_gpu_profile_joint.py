"""The profiler's entries for the operators that an SI step issues as one launch (a linear's data and weight gradient): which they are, that their
times and rates are measured, and that the planners take the table."""
import math

import pytest
import torch

from oracle import plan_ref as P
from paper_2411_15871_amd import harness as H

pytestmark = pytest.mark.gpu

CASES = {
    "llama_bf16": dict(arch="llama", batch=1, seq=1024, hidden=1024, nq=4, nkv=1, d=128, ffn=1408, n_ranks=4, bf16=True),
    "gpt_bf16": dict(arch="gpt", batch=2, seq=264, hidden=520, nq=4, nkv=4, d=128, ffn=1000, n_ranks=4, bf16=True),
    "moe_bf16": dict(arch="moe", batch=1, seq=700, hidden=1024, nq=8, nkv=2, d=128, ffn=768, n_ranks=1, bf16=True, n_experts=8, n_local=2),
    "llama_f32": dict(arch="llama", batch=1, seq=128, hidden=256, nq=4, nkv=4, d=64, ffn=688, n_ranks=2, bf16=False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_joint_entries(name):
    from paper_2411_15871_amd import dhelix as dh
    run = H.LayerRun(CASES[name])
    try:
        alpha, beta = run.strand(0), run.strand(1)
        sa, sb, comm = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        run.fwd(alpha); run.fwd(beta); run.bwd(beta)
        torch.cuda.synchronize()
        print("case", name, flush=True)
        profile = lambda: dh.dh_profile_pairs(run.layer, alpha.fwd_args, beta.bwd_args, run.ws, run.ws_bytes, sa, sb, comm, 3)
        t = profile()
        names = dh.op_names(H.ARCH[run.cfg["arch"]], 1)
        joint = {names[j]: names[t.joint[j] - 1] for j in range(t.n_bwd) if t.joint[j]}
        print({k: round(t.t_joint[names.index(k)] * 1e6, 1) for k in joint}, flush=True)
        assert joint and all(k.endswith("_DGRAD") and v == k.replace("_DGRAD", "_WGRAD") for k, v in joint.items())
        for k, v in joint.items():
            j, w = names.index(k), names.index(v)
            # both products' work is in it; a launch that holds both is there because it is expected to take less than the two
            assert math.isfinite(t.t_joint[j]) and 0.5 * max(t.t_bwd[j], t.t_bwd[w]) <= t.t_joint[j] <= 1.5 * (t.t_bwd[j] + t.t_bwd[w])
            for i in range(t.n_fwd):
                assert 0.02 <= t.rate_fwd_joint[i][j] <= 1.0 and 0.02 <= t.rate_bwd_joint[i][j] <= 1.0
                one = P.segment_cost([0], [0], [t.t_fwd[i]], [t.t_joint[j]], [[t.rate_fwd_joint[i][j]]], [[t.rate_bwd_joint[i][j]]])
                assert abs(dh.dh_segment_cost(t, [i], [j, w]) - one) <= 1e-12
        gf, gb = dh.dh_layer_op_graph(run.layer, 0), dh.dh_layer_op_graph(run.layer, 1)
        plan, predicted, _ = dh.dh_plan_search_lanes(gf, gb, t, dh.lanes(0, 0, 0), 0.0, 200)
        assert abs(dh.dh_plan_cost(gf, gb, t, plan, dh.lanes(0, 0, 0), 0.0) - predicted) <= 1e-9 * predicted
        if name == "llama_bf16":  # weight gradients that ride in an all-reduce's launch are in no other
            dh.dh_layer_set_comm_blocks(run.layer, 8)
            mask = dh.dh_layer_set_fused_collective(run.layer, 3)
            t = profile()
            for bit, op in ((1, "B_FC1_DGRAD"), (2, "B_QKV_DGRAD")):
                assert mask & bit and t.joint[names.index(op)] == 0
    finally:
        run.close()
