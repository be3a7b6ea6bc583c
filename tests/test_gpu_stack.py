"""Several layers under SI on one GPU (forward sweep of one micro-batch co-run with the backward sweep of the
previous one, activations in the shared two-triangle arena) against the fp64 oracle applied layer by layer."""
import numpy as np
import pytest
import torch

from oracle import layer_ref as R
from paper_2411_15871_amd import harness as H
from paper_2411_15871_amd import inputs as gen

pytestmark = pytest.mark.gpu


def rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("bf16,n_layers,n_mb", [(False, 3, 3), (True, 4, 2), (False, 1, 2)])
def test_stack_phases_match_oracle(bf16, n_layers, n_mb):
    from paper_2411_15871_amd import dhelix as dh
    c = dict(batch=2, seq=75, hidden=136, nq=4, nkv=2, d=32, ffn=200, n_ranks=3) if not bf16 else \
        dict(batch=1, seq=330, hidden=264, nq=2, nkv=1, d=128, ffn=328, n_ranks=2)
    T, Hd, tol = c["batch"] * c["seq"], c["hidden"], (2e-2 if bf16 else 1e-5)
    n_qkv = (c["nq"] + 2 * c["nkv"]) * c["d"]
    cfgkw = dict(arch=dh.DH_ARCH_LLAMA, dtype=dh.DH_BF16 if bf16 else dh.DH_F32, batch=c["batch"], seq=c["seq"], hidden=Hd,
                 n_q_heads=c["nq"], n_kv_heads=c["nkv"], head_dim=c["d"], ffn=c["ffn"], eps=1e-5, rope_base=10000.0,
                 n_ranks=c["n_ranks"], comm_blocks=0, n_experts=0, n_local_experts=0)
    stack = dh.dh_stack_create(n_layers, **cfgkw)
    try:
        w_np = [gen.llama_weights(Hd, n_qkv, c["nq"] * c["d"], c["ffn"], bf16, seed=gen.SEED_WEIGHTS + 100 * l) for l in range(n_layers)]
        w = [{k: H.to_dev(v, bf16) for k, v in wl.items()} for wl in w_np]
        g = [{"d" + k: torch.zeros(v.shape, dtype=torch.float32, device="cuda") for k, v in wl.items()} for wl in w_np]
        for l in range(n_layers):
            dh.dh_layer_bind_weights(dh.dh_stack_layer(stack, l), **w[l])
            dh.dh_layer_bind_wgrads(dh.dh_stack_layer(stack, l), **g[l])
        n_peers = c["n_ranks"] - 1
        peers_np = {k: gen.peer_partials(300 + 10 * i, n_peers, T, Hd, bf16) for i, k in enumerate(("ar1", "ar2", "ar3", "ar4"))}
        peers = {k: H.to_dev(v, bf16) for k, v in peers_np.items()}
        xs_np = [gen.strand_input(m, T, Hd, bf16) for m in range(n_mb)]
        douts_np = [gen.strand_upstream_grad(m, T, Hd, bf16) for m in range(n_mb)]
        xs = [H.to_dev(a, bf16) for a in xs_np]; douts = [H.to_dev(a, bf16) for a in douts_np]
        outs = [torch.empty_like(xs[0]) for _ in range(n_mb)]; dxs = [torch.empty_like(xs[0]) for _ in range(n_mb)]
        arena_bytes, ws_bytes = dh.dh_stack_arena_bytes(stack), dh.dh_stack_workspace_bytes(stack)
        assert arena_bytes < dh.dh_stack_unshared_bytes(stack) or n_layers == 1
        arena = torch.empty(arena_bytes, dtype=torch.uint8, device="cuda"); ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
        sa, sb, sc = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        layer0 = dh.dh_stack_layer(stack, 0)
        gf, gb = dh.dh_layer_op_graph(layer0, 0), dh.dh_layer_op_graph(layer0, 1)
        plan = dh.make_plan(list(range(gf.n_ops)), list(range(gb.n_ops)), [(0, 5, 0, 6), (5, gf.n_ops, 6, gb.n_ops)])
        fwd = lambda m: (xs[m], outs[m], peers["ar1"], peers["ar2"])
        bwd = lambda m: (douts[m], dxs[m], peers["ar3"], peers["ar4"])
        with pytest.raises(dh.DhelixError):  # nothing to run backward yet
            dh.dh_stack_phase(stack, None, bwd(0), plan, arena, arena_bytes, ws, ws_bytes, sa, sb, sc)
        print("warm-up", flush=True)
        dh.dh_stack_phase(stack, fwd(0), None, None, arena, arena_bytes, ws, ws_bytes, sa, sb, sc)
        for m in range(1, n_mb):
            print("phase", m, flush=True)
            dh.dh_stack_phase(stack, fwd(m), bwd(m - 1), plan, arena, arena_bytes, ws, ws_bytes, sa, sb, sc)
        with pytest.raises(dh.DhelixError):  # the last micro-batch still waits for its backward
            dh.dh_stack_phase(stack, fwd(0), None, None, arena, arena_bytes, ws, ws_bytes, sa, sb, sc)
        print("cool-down", flush=True)
        dh.dh_stack_phase(stack, None, bwd(n_mb - 1), None, arena, arena_bytes, ws, ws_bytes, sa, sb, sc)
        torch.cuda.synchronize()
        # oracle, layer by layer
        cfg = R.LayerCfg(batch=c["batch"], seq=c["seq"], H=Hd, nq=c["nq"], nkv=c["nkv"], d=c["d"], F=c["ffn"])
        W = [{k: v.astype(np.float64) for k, v in wl.items()} for wl in w_np]
        gsum = [dict() for _ in range(n_layers)]
        for m in range(n_mb):
            h, saved = xs_np[m].astype(np.float64), []
            for l in range(n_layers):
                h, sv = R.llama_fwd(cfg, W[l], h, peers_np)
                saved.append(sv)
            assert rel(H.to_np(outs[m]), h) <= tol, ("out", m)
            d = douts_np[m].astype(np.float64)
            for l in reversed(range(n_layers)):
                d, gr, _ = R.llama_bwd(cfg, W[l], saved[l], d, peers_np)
                for k, v in gr.items():
                    gsum[l][k] = gsum[l].get(k, 0) + v
            assert rel(H.to_np(dxs[m]), d) <= tol, ("dx", m)
        for l in range(n_layers):
            for k, v in gsum[l].items():
                assert rel(H.to_np(g[l][k]), v) <= tol, (l, k)
    finally:
        dh.dh_stack_destroy(stack)


@pytest.mark.parametrize("blocks_alpha,blocks_beta", [(0, 0), (0, 64), (64, 0), (64, 64)])
def test_two_layers_place_their_own_collectives(blocks_alpha, blocks_beta):
    """dh_si_step_layers with unlike block budgets: results as from the two layers apart, bit for bit, and each strand's
    collectives on its communication stream exactly if its own layer's budget sends them there (a whole-chip reduction that
    its strand waits for stays).  Alpha's stream is kept busy first, so that a stream that got work still has it."""
    from paper_2411_15871_amd import dhelix as dh
    cfg = dict(batch=1, seq=1024, hidden=1024, nq=2, nkv=1, d=128, ffn=256, n_ranks=4, bf16=True)
    ra, rb = H.LayerRun(dict(cfg, comm_blocks=blocks_alpha)), H.LayerRun(dict(cfg, comm_blocks=blocks_beta))
    try:
        alpha, beta = ra.strand(0), rb.strand(1)
        sa, sb, sc, scb = (torch.cuda.Stream() for _ in range(4))
        dh.dh_layer_set_beta_comm_stream(ra.layer, scb)
        rb.fwd(beta)
        ra.fwd(alpha)
        rb.bwd(beta)
        torch.cuda.synchronize()
        ref = [alpha.out.clone(), beta.dx.clone()] + [v.clone() for v in rb.g.values()]
        alpha.out.zero_(); beta.dx.zero_(); rb.zero_grads()
        gf, gb = dh.dh_layer_op_graph(ra.layer, 0), dh.dh_layer_op_graph(rb.layer, 1)
        plan = dh.make_plan(list(range(gf.n_ops)), list(range(gb.n_ops)), [(0, gf.n_ops, 0, gb.n_ops)])
        torch.cuda.synchronize()
        with torch.cuda.stream(sa):
            torch.cuda._sleep(50_000_000)
        dh.dh_si_step_layers(ra.layer, rb.layer, alpha.fwd_args, beta.bwd_args, plan, ra.ws, ra.ws_bytes, sa, sb, sc)
        busy = (not sc.query(), not scb.query())
        assert not sa.query()
        torch.cuda.synchronize()
        assert busy == (blocks_alpha > 0, blocks_beta > 0)
        for got, want in zip([alpha.out, beta.dx] + list(rb.g.values()), ref):
            assert torch.equal(got, want)
    finally:
        ra.close()
        rb.close()


class _AddGrad(torch.autograd.Function):
    """Identity whose gradient has a constant added: what the other ranks contribute to a backward reduction."""

    @staticmethod
    def forward(ctx, x, extra):
        ctx.extra = extra
        return x.view_as(x)

    @staticmethod
    def backward(ctx, grad):
        return grad + ctx.extra, None


class _Stored(torch.autograd.Function):
    """A value, and its gradient, as they are after being stored in bf16."""

    @staticmethod
    def forward(ctx, x):
        return x.bfloat16().float()

    @staticmethod
    def backward(ctx, grad):
        return grad.bfloat16().float()


def _float32_layer(c, w, x, peers, st=lambda v: v):
    """The layer (one sequence) in plain float32 torch operations on the device, differentiable; st is applied to every tensor
    that the layer stores."""
    T, nq, nkv, d, F = c["seq"], c["nq"], c["nkv"], c["d"], c["ffn"]
    norm = lambda v, g: v * torch.rsqrt((v * v).mean(-1, keepdim=True) + 1e-5) * g
    qkv = st(_AddGrad.apply(st(norm(x, w["g1"])), peers["ar4"]) @ w["Wqkv"]).view(T, nq + 2 * nkv, d)
    ang = torch.arange(T, device=x.device, dtype=torch.float64)[:, None] * 10000.0 ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    cos, sin = ang.cos().float()[:, None], ang.sin().float()[:, None]
    a, b = qkv[:, : nq + nkv, : d // 2], qkv[:, : nq + nkv, d // 2:]
    rot = st(torch.cat([a * cos - b * sin, a * sin + b * cos], -1))
    future = torch.ones(T, T, dtype=torch.bool, device=x.device).triu(1)
    heads = []
    for h in range(nq):
        k, v = rot[:, nq + h * nkv // nq], qkv[:, nq + nkv + h * nkv // nq]
        heads.append(torch.softmax((rot[:, h] @ k.t().contiguous() / d ** 0.5).masked_fill(future, float("-inf")), -1) @ v)
    x2 = st(x + st(st(st(torch.cat(heads, -1)) @ w["Wo"]) + peers["ar1"]))
    gu = st(_AddGrad.apply(st(norm(x2, w["g2"])), peers["ar3"]) @ w["Wgu"])
    return st(x2 + st(st(st(torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]) @ w["Wd"]) + peers["ar2"]))


def test_stack_of_full_size_layers_against_float32():
    """Four layers of the Llama-8B shard under 8-way tensor parallelism, 4096 tokens: one steady-state phase against the same
    stack in float32.  What bf16 storage of the activations and their gradients costs in four layers is measured beside it,
    by the float32 stack with every stored tensor rounded (its products and sums stay float32): the errors are independent
    roundings in either case, so a result is at most a quarter further off than that."""
    from paper_2411_15871_amd import dhelix as dh
    c = H.CONFIGS["c2_llama8b_tp8"]
    assert c["batch"] == 1
    L, T, Hd, n_qkv = 4, c["seq"], c["hidden"], (c["nq"] + 2 * c["nkv"]) * c["d"]
    g = torch.Generator(device="cuda").manual_seed(17)
    bf = lambda std, *s: (torch.randn(s, generator=g, device="cuda") * std).bfloat16()
    stack = dh.dh_stack_create(L, arch=dh.DH_ARCH_LLAMA, dtype=dh.DH_BF16, batch=1, seq=T, hidden=Hd, n_q_heads=c["nq"], n_kv_heads=c["nkv"],
                               head_dim=c["d"], ffn=c["ffn"], eps=1e-5, rope_base=10000.0, n_ranks=c["n_ranks"], comm_blocks=0, n_experts=0,
                               n_local_experts=0)
    try:
        shapes = {"g1": (Hd,), "Wqkv": (Hd, n_qkv), "Wo": (c["nq"] * c["d"], Hd), "g2": (Hd,), "Wgu": (Hd, 2 * c["ffn"]), "Wd": (c["ffn"], Hd)}
        ws, grads = [], []
        for i in range(L):
            w = {k: bf(0.02, *v) + (1.0 if k in ("g1", "g2") else 0.0) for k, v in shapes.items()}
            gr = {"d" + k: torch.zeros(v, device="cuda") for k, v in shapes.items()}
            dh.dh_layer_bind_weights(dh.dh_stack_layer(stack, i), **w)
            dh.dh_layer_bind_wgrads(dh.dh_stack_layer(stack, i), **gr)
            ws.append(w)
            grads.append(gr)
        peers = {k: bf(1e-2, c["n_ranks"] - 1, T, Hd) for k in ("ar1", "ar2", "ar3", "ar4")}
        xs, douts = [bf(1.0, T, Hd) for _ in range(2)], [bf(1e-2, T, Hd) for _ in range(2)]
        outs, dxs = [torch.empty_like(v) for v in xs], [torch.empty_like(v) for v in xs]
        ab, wb = dh.dh_stack_arena_bytes(stack), dh.dh_stack_workspace_bytes(stack)
        arena, wsp = torch.empty(ab, dtype=torch.uint8, device="cuda"), torch.empty(wb, dtype=torch.uint8, device="cuda")
        sa, sb, sc = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
        gf, gb = dh.dh_layer_op_graph(dh.dh_stack_layer(stack, 0), 0), dh.dh_layer_op_graph(dh.dh_stack_layer(stack, 0), 1)
        plan = dh.make_plan(list(range(gf.n_ops)), list(range(gb.n_ops)), [(0, gf.n_ops, 0, gb.n_ops)])
        torch.cuda.synchronize()
        dh.dh_stack_phase(stack, (xs[0], outs[0], peers["ar1"], peers["ar2"]), None, None, arena, ab, wsp, wb, sa, sb, sc)
        dh.dh_stack_phase(stack, (xs[1], outs[1], peers["ar1"], peers["ar2"]), (douts[0], dxs[0], peers["ar3"], peers["ar4"]), plan, arena, ab,
                          wsp, wb, sa, sb, sc)
        torch.cuda.synchronize()
        sums = {k: v.float().sum(0) for k, v in peers.items()}

        def reference(st):
            w32 = [{k: v.float().requires_grad_() for k, v in w.items()} for w in ws]
            got = {}
            for m in range(2):
                x = xs[m].float().requires_grad_()
                out = x
                for w in w32:
                    out = _float32_layer(c, w, out, sums, st)
                got["out%d" % m] = out.detach()
                if m == 0:
                    out.backward(douts[0].float())
                    got["dx"] = x.grad
                    got.update({"d%s, layer %d" % (k, i): v.grad for i, w in enumerate(w32) for k, v in w.items()})
            return got

        mine = {"out0": outs[0].float(), "out1": outs[1].float(), "dx": dxs[0].float()}
        mine.update({"%s, layer %d" % (k, i): v for i, gr in enumerate(grads) for k, v in gr.items()})
        ref, stored = reference(lambda v: v), reference(_Stored.apply)
        for k, v in ref.items():
            err, storage = (float((t[k] - v).norm() / v.norm()) for t in (mine, stored))
            print("%-16s error %.2e, of storage alone %.2e" % (k, err, storage), flush=True)
            assert err <= 1.25 * storage, k
    finally:
        dh.dh_stack_destroy(stack)
