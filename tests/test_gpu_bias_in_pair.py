"""Bias gradients that ride in the launch of a linear's two gradient products: the bits of dh_colsum.  Widths that end inside a block of 32 columns, row counts
around the 256 row lanes and at the limit of one launch, small layers (carried) and ones whose tiles fill the units (not carried); the launch by itself, and a
layer's four bias gradients each against the gradient it belongs to."""
import ctypes as C

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


class BiasGrad(C.Structure):  # internal to the library, as the launcher is
    _fields_ = [("x", C.c_void_p), ("rows", C.c_int), ("n", C.c_int), ("dst", C.c_void_p)]


LAUNCH = "_Z29dh_launch_gemm_pair_bias_bf16iiiPKDF16bS0_S0_PDF16bPfS0_bPvmP12ihipStream_tPK8BiasGradPb"


# rows, k, n of the products; rows and columns of the sum; whether its blocks find units free
@pytest.mark.parametrize("T,k,n,rows,cols,carried", [(64, 64, 72, 64, 72, True), (1, 64, 64, 1, 8, True), (257, 520, 1000, 257, 1000, True), (528, 1000, 520, 132, 520, True),
                                                     (256, 64, 64, 2048, 40, True), (300, 136, 264, 255, 264, True), (256, 64, 64, 2049, 40, False),
                                                     (1024, 2048, 2056, 1024, 2056, False), (2048, 64, 256, 2048, 4104, False)])
def test_carried_sum(T, k, n, rows, cols, carried):
    print("case", T, k, n, rows, cols, flush=True)
    f = getattr(dh.lib, LAUNCH)
    f.restype, f.argtypes = C.c_int, [C.c_int] * 3 + [C.c_void_p] * 6 + [C.c_bool, C.c_void_p, C.c_size_t, C.c_void_p, C.c_void_p, C.c_void_p]
    gen = torch.Generator(device="cuda").manual_seed(T + rows)
    dY, W, X, x = (torch.randn(s, generator=gen, device="cuda").bfloat16() for s in ((T, n), (k, n), (T, k), (rows, cols)))
    dX, dW = torch.empty(T, k, device="cuda", dtype=torch.bfloat16), torch.zeros(k, n, device="cuda")
    got, want = torch.full((cols + 32,), 2.0, device="cuda"), torch.full((cols + 32,), 2.0, device="cuda")
    nb = max(dh.dh_gemm_workspace_bytes(dh.DH_BF16, 0, 1, T, k, n), dh.dh_gemm_workspace_bytes(dh.DH_BF16, 1, 0, k, n, T), dh.lib.dh_colsum_ws_bytes(rows, cols), 256)
    ws, flag, st = torch.empty(nb, dtype=torch.uint8, device="cuda"), C.c_bool(False), torch.cuda.current_stream().cuda_stream
    sums = BiasGrad(x.data_ptr(), rows, cols, got.data_ptr())
    assert f(T, k, n, dY.data_ptr(), W.data_ptr(), X.data_ptr(), dX.data_ptr(), dW.data_ptr(), None, False, ws.data_ptr(), nb, st, C.addressof(sums),
             C.addressof(flag)) == 0
    assert dh.lib.dh_colsum(dh.DH_BF16, rows, cols, x.data_ptr(), want.data_ptr(), ws.data_ptr(), nb, st) == 0
    torch.cuda.synchronize()
    assert flag.value == carried
    assert torch.equal(got, want) if carried else torch.all(got == 2.0)


@pytest.mark.parametrize("T,hidden,ffn", [(63, 72, 64), (255, 40, 200), (257, 520, 1000), (528, 520, 1000), (2048, 64, 256), (2049, 64, 256)])
def test_each_sum_is_of_its_own_gradient(T, hidden, ffn):
    """A column of a linear's input that is constant over the tokens makes that row of its weight gradient the constant times its bias gradient."""
    print("case", T, hidden, ffn, flush=True)
    run = H.LayerRun(dict(arch="gpt", batch=1, seq=T, hidden=hidden, nq=1, nkv=1, d=64, ffn=ffn, n_ranks=1, bf16=True))
    try:
        w, c, d = run.w, 5, 64
        for i in ("1", "2"):  # a normalised column of ones
            w["g" + i][c], w["b" + i][c] = 0.0, 1.0
        w["Wqkv"][:, 2 * d + c], w["bqkv"][2 * d + c] = 0.0, 1.0  # values of one: so is what attention makes of them
        w["Wgu"][:, c], w["bfc1"][c] = 0.0, 8.0                   # GeLU(8) = 8
        s = run.strand(0)
        run.fwd(s)
        run.bwd(s)
        torch.cuda.synchronize()
        for bias, weight, value, tol in (("dbqkv", "dWqkv", 1.0, 0.0), ("dbfc1", "dWgu", 1.0, 0.0), ("dbfc2", "dWd", 8.0, 0.0), ("dbo", "dWo", 1.0, 2.0 ** -7)):
            got, want = run.g[bias], run.g[weight][c] / value
            assert float(want.norm()) > 0
            # two float32 sums of T terms in different orders (2^-24 of the running sum an addition); attention's row of ones is rounded to bf16
            assert float((got - want).norm()) <= (T * 2.0 ** -24 + 2.0 ** -20 + tol) * float(want.norm()), bias
    finally:
        run.close()
