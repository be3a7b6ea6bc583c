"""A linear's two gradient products asked for as one launch where no launch holds both: a data gradient cut into more K ranges than a paired block
sums, products with more than one round of the largest tiles, and the same with experts' rows.  The layer asks whether a pair pays before it asks
for one, with the device of that moment; the launcher has to be right by itself."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

PAIR = "_Z24dh_launch_gemm_pair_bf16iiiPKDF16bS0_S0_PDF16bPfS0_bPvmP12ihipStream_t"  # the layer's launcher, not part of the C interface


# T, k, n: the data gradient is T x k over n, the weight gradient k x n over T.
@pytest.mark.parametrize("T,k,n", [(1344, 512, 4608), (72, 136, 4096), (4096, 4864, 2048), (256, 256, 512)])
@pytest.mark.parametrize("beside", [False, True])
@pytest.mark.parametrize("ws", [False, True])
def test_pair_launcher_computes_both_products_at_any_size(T, k, n, beside, ws):
    from paper_2411_15871_amd import dhelix as dh
    print("case", T, k, n, beside, ws, flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + n)
    dY, W, X = (torch.randn(s, generator=g, device="cuda").bfloat16() for s in ((T, n), (k, n), (T, k)))
    need = max(dh.dh_gemm_workspace_bytes(dh.DH_BF16, 0, 1, T, k, n), dh.dh_gemm_workspace_bytes(dh.DH_BF16, 1, 0, k, n, T)) if ws else 0
    buf = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    dX, dW = torch.full((T, k), 3.0, device="cuda", dtype=torch.bfloat16), torch.ones(k, n, device="cuda")
    f = getattr(dh.lib, PAIR)
    f.restype, f.argtypes = C.c_int, [C.c_int] * 3 + [C.c_void_p] * 6 + [C.c_bool, C.c_void_p, C.c_size_t, C.c_void_p]
    p = lambda t: t.data_ptr()
    assert f(T, k, n, p(dY), p(W), p(X), p(dX), p(dW), None, beside, p(buf) if need else None, need, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    want_x = torch.mm(dY.double(), W.double().t().contiguous())
    want_w = torch.mm(X.double().t().contiguous(), dY.double()) + 1.0
    # bf16 results: half a unit in the last place an element, 2^-9 in all; float32 sums of up to 4864 exact products
    assert float((dX.double() - want_x).norm() / want_x.norm()) <= 2.0 ** -9
    assert float((dW.double() - want_w).norm() / want_w.norm()) <= 2e-6
