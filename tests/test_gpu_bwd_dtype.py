"""The backward with a bf16 dH (birkhoff4_bwd_ex2, birkhoff8_bwd_ex, autograd on bf16 logits):
exactly the fp32 gradient rounded to nearest even, at sizes around the 64-problem chunk."""
import pytest
import torch

import paper_2606_07574_amd as b4
from tests._gpu import say

pytestmark = pytest.mark.gpu


def same_bits(x, y):
    return x.dtype == y.dtype and torch.equal(torch.nan_to_num(x, nan=-7.0), torch.nan_to_num(y, nan=-7.0))


@pytest.mark.parametrize("n", [4, 8])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B", [1, 63, 64, 65, 257, 1000])
def test_bf16_gradient_is_the_rounded_fp32_gradient(n, dtype, B):
    say(f"test: bf16 dH, n={n}, dP {dtype}, B={B}")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(100 * n + B)
    H = 4.0 * torch.randn(B, n, n, device="cuda:0", generator=g)
    if B > 64:
        H[B // 2, 0, 1] = float("nan")  # a poisoned matrix stays NaN in either dtype
    dP = torch.randn(B, n, n, device="cuda:0", generator=g).to(dtype)
    fwd, bwd = (b4.fwd, b4.bwd) if n == 4 else (b4.fwd8, b4.bwd8)
    P = fwd(H, want_dual=False)[0]
    ref = bwd(P, dP)
    out = torch.full((B + 1, n, n), 3.0, dtype=torch.bfloat16, device="cuda:0")  # last matrix: not written
    fn = b4.lib().birkhoff4_bwd_ex2 if n == 4 else b4.lib().birkhoff8_bwd_ex
    stream = torch.cuda.current_stream().cuda_stream
    assert fn(P.data_ptr(), dP.data_ptr(), b4._dtype_code(dP), out.data_ptr(), b4.BF16, B, stream) == 0
    torch.cuda.synchronize()
    assert same_bits(out[:B], ref.to(torch.bfloat16))
    assert (out[B] == 3.0).all()


@pytest.mark.parametrize("n", [4, 8])
def test_autograd_gradient_of_bf16_logits(n):
    say(f"test: autograd on bf16 logits, n={n}")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n)
    H = torch.randn(3, 67, n, n, device="cuda:0", generator=g).to(torch.bfloat16).requires_grad_(True)
    G = torch.randn(3, 67, n, n, device="cuda:0", generator=g)
    project, bwd = (b4.project, b4.bwd) if n == 4 else (b4.project8, b4.bwd8)
    P = project(H)
    P.backward(G)
    assert same_bits(H.grad, bwd(P.detach(), G).to(torch.bfloat16))


@pytest.mark.parametrize("n", [4, 8])
@pytest.mark.parametrize("B,C", [(1, 8), (67, 136), (130, 264), (65, 520), (9, 4096), (5, 0)])
def test_mixing_gradient_of_bf16_logits(n, B, C):
    say(f"test: mixing, bf16 logits, n={n} B={B} C={C}")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n * 1000 + C)
    H = torch.randn(B, n, n, device="cuda:0", generator=g).to(torch.bfloat16).requires_grad_(True)
    X = torch.randn(B, n, C, device="cuda:0", generator=g).to(torch.bfloat16)
    dY = torch.randn(B, n, C, device="cuda:0", generator=g).to(torch.bfloat16)
    Y = b4.mix(H, X)
    Y.backward(dY)
    P = (b4.fwd if n == 4 else b4.fwd8)(H.detach(), want_dual=False)[0]
    dX, dH = (b4.mix_bwd if n == 4 else b4.mix8_bwd)(P, X, dY)
    assert dH.dtype == torch.float32 and same_bits(H.grad, dH.to(torch.bfloat16))
