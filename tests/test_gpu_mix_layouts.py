"""Residual mixing at the edges of its launch rules: rows of one chunk up to more columns than a
block has waves, lanes and waves that end part-way, token counts around the XCD windows."""
import numpy as np
import pytest
import torch

import paper_2606_07574_amd as b4
import workloads
from tests._gpu import say
from tests.test_gpu_mix import check_case
from tests.test_gpu_n8 import gauss8

pytestmark = pytest.mark.gpu

# chunks of 16 bytes per row, tokens: the short rows (8, 16 and 32 lanes per token), one column
# (four tokens per block), several, and turns of the block's waves or shares of the row
ROWS = [(1, 70), (7, 33), (8, 64), (9, 31), (16, 40), (17, 9), (32, 300), (33, 257), (63, 5), (64, 130), (65, 129),
        (129, 128), (257, 127), (320, 3), (512, 136), (513, 20), (768, 17), (1024, 9), (1025, 5), (2100, 2)]

# enough tokens that the projection and the mixing are launched apart: 2048 columns of 64 chunks
# (n = 8: 1024) at most are fused
APART = [(1, 2049), (8, 2100), (9, 2050), (16, 2051), (17, 2049), (32, 2090), (33, 2049), (64, 2049), (65, 1025),
         (130, 700), (300, 411), (512, 257), (513, 228), (1024, 129), (1025, 121), (2100, 63)]
# the last fused size and the first that is not, with one and with several columns
LINE = [(64, 1024), (64, 1025), (65, 512), (65, 513), (64, 2048), (65, 1024), (512, 128), (512, 129), (512, 256)]


@pytest.mark.parametrize("n", [4, 8])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("nc,B", ROWS + APART + LINE, ids=[f"{c}x{b}" for c, b in ROWS + APART + LINE])
def test_rows(n, dtype, nc, B):
    C = nc * (8 if dtype == torch.bfloat16 else 4)
    say(f"test: mixing layouts, n={n} {dtype} C={C} ({nc} chunks), B={B}")
    rng = np.random.default_rng([n, nc, B])
    H = workloads.gauss(B, 3.0, seed=nc)[0] if n == 4 else gauss8(B, 3.0, nc)[0]
    X = rng.standard_normal((B, n, C), dtype=np.float32)
    G = rng.standard_normal((B, n, C), dtype=np.float32)
    if dtype == torch.bfloat16:
        X, G = (workloads.bf16_to_f32(workloads.bf16_bits(v)) for v in (X, G))
    check_case(H, X, G, dtype, f"n={n} nc={nc} B={B}")


@pytest.mark.parametrize("n", [4, 8])
@pytest.mark.parametrize("h_dtype", [torch.float32, torch.bfloat16])
def test_fused_call_outputs(n, h_dtype):
    """The fused call writes what the projection alone writes, bit for bit, whichever outputs are
    asked for, and reports poisoned tokens and cut step counts in the same way."""
    say(f"test: fused mixing outputs, n={n} {h_dtype}")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n)
    H = (10.0 * torch.randn(70, n, n, device="cuda:0", generator=g)).to(h_dtype)
    H[9, 1, 2], H[33, 0, 0] = float("nan"), float("inf")
    X = torch.randn(70, n, 520, device="cuda:0", generator=g)
    fwd, mfwd = (b4.fwd, b4.mix_fwd) if n == 4 else (b4.fwd8, b4.mix8_fwd)
    same = lambda x, y: torch.equal(torch.nan_to_num(x, nan=-7.0), torch.nan_to_num(y, nan=-7.0))  # noqa: E731
    for max_iter in (64, 3, 0):
        P, dual, it = fwd(H, max_iter=max_iter, want_iters=True)
        for want_dual in (False, True):
            for want_iters in (False, True):
                Y, P2, d2, it2 = mfwd(H, X, max_iter=max_iter, want_dual=want_dual, want_iters=want_iters)
                assert same(P2, P)
                assert (d2 is None) == (not want_dual) and (it2 is None) == (not want_iters)
                assert d2 is None or same(d2, dual)
                assert it2 is None or torch.equal(it2, it)
                ref = (P.double().unsqueeze(-1) * X.double().unsqueeze(1)).sum(2)
                ok = torch.isfinite(ref)
                assert (torch.isfinite(Y) == ok).all()
                assert ((Y.double() - ref)[ok].abs() <= 1e-5 * X.abs().max()).all()
