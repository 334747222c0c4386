"""Residual mixing at the edges of its launch rules: rows of one chunk up to more columns than a
block has waves, lanes and waves that end part-way, token counts around the XCD windows."""
import numpy as np
import pytest
import torch

import paper_2606_07574_amd as b4
import workloads
from tests._gpu import TOL_DH, say
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


# lines that depend on the token count: up to 256 tokens (8 waves with n = 8, 15 and 16 columns whole with n = 4),
# from 4096 tokens with n = 8 (one wave for bf16 rows of at most 96 chunks, two for three columns), from
# 8192 tokens of 15 columns with n = 4
TOKEN_LINES = [(n, d, nc, B) for d in (torch.bfloat16, torch.float32)
               for n, nc, B in [(8, 320, 256), (8, 320, 257), (8, 577, 256), (8, 96, 4095), (8, 96, 4096), (8, 97, 4096),
                                (8, 129, 4095), (8, 129, 4096), (8, 192, 4097), (8, 193, 4096), (4, 960, 256),
                                (4, 960, 257), (4, 1024, 256), (4, 1024, 257), (4, 897, 8191), (4, 897, 8192),
                                (4, 17, 4099), (4, 128, 4101), (4, 129, 4101)]]


@pytest.mark.parametrize("n,dtype,nc,B", TOKEN_LINES, ids=[f"{n}-{str(d)[6:]}-{c}x{b}" for n, d, c, b in TOKEN_LINES])
def test_token_lines(n, dtype, nc, B):
    """Every token of the batch against a float64 product on the GPU; the projection and its
    backward, which the other tests hold to the oracle, on the same P."""
    C = nc * (8 if dtype == torch.bfloat16 else 4)
    say(f"test: mixing layouts by token count, n={n} {dtype} C={C} ({nc} chunks), B={B}")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(nc + B)
    H = 3.0 * torch.randn(B, n, n, device="cuda:0", generator=g)
    X, dY = (torch.randn(B, n, C, device="cuda:0", generator=g).to(dtype) for _ in range(2))
    mfwd, mbwd, bwd = (b4.mix_fwd, b4.mix_bwd, b4.bwd) if n == 4 else (b4.mix8_fwd, b4.mix8_bwd, b4.bwd8)
    Y, P, _, _ = mfwd(H, X)
    dX, dH = mbwd(P, X, dY)
    dP = torch.empty(B, n, n, dtype=torch.float64, device="cuda:0")
    for i in range(n):
        y = sum(P[:, i, j, None].double() * X[:, j].double() for j in range(n))
        s = X.float().abs().sum(1)
        # fp32 sums of n products of |P| <= 1: (n + 1) 2^-24 of the sum of the magnitudes; bf16 results
        # rounded once more (2^-8, as half a unit in the last place is at most that of the value)
        tol = (n + 1) * 2.0 ** -24 * s + (2.0 ** -8 * y.abs() if dtype == torch.bfloat16 else 0) + 1e-30
        assert ((Y[:, i].double() - y).abs() <= tol).all()
        x = sum(P[:, j, i, None].double() * dY[:, j].double() for j in range(n))
        s = dY.float().abs().sum(1)
        tol = (n + 1) * 2.0 ** -24 * s + (2.0 ** -8 * x.abs() if dtype == torch.bfloat16 else 0) + 1e-30
        assert ((dX[:, i].double() - x).abs() <= tol).all()
        for j in range(n):
            dP[:, i, j] = (dY[:, i].double() * X[:, j].double()).sum(1)
    ref = bwd(P, dP.float())
    scale = torch.clamp(ref.abs().amax((1, 2)), min=1.0)
    assert ((dH - ref).abs().amax((1, 2)) / scale).max() <= 2 * TOL_DH  # each within TOL_DH of the exact gradient
