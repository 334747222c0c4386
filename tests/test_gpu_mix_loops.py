"""Residual mixing of more tokens than the launch has blocks for (2^20), and of rows with more columns
than it has shares for: each block then goes round. Every token must have the bits that calls on
parts of the batch, which need no second round, give it; those are held to the oracle elsewhere."""
import pytest
import torch

import paper_2606_07574_amd as b4
from tests._gpu import TOL_DH, say

pytestmark = pytest.mark.gpu

CAP = 1 << 20  # blocks over tokens


def draw(shape, seed, dtype=torch.float32):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.randn(shape, device="cuda:0", generator=g, dtype=dtype)


def parts(B, size):
    return [(i, min(B, i + size)) for i in range(0, B, size)]


# n, dtype, chunks per row, tokens per block: columns of 64 with one, two and four waves, four or two tokens to a
# block; short rows of 8, 16 and 32 lanes per token
FWD = [(4, torch.float32, 33, 4), (4, torch.bfloat16, 65, 4), (4, torch.float32, 129, 1), (8, torch.float32, 33, 2),
       (8, torch.bfloat16, 65, 1), (4, torch.float32, 1, 32), (4, torch.bfloat16, 9, 4), (4, torch.bfloat16, 17, 8),
       (8, torch.float32, 1, 32), (8, torch.bfloat16, 9, 4)]
BWD = [(4, torch.float32, 33, 1), (4, torch.bfloat16, 65, 1), (8, torch.float32, 33, 1), (8, torch.float32, 65, 1),
       (8, torch.bfloat16, 65, 1), (8, torch.bfloat16, 129, 1), (4, torch.float32, 1, 32), (4, torch.bfloat16, 9, 4),
       (4, torch.float32, 17, 8), (8, torch.float32, 1, 32), (8, torch.bfloat16, 9, 4), (8, torch.float32, 17, 8)]
ids = lambda cases: [f"{n}-{str(d)[6:]}-{nc}" for n, d, nc, _ in cases]  # noqa: E731


@pytest.mark.parametrize("n,dtype,nc,tokens", FWD, ids=ids(FWD))
def test_forward_past_the_grid(n, dtype, nc, tokens):
    B, C = CAP * tokens + 3 * tokens + 1, nc * (8 if dtype == torch.bfloat16 else 4)
    say(f"test: mixing forward past the grid, n={n} {dtype} C={C}, B={B}")
    H, X = draw((B, n, n), nc), draw((B, n, C), nc + 1, dtype)
    fwd = b4.mix_fwd if n == 4 else b4.mix8_fwd
    Y, P, _, _ = fwd(H, X)
    for i, j in parts(B, CAP * tokens // 2):
        y, p, _, _ = fwd(H[i:j], X[i:j])
        if j - i >= CAP // 2:  # the last few tokens alone take another layout of the projection
            assert torch.equal(Y[i:j], y) and torch.equal(P[i:j], p)
    k = 3 * tokens + 5  # so they are mixed by the batch's P here
    ref = sum(P[-k:, :, j, None].double() * X[-k:, None, j].double() for j in range(n))
    tol = (n + 1) * 2.0 ** -24 * X[-k:].float().abs().sum(1, keepdim=True)
    assert ((Y[-k:].double() - ref).abs() <= tol + (2.0 ** -8 * ref.abs() if dtype == torch.bfloat16 else 0)).all()


@pytest.mark.parametrize("n,dtype,nc,tokens", BWD, ids=ids(BWD))
def test_backward_past_the_grid(n, dtype, nc, tokens):
    B, C = CAP * tokens + 3 * tokens + 1, nc * (8 if dtype == torch.bfloat16 else 4)
    say(f"test: mixing backward past the grid, n={n} {dtype} C={C}, B={B}")
    P = torch.softmax(draw((B, n, n), nc), -1)
    X, dY = draw((B, n, C), nc + 1, dtype), draw((B, n, C), nc + 2, dtype)
    bwd = b4.mix_bwd if n == 4 else b4.mix8_bwd
    dX, dH = bwd(P, X, dY)
    half = CAP * tokens // 2
    for i, j in [(0, half), (half, 2 * half), (B - half, B)]:  # parts of one size: one layout
        x, h = bwd(P[i:j], X[i:j], dY[i:j])
        assert torch.equal(dX[i:j], x) and torch.equal(dH[i:j], h)


@pytest.mark.parametrize("n,waves", [(4, 16), (8, 4)])
def test_rows_past_the_grid(n, waves):
    """One token whose row has more columns than 32768 blocks of `waves` columns."""
    nc = 64 * waves * 32768 + 64 * waves + 65
    say(f"test: mixing of one long row, n={n}, {nc} chunks")
    H, X = draw((1, n, n), 1), draw((1, n, 4 * nc), 2)
    fwd, bwd = (b4.mix_fwd, b4.mix_bwd) if n == 4 else (b4.mix8_fwd, b4.mix8_bwd)
    Y, P, _, _ = fwd(H, X)
    dX, dH = bwd(P, X, Y)
    dP = torch.zeros(1, n, n, dtype=torch.float64, device="cuda:0")
    for i, j in parts(4 * nc, 1 << 25):
        x, y = X[:, :, i:j].contiguous(), Y[:, :, i:j].contiguous()
        y2, p2, _, _ = fwd(H, x)
        assert torch.equal(p2, P) and torch.equal(y2, y)
        assert torch.equal(dX[:, :, i:j], bwd(P, x, y)[0])
        for a in range(n):
            dP[:, a] += (y[:, a, None].double() * x.double()).sum(-1)
    ref = (b4.bwd if n == 4 else b4.bwd8)(P, dP.float())
    # a lane adds up to 5 * 10^5 products one by one: sqrt(5 * 10^5) 2^-24 = 4e-5 of their sum's size,
    # inside the bound of two gradients that are each within TOL_DH
    assert (dH - ref).abs().max() / ref.abs().max().clamp(min=1.0) <= 2 * TOL_DH
