"""Forward kernels whose waves end one after the other: every problem of the batch is solved
exactly once at sizes around the rules' lines. A small set of problems is repeated over the
batch; each copy must give the bits of the first, and the first must match the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_07574_amd as b4
import workloads
from oracle import birkhoffn as on
from tests._gpu import TOL_P, say, to_dev

pytestmark = pytest.mark.gpu


def repeated(x, B):
    d = to_dev(x)
    return torch.cat([d] * (-(-B // x.shape[0])))[:B].contiguous()


def same_copies(t, n):
    full = t.shape[0] // n * n
    assert torch.equal(t[:full].view(-1, n, *t.shape[1:]), t[:n].expand(full // n, *t[:n].shape))
    assert torch.equal(t[full:], t[:t.shape[0] - full])


# 4 x 4: blocks of one CU share its batches of 64; past sixteen of them, half and a quarter of the
# rest (at most 24 and 14; 5/8 and 3/8 of fewer than 28) are left to the other waves. 16384 problems are one batch per block.
@pytest.mark.parametrize("B", [32769, 100003, 16384 * 7 - 1, 16384 * 16, 16384 * 16 + 1, 16384 * 18, 16384 * 20,
                               16384 * 25, 16384 * 32 + 77, 16384 * 43, 16384 * 44, 1 << 20, 16384 * 72 + 5, 3000001])
def test_projection(B):
    say(f"test: staggered 4x4 forward, B={B}")
    H = np.concatenate([workloads.gauss(401, s, seed=5)[0] for s in (1.0, 10.0, 50.0)])
    n = H.shape[0]
    Hd = repeated(H, B)
    out = torch.full((B, 4, 4), float("nan"), device="cuda:0")
    P, _, it = b4.fwd(Hd, want_dual=False, want_iters=True, out=out, variant=b4.THROUGHPUT)
    assert (it >= 0).all()
    assert np.abs(P[:n].cpu().numpy() - oracle.fwd(H.astype(np.float64))[0]).max() <= TOL_P
    same_copies(P, n)
    P2, dual, _ = b4.fwd(Hd, variant=b4.THROUGHPUT)
    same_copies(P2, n)
    same_copies(dual, n)


# 4 x 4 OT: ranges of 64 problems below 112 per wave (4096 waves), of equal length up to 191, then
# four classes of waves up to 3 * 2^19 problems, and 8192 ranges
@pytest.mark.parametrize("B", [64 * 4096 + 1, 111 * 4096, 111 * 4096 + 1, 191 * 4096, 191 * 4096 + 1, 1 << 20, (1 << 20) + 77, 3 * (1 << 19) - 1, 3 * (1 << 19)])
def test_ot(B):
    say(f"test: staggered 4x4 OT forward, B={B}")
    rng = np.random.default_rng(B)
    n = 1009
    M = (2.0 * rng.standard_normal((n, 4, 4))).astype(np.float32)
    a = rng.uniform(0.2, 2.0, (n, 4)).astype(np.float32)
    b = rng.uniform(0.2, 2.0, (n, 4))
    b = (b * (a.astype(np.float64).sum(1) / b.sum(1))[:, None]).astype(np.float32)
    T, dual, it = b4.ot_fwd(*(repeated(x, B) for x in (M, a, b)), 0.5, want_iters=True)
    assert (it >= 0).all()
    b64 = b.astype(np.float64)
    b64 *= (a.astype(np.float64).sum(1) / b64.sum(1))[:, None]
    ref = on.ot_fwd(M.astype(np.float64), a.astype(np.float64), b64, 0.5)[0]
    assert np.abs(T[:n].cpu().numpy() - ref).max() <= 2e-5  # masses up to 2: twice the bound at unit mass
    same_copies(T, n)
    same_copies(dual, n)


# 8 x 8: 2048 waves of 32-problem batches; no stagger below 4 full rounds, then 2, 3 and 6 batches.
# Per line: one batch short of it, the line, a ragged size past it, and the last size of the
# round, whose remainder gives the early blocks the most extra batches.
SIZES8 = [65536 * r + off for r in (4, 7, 32) for off in (-32, 0, 33, 65536 - 33)]


@pytest.mark.parametrize("B", [131072 + 33] + SIZES8)
def test_projection8(B):
    say(f"test: staggered 8x8 forward, B={B}")
    rng = np.random.default_rng(B)
    H = np.concatenate([s * rng.standard_normal((301, 8, 8)) for s in (1.0, 10.0)]).astype(np.float32)
    n = H.shape[0]
    Hd = repeated(H, B)
    P, _, it = b4.fwd8(Hd, want_dual=False, want_iters=True)
    assert (it >= 0).all()
    assert np.abs(P[:n].cpu().numpy() - on.fwd(H.astype(np.float64))[0]).max() <= TOL_P
    same_copies(P, n)
    same_copies(it, n)
    P2, dual, _ = b4.fwd8(Hd)
    assert torch.equal(P2, P)
    same_copies(dual, n)


@pytest.mark.parametrize("B", [65536 * 4 - 32, 65536 * 5 - 33, 65536 * 6 + 1])
def test_ot8(B):
    say(f"test: staggered 8x8 OT forward, B={B}")
    rng = np.random.default_rng(B)
    n = 601
    M = (2.0 * rng.standard_normal((n, 8, 8))).astype(np.float32)
    a = rng.uniform(0.2, 2.0, (n, 8)).astype(np.float32)
    b = rng.uniform(0.2, 2.0, (n, 8))
    b = (b * (a.astype(np.float64).sum(1) / b.sum(1))[:, None]).astype(np.float32)
    T, dual, it = b4.ot8_fwd(*(repeated(x, B) for x in (M, a, b)), 0.5, want_iters=True)
    assert (it >= 0).all()
    b64 = b.astype(np.float64)
    b64 *= (a.astype(np.float64).sum(1) / b64.sum(1))[:, None]
    ref = on.ot_fwd(M.astype(np.float64), a.astype(np.float64), b64, 0.5)[0]
    assert np.abs(T[:n].cpu().numpy() - ref).max() <= 2e-5  # as above
    for t in (T, dual, it):
        same_copies(t, n)
