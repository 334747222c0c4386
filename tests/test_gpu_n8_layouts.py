"""The 8 x 8 forward chooses by batch size how many lanes share a problem (1, 2 or 4 rows per
lane, then one problem per lane). Each layout solves the same hard problems at both ends of its
range: unit-scale and large logits, near-permutations, poisoned matrices, a cut step count."""
import numpy as np
import pytest
import torch

import paper_2606_07574_amd as b4
from oracle import birkhoffn as on
from tests._gpu import TOL_DH, say, to_dev
from tests.test_gpu_n8 import check, gauss8, near_perm8
from tests.test_gpu_ot8 import check as check_ot, problem

pytestmark = pytest.mark.gpu

SIZES = [8191, 8192, 8193, 16384, 16385, 65536, 65537]


def tiled(x, B):
    """x repeated along the batch up to B."""
    k = -(-B // x.shape[0])
    return torch.cat([x] * k)[:B].contiguous()


def copies_agree(t, n):
    """Every repetition of the first n results is the same bit for bit."""
    t = torch.nan_to_num(t, nan=-7.0) if t.is_floating_point() else t
    return all(torch.equal(t[i:i + n], t[:min(n, t.shape[0] - i)]) for i in range(n, t.shape[0], n))


@pytest.mark.parametrize("B", SIZES)
def test_projection_layouts(B):
    say(f"test: 8x8 layouts, B={B}")
    H = np.concatenate([gauss8(601, s, 7)[0] for s in (0.1, 1.0, 5.0, 20.0, 50.0)] + [near_perm8(501, 20.0, 0.1, 8),
                                                                                    near_perm8(501, 60.0, 0.1, 9)])
    n = H.shape[0]
    Hd = tiled(to_dev(H), B)
    P, dual, it = b4.fwd8(Hd, want_iters=True)
    assert (it >= 0).all()
    check(H, P[:n].cpu().numpy(), dual[:n].cpu().numpy(), label=f"B={B}")
    assert copies_agree(P, n) and copies_agree(dual, n) and copies_agree(it, n)
    # outputs that are not asked for change nothing
    assert torch.equal(b4.fwd8(Hd, want_dual=False)[0], P)
    assert torch.equal(b4.fwd8(Hd, want_dual=True)[1], dual)


@pytest.mark.parametrize("B", SIZES)
def test_projection_layouts_status(B):
    say(f"test: 8x8 layouts, poisoned and unconverged matrices, B={B}")
    H = gauss8(301, 20.0, 11)[0]
    H[5, 7, 2], H[6, 0, 0], H[300, 3, 7] = np.nan, np.inf, -np.inf
    Hd = tiled(to_dev(H), B)
    bad = torch.zeros(301, dtype=torch.bool)
    bad[[5, 6, 300]] = True
    bad = tiled(bad, B).cuda()
    P, dual, it = b4.fwd8(Hd, max_iter=2, want_iters=True)
    assert (it[bad] == b4.NON_FINITE).all() and torch.isnan(P[bad]).all() and torch.isnan(dual[bad]).all()
    assert (it[~bad] != b4.NON_FINITE).all() and torch.isfinite(P[~bad]).all()
    assert (it[~bad] == b4.NOT_CONVERGED).any()
    rows = (P[~bad].double().sum(-1) - 1).abs().max()
    assert rows < 1e-6  # an unconverged result is still a row softmax
    P0, _, it0 = b4.fwd8(Hd, max_iter=0, want_iters=True)  # the centred start itself
    h = Hd[~bad].double()
    ref = torch.softmax(h + (h.mean(1)[:, -1:] - h.mean(1))[:, None, :], -1)
    assert (P0[~bad].double() - ref).abs().max() < 1e-5 and (it0[~bad] == b4.NOT_CONVERGED).all()


@pytest.mark.parametrize("B", SIZES)
def test_ot_layouts(B):
    say(f"test: 8x8 OT layouts, B={B}")
    M, a, b = problem(1501, 5.0, 13)[:3]
    n = M.shape[0]
    Md, ad, bd = (tiled(to_dev(x), B) for x in (M, a, b))
    T, dual, it = b4.ot8_fwd(Md, ad, bd, 0.5, want_iters=True)
    assert (it >= 0).all()
    check_ot(M, a, b, 0.5, T[:n].cpu().numpy(), dual[:n].cpu().numpy(), label=f"B={B}")
    assert copies_agree(T, n) and copies_agree(dual, n)


# fp32 dH: blocks of four waves from 65537 problems to 262144 but for the quarter after 196608 (OT:
# from 81921 to 114688), one-wave blocks elsewhere
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("B", [65536, 65537, 131072 + 63, 196608, 196609, 229376, 229377, 262144, 262145])
def test_backward_layouts(dtype, B):
    say(f"test: 8x8 backward layouts, dP {dtype}, B={B}")
    H, dP = gauss8(1501, 5.0, 17)
    n = H.shape[0]
    P = b4.fwd8(to_dev(H), want_dual=False)[0]
    dPd = to_dev(dP, dtype)
    ref = on.bwd(P.double().cpu().numpy(), dPd.double().cpu().numpy())
    out = torch.full((B + 1, 8, 8), 3.0, device="cuda:0")  # the last matrix is not written
    dH = b4.bwd8(tiled(P, B), tiled(dPd, B), out=out[:B])
    e = np.abs(dH[:n].cpu().numpy() - ref).max(axis=(1, 2)) / np.maximum(1.0, np.abs(ref).max(axis=(1, 2)))
    assert e.max() <= TOL_DH
    assert copies_agree(dH, n) and (out[B] == 3.0).all()


@pytest.mark.parametrize("B", [81920, 81921, 98304 + 1, 114688, 114689])
def test_ot_backward_layouts(B):
    say(f"test: 8x8 OT backward layouts, B={B}")
    M, a, b, G = problem(1501, 2.0, 19)
    n = M.shape[0]
    T = b4.ot8_fwd(*(to_dev(x) for x in (M, a, b)), 0.5, want_dual=False)[0]
    dM = b4.ot8_bwd(tiled(T, B), tiled(to_dev(a), B), tiled(to_dev(G), B), 0.5)
    ref = on.ot_bwd(T.double().cpu().numpy(), a.astype(np.float64), G.astype(np.float64), 0.5)
    e = np.abs(dM[:n].cpu().numpy() - ref).max(axis=(1, 2)) / np.maximum(1.0, np.abs(ref).max(axis=(1, 2)))
    assert e.max() <= TOL_DH
    assert copies_agree(dM, n)


@pytest.mark.parametrize("B", [65537, 196609])
def test_mixing_backward_layouts(B):
    """dP turned into dH in its own memory: as the backward of the separately computed dP."""
    say(f"test: 8x8 backward in place, B={B}")
    H = gauss8(601, 5.0, 23)[0]
    P = tiled(b4.fwd8(to_dev(H), want_dual=False)[0], B)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(B)
    X, dY = (torch.randn(B, 8, 4, device="cuda:0", generator=g) for _ in range(2))
    _, dH = b4.mix8_bwd(P, X, dY)
    dP = (dY.double().unsqueeze(2) * X.double().unsqueeze(1)).sum(-1)
    ref = b4.bwd8(P, dP.float())
    scale = torch.clamp(ref.abs().amax((1, 2)), min=1.0)
    assert ((dH - ref).abs().amax((1, 2)) / scale).max() <= 2 * TOL_DH  # two gradients within TOL_DH of the exact one
