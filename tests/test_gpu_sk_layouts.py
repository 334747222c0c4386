"""Sinkhorn-Knopp kernels at the edges of their layouts: four lanes per problem, one problem per
lane for many steps of a large batch, register and LDS backward, ragged batches; the fp64
oracle's map and its reverse-mode gradient."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_07574_amd as b4
import workloads
from tests._gpu import bits_to_dev, say, to_dev

pytestmark = pytest.mark.gpu


def check(H, dP, Hd, dPd, steps, label):
    P, dH = b4.sk_fwd(Hd, steps), b4.sk_bwd(Hd, dPd, steps)
    torch.cuda.synchronize()
    n = H.shape[0]
    Pr = oracle.sk_fwd(H.astype(np.float64), steps)
    dHr = oracle.sk_bwd(H.astype(np.float64), dP.astype(np.float64), steps)
    pe = np.abs(P[:n].cpu().numpy() - Pr).max()
    he = (np.abs(dH[:n].cpu().numpy() - dHr).max(axis=(1, 2)) / np.maximum(1.0, np.abs(dHr).max(axis=(1, 2)))).max()
    say(f"  [{label}] P err={pe:.2e} dH rel err={he:.2e}")
    # each of the 2 n half-steps rounds four products, their sum and a reciprocal (1 ulp): the
    # relative error of an entry of P stays below 2 n * 8 * 2^-24; the gradient takes each step
    # twice
    bound = 16 * steps * 2.0 ** -24
    assert pe <= bound and he <= 4 * bound
    return P, dH


@pytest.mark.parametrize("B", [1, 3, 15, 16, 17, 63, 64, 65, 1001])
@pytest.mark.parametrize("steps", [1, 2, 20, 33])
def test_ragged(B, steps):
    say(f"test: Sinkhorn layouts, B={B}, {steps} steps")
    H, dP = workloads.gauss(B, 2.0, seed=B + steps)
    check(H, dP, to_dev(H), to_dev(dP), steps, f"B={B} n={steps}")
    Hb, Gb = workloads.bf16_bits(H), workloads.bf16_bits(dP)
    check(workloads.bf16_to_f32(Hb), workloads.bf16_to_f32(Gb), bits_to_dev(Hb), bits_to_dev(Gb), steps, "bf16")


# lines of the forward's layouts: fp32 13 steps and 31 * 2^14 problems, bf16 12 steps and 11 * 2^15,
# from 32 steps on 2^18
@pytest.mark.parametrize("dtype,steps,B", [(d, s, b) for d, steps, line in ((torch.float32, (12, 13, 20), 31 << 14),
                                                                            (torch.bfloat16, (11, 12, 20), 11 << 15))
                                           for s in steps for b in (line - 1, line)]
                         + [(d, s, b) for d in (torch.float32, torch.bfloat16) for s in (31, 32)
                            for b in ((1 << 18) - 1, 1 << 18)] + [(torch.float32, 20, (1 << 19) + 77)])
def test_large(dtype, B, steps):
    say(f"test: Sinkhorn layouts, {dtype}, B={B}, {steps} steps")
    H, dP = workloads.gauss(5003, 3.0, seed=steps)
    if dtype == torch.bfloat16:
        H, dP = (workloads.bf16_to_f32(workloads.bf16_bits(x)) for x in (H, dP))
    k = -(-B // 5003)
    Hd, dPd = (torch.cat([to_dev(x, dtype)] * k)[:B].contiguous() for x in (H, dP))
    P, dH = check(H, dP, Hd, dPd, steps, f"B={B} n={steps}")
    for i in range(5003, B, 5003):  # every copy of the problems gives the same bits
        m = min(5003, B - i)
        assert torch.equal(P[i:i + m], P[:m]) and torch.equal(dH[i:i + m], dH[:m])


# backward with the iterates in LDS: 160 KB hold 512 n bytes per wave of 16 problems with both
# iterates; a batch that 256 CUs do not hold at once keeps the v^(k) alone (16 steps: up to four
# rounds of waves; 11 and fewer: never)
@pytest.mark.parametrize("steps,B", [(11, 4096 * 28 + 1), (12, 4096 * 26), (12, 4096 * 26 + 1), (16, 4096 * 80),
                                     (16, 4096 * 80 + 1), (33, 4096 * 9), (33, 4096 * 9 + 1), (48, 4096 * 6 + 77)])
def test_backward_in_lds(steps, B):
    say(f"test: Sinkhorn backward in LDS, B={B}, {steps} steps")
    H, dP = workloads.gauss(2003, 3.0, seed=steps)
    k = -(-B // 2003)
    Hd, dPd = (torch.cat([to_dev(x)] * k)[:B].contiguous() for x in (H, dP))
    _, dH = check(H, dP, Hd, dPd, steps, f"B={B} n={steps}")
    small = b4.sk_bwd(Hd[:2003], dPd[:2003], steps)  # both iterates kept
    for i in range(0, B, 2003):
        assert torch.equal(dH[i:i + 2003], small[:min(2003, B - i)])
