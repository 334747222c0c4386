"""Performance cases: the work that a program using this library has it do, through the
public entry points of ``paper_2606_07574_amd``.

Every case names a path, a logit family and its sizes; ``prepare`` draws the inputs on the
GPU from a seed, ``run`` makes one pass, ``exact`` gives the same results in float64 with
plain torch. The logit families are the workloads of this repository: N(0, sigma^2), the
mixture of Gaussian and near-permutation matrices, and N(0, s^2) with s log-uniform.

Paths
  pair     fwd without the dual, then bwd, on 4x4 matrices (a program with its own autograd)
  fwd      fwd with P and the dual (inference, or a consumer of the potentials)
  project  project / project8 under autograd: P and the gradient of the logits
  ot       ot / ot8 under autograd: transport plans and the gradient of the costs
  sk       sk_fwd and sk_bwd, the Sinkhorn-Knopp baseline
  mix      mix under autograd: the residual mixing of a training step
  mixfwd   mix_fwd / mix8_fwd alone: the residual mixing of inference
"""
import math

import torch

import paper_2606_07574_amd as b4

F32, BF16 = "f32", "bf16"
DTYPES = {F32: torch.float32, BF16: torch.bfloat16}


def listed():
    return [
        # a few sequences' tokens in one layer, at the logit scale of the runtime sweep in the
        # paper: a call whose latency counts
        dict(name="pair4_small", path="pair", n=4, logits="gauss", sigma=10.0, dtype=F32, B=2048),
        # a large batch of unit-scale logits with the potentials, fp32
        dict(name="fwd4_dual", path="fwd", n=4, logits="gauss", sigma=1.0, dtype=F32, B=1 << 20),
        # the benchmark's mixture at its full size in bf16: a whole step's tokens of all layers
        dict(name="project4_large", path="project", n=4, logits="mixture", sigma=0.0, dtype=BF16, B=1 << 24),
        # logits of every scale from 0.1 to 50, fp32, a ragged batch
        dict(name="pair4_scales", path="pair", n=4, logits="logunif", sigma=50.0, dtype=F32, B=3_000_001),
        # one micro-batch's tokens with eight residual streams, the latency side of 8x8
        dict(name="project8_small", path="project", n=8, logits="gauss", sigma=1.0, dtype=F32, B=4096),
        # 8x8 matrices of many layers at once, bf16, a ragged batch
        dict(name="project8_large", path="project", n=8, logits="mixture", sigma=0.0, dtype=BF16, B=1_000_003),
        # general marginals and regulariser, 4x4 and 8x8
        dict(name="ot4", path="ot", n=4, eta=0.5, B=1_048_653),
        dict(name="ot8", path="ot", n=8, eta=0.5, B=200_003),
        # the twenty-step baseline that the projection is compared with
        dict(name="sk20", path="sk", n=4, logits="gauss", sigma=5.0, dtype=F32, steps=20, B=1 << 20),
        # a training micro-batch's residual mixing: four streams, 32 K tokens of width 4096
        dict(name="mix4_train", path="mix", n=4, logits="mixture", sigma=0.0, dtype=BF16, B=32768, C=4096),
        # the same with eight streams and 8 K tokens
        dict(name="mix8_train", path="mix", n=8, logits="mixture", sigma=0.0, dtype=BF16, B=8192, C=4096),
        # residual mixing of a decoding batch: few tokens, forward only
        dict(name="mix4_decode", path="mixfwd", n=4, logits="gauss", sigma=1.0, dtype=BF16, B=96, C=4096),
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["pair", "fwd", "project", "project", "ot", "sk", "mix", "mix", "mixfwd"])
    n = rng.choice([4, 8]) if path in ("project", "ot", "mix", "mixfwd") else 4
    dtype = rng.choice([F32, BF16])
    if path == "ot":
        return dict(path=path, n=n, eta=rng.choice([0.25, 0.5, 1.0]), B=_log(rng, 500, 2_000_000 if n == 4 else 400_000))
    logits = rng.choice(["gauss", "gauss", "mixture", "logunif"])
    # the dual of weakly coupled columns is not determined in 32 bits: unit-scale logits there
    sigma = rng.choice([1.0, 2.0]) if path == "fwd" else rng.choice([1.0, 5.0, 10.0])
    if path == "fwd":
        logits = "gauss"
    if path == "sk":
        logits, sigma = "gauss", rng.choice([1.0, 5.0])
    sigma = {"gauss": sigma, "mixture": 0.0, "logunif": 50.0 if n == 4 else 10.0}[logits]
    case = dict(path=path, n=n, logits=logits, sigma=sigma, dtype=dtype)
    if path in ("mix", "mixfwd"):
        case["C"] = 8 * _log(rng, 16, 640)
        most = 1 << 29  # values of X: what the largest listed case moves
        case["B"] = _log(rng, 8, min(32768, most // (n * case["C"])))
        return case
    if path == "sk":
        case["steps"] = rng.choice([10, 20, 20, 30])
        case["B"] = _log(rng, 500, 2_000_000)
        return case
    case["B"] = _log(rng, 300, 12_000_000 if n == 4 else 1_500_000)
    return case


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _logits(case, g, dev):
    B, n = case["B"], case["n"]
    Z = torch.randn(B, n, n, device=dev, generator=g)
    kind = case["logits"]
    if kind == "gauss":
        Z *= case["sigma"]
    elif kind == "logunif":
        Z *= torch.exp(torch.empty(B, 1, 1, device=dev).uniform_(math.log(0.1), math.log(case["sigma"]), generator=g))
    else:  # half sigma N(0,1), sigma from {1, 5, 20}; half 20 Pi + 0.1 N(0,1)
        near = torch.randint(0, 2, (B, 1, 1), device=dev, generator=g) == 1
        s = torch.tensor([1.0, 5.0, 20.0], device=dev)[torch.randint(0, 3, (B, 1, 1), device=dev, generator=g)]
        Z *= torch.where(near, torch.tensor(0.1, device=dev), s)
        perm = torch.argsort(torch.rand(B, n, device=dev, generator=g), dim=1)
        Z.scatter_add_(2, perm[:, :, None], torch.where(near, 20.0, 0.0).expand(B, n, 1))
    return Z.to(DTYPES[case["dtype"]])


def prepare(case, seed):
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    path, n, B = case["path"], case["n"], case["B"]
    s = {"case": case}
    if path == "ot":
        s["M"] = 2.0 * torch.randn(B, n, n, device=dev, generator=g)
        s["a"] = 0.2 + 1.8 * torch.rand(B, n, device=dev, generator=g)
        b = (0.2 + 1.8 * torch.rand(B, n, device=dev, generator=g)).double()
        s["b"] = (b * (s["a"].double().sum(1, keepdim=True) / b.sum(1, keepdim=True))).float()
        s["M"].requires_grad_(True)
        s["dT"] = torch.randn(B, n, n, device=dev, generator=g)
        return s
    s["H"] = _logits(case, g, dev)
    if path in ("mix", "mixfwd"):
        C, dt = case["C"], DTYPES[case["dtype"]]
        s["X"] = torch.randn(B, n, C, device=dev, generator=g, dtype=dt)
        if path == "mix":
            s["dY"] = torch.randn(B, n, C, device=dev, generator=g, dtype=dt)
            s["H"].requires_grad_(True)
            s["X"].requires_grad_(True)
        return s
    if path in ("pair", "sk"):
        s["dP"] = torch.randn(B, n, n, device=dev, generator=g).to(DTYPES[case["dtype"]])
    elif path == "project":
        s["dP"] = torch.randn(B, n, n, device=dev, generator=g)  # P is fp32, so is its gradient
        s["H"].requires_grad_(True)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    path, n = case["path"], case["n"]
    if path == "pair":
        P, _, _ = b4.fwd(s["H"], want_dual=False)
        return P, b4.bwd(P, s["dP"])
    if path == "fwd":
        P, dual, _ = b4.fwd(s["H"])
        return P, dual
    if path == "project":
        P = (b4.project if n == 4 else b4.project8)(s["H"])
        (dH,) = torch.autograd.grad(P, s["H"], s["dP"])
        return P.detach(), dH
    if path == "ot":
        T = (b4.ot if n == 4 else b4.ot8)(s["M"], s["a"], s["b"], case["eta"])
        (dM,) = torch.autograd.grad(T, s["M"], s["dT"])
        return T.detach(), dM
    if path == "sk":
        return b4.sk_fwd(s["H"], case["steps"]), b4.sk_bwd(s["H"], s["dP"], case["steps"])
    if path == "mix":
        Y = b4.mix(s["H"], s["X"])
        dH, dX = torch.autograd.grad(Y, (s["H"], s["X"]), s["dY"])
        return Y.detach(), dX, dH
    Y, P, _, _ = (b4.mix_fwd if n == 4 else b4.mix8_fwd)(s["H"], s["X"])
    return Y, P


def work(case):
    """Bytes: each input read and each output written once. Operations: the mean Newton (or
    Sinkhorn) steps of the family times one step's multiplications and additions, and the
    contractions."""
    path, n, B = case["path"], case["n"], case["B"]
    m = n * n
    size = 2 if case.get("dtype") == BF16 else 4
    steps = {"gauss": 2.8, "mixture": 2.4, "logunif": 4.1}.get(case.get("logits"), 5.2)
    if case.get("logits") == "gauss" and case["sigma"] > 3.0:
        steps = 5.8
    # one Newton step: column scaling and row sums 4 m, weights n m, elimination n^3 / 3
    forward = B * (steps * (4 * m + n * m + n ** 3 / 3) + 4 * m)
    backward = B * (2 * n * m + 2 * n ** 3 / 3 + 4 * m)
    if path == "pair":
        return {"bytes": B * m * (2 * size + 8), "flops": forward + backward}
    if path == "fwd":
        return {"bytes": B * (m * (size + 4) + 8 * n), "flops": forward}
    if path == "project":
        return {"bytes": B * m * (2 * size + 8), "flops": forward + backward}
    if path == "ot":
        return {"bytes": B * (m * 16 + 8 * n), "flops": forward + backward}
    if path == "sk":
        return {"bytes": B * m * (2 * size + 8), "flops": B * case["steps"] * (4 * m + 10 * m)}
    streams = B * n * case["C"]
    if path == "mix":
        return {"bytes": streams * 4 * size + 2 * B * m * size, "flops": forward + backward + 6 * n * streams}
    return {"bytes": streams * 2 * size + B * m * (size + 4), "flops": forward + 2 * n * streams}


def tolerance(case):
    """Against ``exact``, over listed and drawn cases, the library's fp32 outputs are at most
    7.4e-7 off in the 2-norm (iterations that stop at a column residual of 1e-6) and 3.1e-5
    in the worst value; bf16 outputs are one rounding off, 1.7e-3 and 2^-8. Another correct
    implementation differs from this one by up to about four times that."""
    if case.get("dtype") == BF16 and case["path"] in ("project", "mix", "mixfwd"):
        return {"rel": 6e-3, "max": 2e-2}
    return {"rel": 3e-6, "max": 1.5e-4}


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------
def _eliminate(W, q, r):
    """Solve (Laplacian of the weights W [B,k,k] + diag(q)) x = r by elimination whose pivots
    are sums of non-negative terms; r [B,k,m]."""
    W, q, r = W.clone(), q.clone(), r.clone()
    k = W.shape[-1]
    piv = []
    for p in range(k):
        d = (q[:, p] + W[:, p, p + 1:].sum(-1)).clamp_min(1e-300)
        piv.append(d)
        if p + 1 < k:
            f = W[:, p, p + 1:] / d[:, None]
            W[:, p + 1:, p + 1:] += f[:, :, None] * W[:, p, None, p + 1:]
            q[:, p + 1:] += f * q[:, p, None]
            r[:, p + 1:] += f[:, :, None] * r[:, p, None]
    x = torch.zeros_like(r)
    for p in reversed(range(k)):
        x[:, p] = (r[:, p] + (W[:, p, p + 1:, None] * x[:, p + 1:]).sum(1)) / piv[p][:, None]
    return x


def _solve(h, a, b):
    """Entropic transport with unit regulariser in float64 by damped Newton steps on the
    column potentials x (x_n = 0): T_ij = a_i softmax_j(h_ij + x_j) with column sums b."""
    n = h.shape[-1]
    x = h.mean(1)[:, -1:] - h.mean(1) + (b / b[:, -1:]).log()

    def at(hh, xx, aa, bb):
        v = hh + xx[:, None, :]
        T = aa[:, :, None] * torch.softmax(v, -1)
        f = (aa * torch.logsumexp(v, -1)).sum(-1) - (bb * xx).sum(-1)
        g = T.sum(1) - bb
        g[:, -1] = 0.0  # x_n is fixed: its column takes what the marginals' sums differ by
        return T, f, g

    T, f, g = at(h, x, a, b)
    live = torch.arange(h.shape[0], device=h.device)
    lam = torch.full_like(f, 1e-6)
    for _ in range(400):
        live = live[g[live].abs().amax(-1) > 2e-13 * n]
        if not live.numel():
            break
        Tl, gl, al, bl, hl = T[live], g[live], a[live], b[live], h[live]
        W = (Tl / al[:, :, None]).transpose(1, 2).contiguous() @ Tl
        mu = lam[live] * gl.abs().amax(-1)
        d = -_eliminate(W[:, :-1, :-1], W[:, :-1, -1] + mu[:, None], gl[:, :-1, None])[:, :, 0]
        d = torch.cat([d, torch.zeros_like(d[:, :1])], 1)
        d *= (8.0 / (d.amax(-1) - d.amin(-1)).clamp_min(1e-300)).clamp_max(1.0)[:, None]
        Tn, fn, gn = at(hl, x[live] + d, al, bl)
        slope = (gl * d).sum(-1)
        # once f no longer resolves the decrease a smaller gradient decides
        floor = 1e-14 * (1.0 + f[live].abs() + hl.abs().amax((1, 2)))
        ok = (fn - f[live] <= 1e-4 * slope) | (((fn - f[live]).abs() <= floor) & (gn.norm(dim=-1) < gl.norm(dim=-1)))
        took = live[ok]
        x[took] += d[ok]
        T[took], f[took], g[took] = Tn[ok], fn[ok], gn[ok]
        lam[live] = torch.where(ok, (lam[live] / 16).clamp_min(1e-6), lam[live] * 16)
    return T, x - x[:, -1:]


def _vjp(T, a, G):
    """dL/dh of T(h) for dL/dT = G: the implicit derivative, with antisymmetric flows."""
    S = T / a[:, :, None]
    n = T.shape[-1]
    W = S.transpose(1, 2).contiguous() @ T
    F = torch.zeros_like(W)
    for i in range(n):
        t, g = T[:, i], G[:, i]
        F += (S[:, i, :, None] * t[:, None, :]) * (g[:, :, None] - g[:, None, :])
    # elimination that keeps the right-hand sides as flows on the edges
    piv = []
    for p in range(n - 1):
        d = W[:, p, p + 1:].sum(-1).clamp_min(1e-300)
        piv.append(d)
        if p + 1 < n - 1:
            f = W[:, p, p + 1:] / d[:, None]
            fl = F[:, p, p + 1:]
            F[:, p + 1:, p + 1:] += f[:, :, None] * fl[:, None, :] - fl[:, :, None] * f[:, None, :]
            W[:, p + 1:, p + 1:] += f[:, :, None] * W[:, p, None, p + 1:]
    w = torch.zeros_like(T[:, 0])
    for p in reversed(range(n - 1)):
        w[:, p] = (F[:, p, p + 1:].sum(-1) + (W[:, p, p + 1:] * w[:, p + 1:]).sum(-1)) / piv[p]
    psi = G - w[:, None, :]
    return T * (psi - (S * psi).sum(-1, keepdim=True))


def _parts(B, n, work_n):
    """Ranges of problems whose temporaries stay small."""
    step = max(1, work_n // (n * n))
    return [slice(i, min(B, i + step)) for i in range(0, B, step)]


def exact(case, seed):
    s = prepare(case, seed)
    path, n, B = case["path"], case["n"], case["B"]
    outs = []
    for part in _parts(B, n, 1 << 26 if path in ("pair", "fwd", "project", "ot") else 1 << 16):
        if path == "ot":
            h = -s["M"].detach()[part].double() / case["eta"]
            a, b = s["a"][part].double(), s["b"][part].double()
            T, _ = _solve(h, a, b)
            outs.append((T, -_vjp(T, a, s["dT"][part].double()) / case["eta"]))
            continue
        h = s["H"].detach()[part].double()
        one = torch.ones_like(h[:, 0])
        if path == "sk":
            hh = h.requires_grad_(True)
            A = torch.exp(hh - hh.amax(-1, keepdim=True).detach())
            v = one
            for _ in range(case["steps"]):
                u = 1.0 / (A * v[:, None, :]).sum(-1)
                v = 1.0 / (A * u[:, :, None]).sum(1)
            P = u[:, :, None] * A * v[:, None, :]
            (dH,) = torch.autograd.grad(P, hh, s["dP"][part].double())
            outs.append((P.detach(), dH))
            continue
        P, x = _solve(h, one, one)
        if path == "fwd":
            outs.append((P, torch.cat([-torch.logsumexp(h + x[:, None, :], -1), x], -1)))
        elif path in ("pair", "project"):
            outs.append((P, _vjp(P, one, s["dP"][part].double())))
        else:
            X = s["X"].detach()[part].double()
            Y = sum(P[:, :, j, None] * X[:, None, j] for j in range(n))
            if path == "mixfwd":
                outs.append((Y.float(), P))  # float32 holds the result far past the streams' rounding
                continue
            dY = s["dY"][part].double()
            dX = sum(P[:, i, :, None] * dY[:, None, i] for i in range(n))
            dP = torch.stack([(dY[:, i, None] * X).sum(-1) for i in range(n)], 1)
            outs.append((Y.float(), dX.float(), _vjp(P, one, dP)))
    return tuple(torch.cat(k) for k in zip(*outs))
