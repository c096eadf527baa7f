"""Timed cases of the framework: quantizing one linear layer and using the
quantized layer, each through the package's public calls.

Two kinds of program use this package.  One quantizes a model layer by layer:
calibration activations of a layer are on the GPU, and the layer is quantized
in one call (``quantize_layer``), or in the staged form (``LayerSolver``) when
the activations come in chunks, when several JTA knobs are wanted on one
factor, or when damping and knob are searched per layer.  The other applies
quantized layers (``pack_codes``, ``dequant_matmul``): over whole calibration
sequences to form the next layer's runtime activations, or over the few
tokens of a decoding step.

Inputs are synthetic with the distributions of the package's own workloads:
Gaussian weights, activations with log-normal channel scales and 1% outlier
channels, runtime activations 2% away from the full-precision ones.
"""

import math

import torch

import paper_2602_08376_amd as ok

LAMBDA = 0.01

# Estimated seconds of a drawn case: below the largest listed one's time.
_COST_LIMIT = 0.9


def listed():
    layer = dict(kind="layer", alpha=0.5, scheme="asym", order="none")
    staged = dict(kind="sweep", scheme="asym", order="none")
    product = dict(kind="product", group=128, perm=False)
    return [
        # a toy layer as unit tests and smoke checks quantize it: latency and
        # launches only
        dict(layer, name="tiny layer 64x128", n=64, m=128, T=512, bits=4, group=128, K=4),
        # sizes that divide nothing, a ragged last group and token rows
        # without 16-byte alignment; act order with the scale groups of W
        dict(layer, name="ragged layer 1000x2500", n=1000, m=2500, T=20001, bits=3, group=128,
             K=8, scheme="sym", order="static"),
        # the attention projection of a 7B model on 128 x 2048 tokens: the
        # benchmark's default workload
        dict(layer, name="attention 4096x4096", n=4096, m=4096, T=262144, bits=4, group=128, K=16),
        # its MLP down projection: the wide lattice, 3-bit codes
        dict(layer, name="down_proj 4096x11008", n=4096, m=11008, T=262144, bits=3, group=128,
             K=16),
        # a 13B up projection with the JTA knob swept over {0, 0.5, 1} on one
        # factor and many Klein samples: the decoder's share at its largest
        dict(staged, name="up_proj sweep 13824x5120", n=13824, m=5120, T=262144, chunks=1, bits=3,
             group=128, K=32, mus=3),
        # a shard of a 70B down projection, activations streamed in chunks:
        # the largest lattice (blocked factor, triangular solve)
        dict(staged, name="shard 8192x28672", n=8192, m=28672, T=16384, chunks=2, bits=4,
             group=128, K=16, mus=1),
        # per-layer search of damping and knob on sums that are already there:
        # two factors, two knobs each
        dict(kind="search", name="knob search 4096x4096", n=4096, m=4096, T=32768, bits=4,
             group=128, K=16, lambdas=2, mus=2, scheme="asym", order="none"),
        # packing the codes of an 8B up projection for storage and use
        dict(kind="pack", name="pack 14336x4096", n=14336, m=4096, bits=4, perm=False),
        # the quantized layer over 16 calibration sequences (X~ of the next
        # layer, or prefill)
        dict(product, name="product prefill 32768", n=4096, m=4096, T=32768, bits=4),
        # an odd number of tokens, 3-bit fields across words, codes packed in
        # act order
        dict(product, name="product ragged 1999", n=4096, m=11008, T=1999, bits=3, perm=True),
        # one token: a decoding step
        dict(product, name="product decode 1", n=4096, m=4096, T=1, bits=4),
        # a small batch of decoding sequences
        dict(product, name="product decode 24", n=14336, m=4096, T=24, bits=4),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def size(lo, hi, step):
        """Log-uniform; half of the draws multiples of `step`, half any number."""
        v = log_int(lo, hi)
        return max(lo, v // step * step) if rng.random() < 0.5 else v

    while True:
        kind = rng.choice(["layer", "layer", "layer", "sweep", "search", "pack", "product",
                           "product", "product"])
        bits = rng.choice([2, 3, 4, 4])
        if kind == "product":
            c = dict(kind=kind, n=size(1024, 14336, 128), m=size(1024, 14336, 128),
                     T=size(1, 32768, 8), bits=bits, group=rng.choice([64, 128, 128]),
                     perm=rng.random() < 0.3)
            if c["n"] * c["m"] * c["T"] > 1.1e12:
                continue
            return c
        if kind == "pack":
            return dict(kind=kind, n=size(1024, 14336, 128), m=size(1024, 14336, 128), bits=bits,
                        perm=rng.random() < 0.3)
        c = dict(kind=kind, n=size(64, 14336, 64), m=size(128, 14336, 64), T=size(512, 262144, 64),
                 bits=bits, group=rng.choice([64, 128, 128]), K=rng.choice([0, 5, 8, 16, 25]),
                 scheme=rng.choice(["asym", "asym", "sym"]),
                 order=rng.choice(["none", "none", "none", "position", "static"]))
        if kind == "layer":
            c["alpha"] = rng.choice([0.5, 0.6, 0.6, 1.0])
        else:
            c["mus"] = rng.choice([1, 2, 3]) if kind == "sweep" else rng.choice([1, 2])
            if kind == "sweep":
                c["chunks"] = rng.choice([1, 2, 4])
                c["T"] = max(c["chunks"], c["T"] // c["chunks"] * c["chunks"])
            else:
                c["lambdas"] = 2
                c["T"] = min(c["T"], 32768)
        if _cost(c) <= _COST_LIMIT and 8 * c["m"] * c["T"] <= 24e9:
            return c


def _cost(case):
    """A rough number of seconds of one pass, for the limit of draw()."""
    n, m, T, K = case["n"], case["m"], case["T"], case["K"]
    sums = 0 if case["kind"] == "search" else 3 * m * m * T / 2e14
    solves = case.get("mus", 1) * case.get("lambdas", 1)
    return (sums + case.get("lambdas", 1) * (2 * m ** 3 / 2e13 + m * 1e-6)
            + solves * (m * m * n * (K + 1) / 6e13 + 4 * m * m * n / 4e13))


# ---- inputs -----------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _activations(m, T, g):
    """(X_ref, X_q) [m, T] float32: log-normal channel scales with 1% of the
    channels 50 times larger, and X_q 2% of a channel's scale away."""
    sig = torch.exp(torch.randn(m, 1, generator=g, device="cuda"))
    out = torch.randperm(m, generator=g, device="cuda")[: max(1, round(0.01 * m))]
    sig[out] *= 50.0
    X = torch.empty(m, T, device="cuda")
    Xq = torch.empty(m, T, device="cuda")
    for r in range(0, m, 1024):
        e = min(m, r + 1024)
        X[r:e] = torch.randn(e - r, T, generator=g, device="cuda").mul_(sig[r:e])
        Xq[r:e] = torch.randn(e - r, T, generator=g, device="cuda").mul_(0.02 * sig[r:e]).add_(X[r:e])
    return X, Xq


def _weights(n, m, g):
    return torch.randn(n, m, generator=g, device="cuda").mul_(0.02)


_ORDERS = {"none": False, "position": True, "static": "static"}


def _mus(case):
    return [0.5, 0.0, 1.0][: case["mus"]]


def _lambdas(case):
    return [0.005, 0.02][: case["lambdas"]]


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    st = dict(case=case, seed=int(seed) % 1000)
    if kind in ("layer", "sweep", "search"):
        st["W"] = _weights(case["n"], case["m"], g)
        X, Xq = _activations(case["m"], case["T"], g)
        if kind == "layer":
            st["X"], st["Xq"] = X, Xq
        elif kind == "sweep":   # token chunks as they are streamed, each a tensor of its own
            c = case["chunks"]
            st["chunks"] = ([(X, Xq)] if c == 1 else
                            [(a.contiguous(), b.contiguous())
                             for a, b in zip(X.chunk(c, 1), Xq.chunk(c, 1))])
        else:
            s = _solver(case, st["seed"], keep_gram=True)
            s.accumulate(X, Xq)
            st["solver"] = s
        return st
    n, m, bits = case["n"], case["m"], case["bits"]
    codes = torch.randint(0, 1 << bits, (n, m), generator=g, device="cuda", dtype=torch.uint8)
    st["perm"] = (torch.randperm(m, generator=g, device="cuda").to(torch.int32)
                  if case["perm"] else None)
    if kind == "pack":
        st["codes"] = codes
        return st
    G = ok.num_groups(m, case["group"])
    # scales and zero points of min-max groups of Gaussian weights
    qmax = (1 << bits) - 1
    lo = 0.05 + 0.005 * torch.randn(n, G, generator=g, device="cuda")
    hi = 0.05 + 0.005 * torch.randn(n, G, generator=g, device="cuda")
    st["scales"] = (lo + hi) / qmax
    st["zeros"] = torch.round(lo / st["scales"])
    st["packed"] = ok.pack_codes(codes, bits, perm=st["perm"])
    sig = torch.exp(torch.randn(m, 1, generator=g, device="cuda"))
    X = torch.empty(m, case["T"], dtype=torch.float16, device="cuda")
    for r in range(0, m, 4096):
        e = min(m, r + 4096)
        X[r:e] = torch.randn(e - r, case["T"], generator=g, device="cuda").mul_(sig[r:e])
    st["X"] = X
    st["codes"] = codes if case["perm"] is False else codes[:, st["perm"].long()]
    return st


def _solver(case, seed, keep_gram=False):
    return ok.LayerSolver(case["m"], case["n"], case["bits"], case["group"], case["K"], seed,
                          lambda_rel=LAMBDA, scheme=case["scheme"],
                          act_order=_ORDERS[case["order"]], keep_gram=keep_gram)


def _result(q):
    return dict(codes=q.codes, scales=q.scales, zeros=q.zeros, residuals=q.residuals,
                winner=q.winner)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "layer":
        return _result(ok.quantize_layer(
            state["W"], state["X"], state["Xq"], case["alpha"], case["bits"], case["group"],
            case["K"], state["seed"], lambda_rel=LAMBDA, scheme=case["scheme"],
            act_order=_ORDERS[case["order"]]))
    if kind == "sweep":
        s = _solver(case, state["seed"])
        s.set_weights(state["W"])
        for X, Xq in state["chunks"]:
            s.accumulate(X, Xq)
        out = [_result(s.solve(state["W"], mu)) for mu in _mus(case)]
        s.close()
        return out
    if kind == "search":
        s = state["solver"]
        out = []
        for lam in _lambdas(case):
            s.set_knobs(lambda_rel=lam)
            out += [_result(s.solve(state["W"], mu)) for mu in _mus(case)]
        return out
    if kind == "pack":
        return ok.pack_codes(state["codes"], case["bits"], perm=state["perm"])
    return ok.dequant_matmul(state["packed"], state["scales"], state["zeros"], case["m"],
                             case["bits"], case["group"], state["X"], perm=state["perm"])


# ---- what a pass cannot do without --------------------------------------------


def work(case):
    n, m, kind = case["n"], case["m"], case["kind"]
    words = (m * case["bits"] + 31) // 32
    if kind == "pack":
        return dict(bytes=n * m + 4 * n * words, flops=0)
    G = ok.num_groups(m, case["group"])
    if kind == "product":
        T = case["T"]
        return dict(bytes=4 * n * words + 8 * n * G + 2 * m * T + 4 * n * T, flops=2 * n * m * T)
    T, K = case["T"], case["K"]
    solves = case.get("mus", 1) * case.get("lambdas", 1)
    crosses = case.get("alpha", 0.5) != 1.0
    # sums: half a Gram and the cross term (or its projection on the weights);
    # factor; relaxed solution of n columns; one triangular product per path
    sums = m * m * T + (min(2 * m * m, 4 * n * m) * T if crosses else 0)
    inputs = 4 * n * m + (8 if crosses else 4) * m * T
    if kind == "search":
        sums, inputs = 0, 4 * n * m + 8 * m * m
    solve = (2 if crosses else 1) * m * m * n + m * m * n * (K + 1)
    return dict(bytes=inputs + solves * (n * m + 8 * n * G + 12 * n),
                flops=sums + case.get("lambdas", 1) * m ** 3 / 3 + solves * solve)


def tolerance(case):
    kind = case["kind"]
    if kind == "pack":
        return "exact"
    if kind == "product":
        # float32 sums of m products of fp16 values
        return dict(rel=2.5e-6, max=3e-5)
    # Decisions at near-ties (a centre within the rounding of the sums of a
    # rounding boundary, a uniform within it of a weight sum) may go either
    # way; the column's later codes and its residual then differ a little
    # (one column of the narrowest layers: half a percent of the codes).
    return dict(rel=1e-4, max=0.02, differ=0.01)


# ---- the same in 64 bits --------------------------------------------------------


def exact(case, seed):
    kind = case["kind"]
    if kind == "pack":
        return None
    if kind == "product":
        return _exact_product(prepare(case, seed))
    paths = case["n"] * (case["K"] + 1)
    solves = case.get("mus", 1) * case.get("lambdas", 1)
    whole = (case["m"] <= 4096 and paths <= 70000 and solves == 1 and kind == "layer")
    if kind == "layer" and not whole and case["order"] != "position":
        # scales and zero points depend on the weights alone
        S, Z = _exact_scales(_weights(case["n"], case["m"], _gen(seed)).double(), case)
        return dict(codes=None, scales=S, zeros=Z, residuals=None, winner=None)
    return _exact_layer(prepare(case, seed)) if whole else None


def _exact_product(st):
    case = st["case"]
    m, g = case["m"], case["group"]
    S = st["scales"].double().repeat_interleave(g, 1)[:, :m]
    Z = st["zeros"].double().repeat_interleave(g, 1)[:, :m]
    # W_hat as it is defined: the product in float32, then in fp16
    W = ((S * (st["codes"].double() - Z)).float().half()).double()
    X = st["X"] if st["perm"] is None else st["X"][st["perm"].long()]
    Y = torch.empty(case["n"], case["T"], dtype=torch.float64, device="cuda")
    for t in range(0, case["T"], 4096):
        Y[:, t:t + 4096] = W @ X[:, t:t + 4096].double()
    return Y


def _exact_scales(W, case):
    """(S, Z) [n, G] of the groups of W's columns, S rounded to float32 as stored."""
    n, m = W.shape
    g = min(case["group"], m)
    G = ok.num_groups(m, case["group"])
    P = torch.zeros(n, G * g, dtype=torch.float64, device=W.device)
    P[:, :m] = W
    P = P.view(n, G, g)
    if case["scheme"] == "sym":
        a = P.abs().amax(2)
        half = 1 << (case["bits"] - 1)
        S = (torch.where(a == 0, 1.0, a) / (half - 1)).float().double()
        return S, torch.full_like(S, half)
    lo, hi = P.amin(2).clamp(max=0.0), P.amax(2).clamp(min=0.0)
    none = lo == hi
    lo, hi = torch.where(none, -1.0, lo), torch.where(none, 1.0, hi)
    S = ((hi - lo) / ((1 << case["bits"]) - 1)).float().double()
    return S, torch.round(-lo / S)


def _log_rho(m, K):
    """ln(rho) with K = (e rho)^(2 m / rho)."""
    if K <= 1:
        return math.inf
    if math.log(K) >= 2 * m:
        return 0.0
    lo, hi = 0.0, 100.0
    for _ in range(200):
        x = 0.5 * (lo + hi)
        lo, hi = (x, hi) if 2 * m * (1 + x) * math.exp(-x) > math.log(K) else (lo, x)
    return 0.5 * (lo + hi)


def _uniform(seed, i, j, k):
    """Philox4x32-10 of counter (i, j, k, 0) and key (seed, 0), as a double in [0, 1)."""
    mask = 0xFFFFFFFF
    c0, c1, c2, c3 = torch.full_like(j, i), j, k, torch.zeros_like(j)
    k0, k1 = seed & mask, seed >> 32
    for r in range(10):
        if r:
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57   # the bits of the 64-bit products
        c0, c1, c2, c3 = (((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask,
                          ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask)
    return ((c0 >> 5).double() * 67108864.0 + (c1 >> 6).double()) / 9007199254740992.0


def _exact_layer(st):
    case = st["case"]
    n, m, K, bits = case["n"], case["m"], case["K"], case["bits"]
    qmax = (1 << bits) - 1
    W = st["W"].double()
    H = torch.zeros(m, m, dtype=torch.float64, device="cuda")
    E = torch.zeros_like(H)
    for t in range(0, case["T"], 8192):
        Xq = st["Xq"][:, t:t + 8192].double()
        D = st["X"][:, t:t + 8192].double() - Xq
        H += Xq @ Xq.T
        E += Xq @ D.T
    perm = torch.arange(m, device="cuda")
    group = perm // min(case["group"], m)
    if case["order"] != "none":
        perm = torch.sort(torch.diagonal(H), stable=True).indices
        H, E = H[perm][:, perm], E[perm][:, perm]
    Wp = W[:, perm]
    if case["order"] == "static":
        S, Z = _exact_scales(W, case)
        group = group[perm]
    else:
        S, Z = _exact_scales(Wp, case)
    H.diagonal().add_(LAMBDA * torch.diagonal(H).mean())
    L = torch.linalg.cholesky(H.cpu())
    V = torch.cholesky_solve((E @ Wp.T).cpu(), L).cuda()
    L = L.cuda()
    Sx = S[:, group]                                           # [n, m]
    target = Wp + (1.0 - case["alpha"]) * V.T + Sx * Z[:, group]   # s qbar
    gq = (target @ L).T                                        # R (s qbar), [m, n]
    kp1 = K + 1
    col = torch.arange(n, device="cuda").repeat_interleave(kp1)
    kk = torch.arange(kp1, device="cuda").repeat(n)
    alpha = _log_rho(m, K) / ((torch.diagonal(L) * Sx) ** 2).amin(1)
    box = torch.arange(qmax + 1, dtype=torch.float64, device="cuda")
    E_ = torch.zeros(m, n * kp1, dtype=torch.float64, device="cuda")   # s q of the decided rows
    Q = torch.zeros(m, n * kp1, dtype=torch.uint8, device="cuda")
    resid = torch.zeros(n * kp1, dtype=torch.float64, device="cuda")
    for b in range((m - 1) // 64 * 64, -1, -64):
        e = min(m, b + 64)
        z = gq[b:e][:, col] - L[e:, b:e].T @ E_[e:]
        for i in range(e - 1, b - 1, -1):
            s = Sx[:, i][col]
            rb = L[i, i] * s
            c = z[i - b] / rb
            q = torch.round(c).clamp(0, qmax)
            if K > 1:
                kappa = alpha[col] * rb * rb
                lw = -kappa[:, None] * (c[:, None] - box) ** 2
                cum = torch.exp(lw - lw.amax(1, keepdim=True)).cumsum(1)
                hit = (_uniform(st["seed"], i, col, kk) * cum[:, -1])[:, None] < cum
                q = torch.where(kk > 0, (~hit).sum(1).clamp(max=qmax).double(), q)
            resid += (rb * (q - c)) ** 2
            Q[i] = q.to(torch.uint8)
            E_[i] = s * q
            if i > b:
                z[: i - b] -= L[i, b:i][:, None] * E_[i][None, :]
    resid = resid.view(n, kp1)
    best = resid.argmin(1)
    codes = torch.empty(n, m, dtype=torch.uint8, device="cuda")
    codes[:, perm] = Q.T[torch.arange(n, device="cuda") * kp1 + best]
    return dict(codes=codes, scales=S, zeros=Z, residuals=resid.gather(1, best[:, None])[:, 0],
                winner=best.to(torch.int32))
