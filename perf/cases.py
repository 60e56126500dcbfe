"""Performance cases of the attention backward-over-backward path.

Each case is one call, or the chain of calls, that a program makes through the
public entry points of paper_2609_24089_amd:

  fwd   attn_fwd_lse: inference, or the first half of a training step
  grad  attn_fwd_lse + attn_bwd: an ordinary training step of the layer
  bob   bob(): forward, first backward, BoB Pass 1 and Pass 2 (all outputs)
  hvp   attention() under torch.autograd: a Hessian-vector product of a
        squared-error loss through the layer (forward, first backward with
        create_graph, and the double backward, which adds a second first
        backward for the loss curvature)

A case is a dict: entry, dtype ("bf16" or "f32"), B, H, Hkv (key/value heads),
N, d, causal, qk (the factor on Q and K, as in the workload recipe).
"""
import math

import torch

import paper_2609_24089_amd as fb


def _case(name, entry, B, H, N, d, dtype="bf16", Hkv=None, causal=False, qk=1.0):
    return {"name": name, "entry": entry, "dtype": dtype, "B": B, "H": H, "Hkv": Hkv or H, "N": N, "d": d,
            "causal": causal, "qk": qk}


def listed():
    return [
        # the smallest workload of the repository: one head, fp32, latency and launches
        _case("tiny_f32_bob", "bob", 1, 1, 256, 64, dtype="f32"),
        # one short sequence through a 12-head layer: a curvature probe inside a small model
        _case("short_causal_hvp", "hvp", 1, 12, 1024, 64, causal=True),
        # a ragged length and few heads: neither the tiles nor the grid come out even
        _case("ragged_bob", "bob", 2, 4, 777, 128),
        # prefill of one prompt with grouped key/value heads
        _case("prefill_gqa_fwd", "fwd", 1, 32, 2048, 128, Hkv=8, causal=True),
        # an ordinary training step (no double backward) at the causal B4 H12 shape
        _case("train_causal_grad", "grad", 4, 12, 4096, 64, causal=True),
        # the small dense benchmark configuration
        _case("dense_n4096_d64_bob", "bob", 2, 8, 4096, 64),
        # the benchmark's headline configuration, the largest case
        _case("dense_n16384_d128_bob", "bob", 1, 16, 16384, 128, qk=0.5),
        # one long single-head sequence, as in the length sweep
        _case("long_single_head_bob", "bob", 1, 1, 65536, 64),
        # head-dim sweep at the causal B4 H12 shape: the narrowest heads
        _case("causal_n4096_d32_bob", "bob", 4, 12, 4096, 32, causal=True),
        # the widest heads
        _case("dense_n8192_d256_bob", "bob", 1, 16, 8192, 256),
        # grouped key/value heads, causal, ragged length
        _case("gqa_causal_n4099_bob", "bob", 1, 16, 4099, 128, Hkv=4, causal=True),
        # fp32 end to end: verification runs and optimizers that keep curvature in fp32
        _case("f32_causal_bob", "bob", 2, 8, 2000, 64, dtype="f32", causal=True),
    ]


def _pairs(c):
    """Unmasked (query, key) pairs of all query heads."""
    n = c["N"]
    return c["B"] * c["H"] * (n * (n + 1) // 2 if c["causal"] else n * n)


# Contractions of 2 d FLOPs per (query, key) pair that each step needs: forward
# 2 (S, P V); first backward 5 (S, dP, dQ, dK, dV); BoB 12 (the closed form's
# minimum: S, dP, two for F, C and seven output contractions).
_CONTRACTIONS = {"fwd": 2, "grad": 2 + 5, "bob": 2 + 5 + 12, "hvp": 2 + 5 + 12 + 5}


def _cost(c):
    """Work in units that compare the two data types (fp32 MFMA runs at 1/16 of the bf16 rate)."""
    return _pairs(c) * 2 * c["d"] * _CONTRACTIONS[c["entry"]] * (16 if c["dtype"] == "f32" else 1)


def draw(rng):
    top = max(_cost(c) for c in listed())
    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        d = rng.choice((32, 64, 64, 64, 128, 128, 128) if dtype == "f32" else (32, 64, 64, 64, 128, 128, 128, 256))
        G = rng.choice((1, 1, 1, 1, 2, 4, 8))
        Hkv = rng.choice((1, 2, 3, 4, 6, 8, 12, 16))
        entry = rng.choice(("fwd", "grad", "grad", "bob", "bob", "bob", "bob", "hvp", "hvp"))
        N = int(round(math.exp(rng.uniform(math.log(64), math.log(65536)))))
        if rng.random() < 0.4:  # whole tiles, as many programs pad to
            N = max(64, N // 64 * 64)
        c = {"entry": entry, "dtype": dtype, "B": rng.choice((1, 1, 1, 2, 4)), "H": Hkv * G, "Hkv": Hkv, "N": N,
             "d": d, "causal": rng.random() < 0.5, "qk": rng.choice((0.5, 1.0))}
        if c["H"] <= 48 and _cost(c) <= top:
            return c


def _inputs(case, seed):
    """Q, K, V, dO, U_Q, U_K, U_V by the workload recipe (N(0, 1), Q and K times qk, cast to the type)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    out = {}
    for name in ("Q", "K", "V", "dO", "UQ", "UK", "UV"):
        h = case["Hkv"] if name in ("K", "V", "UK", "UV") else case["H"]
        x = torch.randn((case["B"], h, case["N"], case["d"]), generator=gen, device="cuda", dtype=torch.float32)
        if name in ("Q", "K"):
            x = x * case["qk"]
        out[name] = x.to(dt)
    return out


def _scale(case):
    return 1.0 / math.sqrt(case["d"])


def prepare(case, seed):
    x = _inputs(case, seed)
    st = {"case": dict(case), "scale": _scale(case), **x}
    if case["entry"] == "hvp":
        for name in ("Q", "K", "V"):
            st[name].requires_grad_(True)
    return st


def run(st):
    c, scale = st["case"], st["scale"]
    causal = bool(c["causal"])
    q, k, v = st["Q"], st["K"], st["V"]
    if c["entry"] == "fwd":
        O, L = fb.attn_fwd_lse(q, k, v, scale, causal)
        return {"O": O, "L": L}
    if c["entry"] == "grad":
        O, L = fb.attn_fwd_lse(q, k, v, scale, causal)
        dQ, dK, dV, D = fb.attn_bwd(q, k, v, O, st["dO"], L, scale, causal)
        return {"O": O, "L": L, "D": D, "dQ": dQ, "dK": dK, "dV": dV}
    u = (st["UQ"], st["UK"], st["UV"])
    if c["entry"] == "bob":
        return fb.bob(q, k, v, st["dO"], *u, scale, causal)
    # Hessian-vector product of |O - Y|^2 / 2 along (U_Q, U_K, U_V); the target Y is st["dO"]
    O = fb.attention(q, k, v, scale, causal)
    g = torch.autograd.grad(O, (q, k, v), grad_outputs=O - st["dO"], create_graph=True)
    h = torch.autograd.grad(g, (q, k, v), grad_outputs=u)
    return {"O": O.detach(), "dQ": g[0].detach(), "dK": g[1].detach(), "dV": g[2].detach(), "hQ": h[0], "hK": h[1],
            "hV": h[2]}


def work(case):
    flops = _pairs(case) * 2 * case["d"] * _CONTRACTIONS[case["entry"]]
    size = 4 if case["dtype"] == "f32" else 2
    qn = case["B"] * case["H"] * case["N"]
    kn = case["B"] * case["Hkv"] * case["N"]
    # (query-side matrices, key-side matrices, fp32 row vectors) read once or written once
    q, k, r = {"fwd": (2, 2, 1), "grad": (4, 4, 2), "bob": (7, 8, 4), "hvp": (6, 8, 0)}[case["entry"]]
    return {"bytes": (q * qn + k * kn) * case["d"] * size + r * qn * 4, "flops": flops}


def tolerance(case):
    # bf16: MFMA operands and outputs carry 8 bits; two layouts of the column
    # kernels differ by up to 2.5e-3 in the 2-norm.  fp32: sums in another order.
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}


def exact(case, seed):
    """The closed forms in float64, a block of query rows of one head at a time."""
    x = {n: t.double() for n, t in _inputs(case, seed).items()}
    B, H, Hkv, N, d = (case[n] for n in ("B", "H", "Hkv", "N", "d"))
    entry, tau, G = case["entry"], _scale(case), case["H"] // case["Hkv"]
    second = entry in ("bob", "hvp")
    like_q, like_k = (lambda: torch.zeros_like(x["Q"])), (lambda: torch.zeros_like(x["K"]))
    rows_like = lambda: torch.zeros(B, H, N, dtype=torch.float64, device="cuda")  # noqa: E731
    r = {n: like_q() for n in ("O", "dQ", "Qt", "dOt", "cQ")}
    r.update({n: like_k() for n in ("dK", "dV", "Kt", "Vt", "cK", "cV")})
    r.update({n: rows_like() for n in ("L", "D", "alpha", "E")})
    step = max(1, min(N, (1 << 26) // N))
    key = torch.arange(N, device="cuda")
    for b in range(B):
        for h in range(H):
            kh = h // G
            K, V = x["K"][b, kh], x["V"][b, kh]
            for i in range(0, N, step):
                s = slice(i, min(N, i + step))
                Q = x["Q"][b, h, s]
                S = tau * (Q @ K.T)
                if case["causal"]:
                    S.masked_fill_(key[None, :] > key[s, None], -math.inf)
                L = torch.logsumexp(S, 1)
                P = torch.exp(S - L[:, None])
                del S
                O = P @ V
                r["O"][b, h, s], r["L"][b, h, s] = O, L
                if entry == "fwd":
                    continue
                dO = O - x["dO"][b, h, s] if entry == "hvp" else x["dO"][b, h, s]
                D = (dO * O).sum(1)
                dP = dO @ V.T
                dS = P * (dP - D[:, None])
                r["D"][b, h, s] = D
                r["dQ"][b, h, s] = tau * (dS @ K)
                r["dK"][b, kh] += tau * (dS.T @ Q)
                r["dV"][b, kh] += P.T @ dO
                if not second:
                    continue
                UQ, UK, UV = x["UQ"][b, h, s], x["UK"][b, kh], x["UV"][b, kh]
                F = tau * (UQ @ K.T + Q @ UK.T)
                alpha = (P * F).sum(1)
                Pt = dO @ UV.T + F * (dP - D[:, None]) - alpha[:, None] * dP
                E = (P * Pt).sum(1)
                Ph = P * (F - alpha[:, None])
                del F, dP
                St = P * (Pt - E[:, None])
                del Pt
                dOt = P @ UV + Ph @ V
                r["alpha"][b, h, s], r["E"][b, h, s], r["dOt"][b, h, s] = alpha, E, dOt
                r["Qt"][b, h, s] = tau * (St @ K + dS @ UK)
                r["Kt"][b, kh] += tau * (St.T @ Q + dS.T @ UQ)
                r["Vt"][b, kh] += Ph.T @ dO
                if entry == "hvp":  # the loss curvature: a first backward with upstream dOt
                    dS = P * (dOt @ V.T - (dOt * O).sum(1)[:, None])
                    r["cQ"][b, h, s] = tau * (dS @ K)
                    r["cK"][b, kh] += tau * (dS.T @ Q)
                    r["cV"][b, kh] += P.T @ dOt
    if entry == "hvp":
        return {"O": r["O"], "dQ": r["dQ"], "dK": r["dK"], "dV": r["dV"], "hQ": r["Qt"] + r["cQ"],
                "hK": r["Kt"] + r["cK"], "hV": r["Vt"] + r["cV"]}
    names = {"fwd": ("O", "L"), "grad": ("O", "L", "D", "dQ", "dK", "dV"),
             "bob": ("Qt", "Kt", "Vt", "dOt", "alpha", "E", "O", "L", "D", "dQ", "dK", "dV")}[entry]
    return {n: r[n] for n in names}
