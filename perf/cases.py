"""Performance cases: the calls that a program makes of this library, with their sizes.

Each case is one pass through the public entry points, on tensors a training or serving
program has in hand.  Kinds of pass:

  step       hash Q and K, forward, backward (a training step of one attention layer)
  train      forward and backward on codes in hand (the backward reuses the forward's codes)
  infer      N-YOSO inference: l2-normalise Q and K, hash them, forward, l2-normalise Y
  star       *YOSO's backward on codes in hand
  expect     YOSO-E, forward or backward
  noalloc    the backward that allocates nothing, outputs in place (serving loops, graph capture)
  hash       Q and K hashed, by the dense projection or by the fast hash

Sizes are those of workloads.py (BERT-base at 512 tokens, the LRA lengths, two longer
contexts) and odd ones of the same ranges.  Inputs as there: Q, K unit rows (Gaussian, or 16
clustered directions per head), V and dY Gaussian, R Gaussian.  Codes "in hand" are those of
Q and K under R, signs taken in 64 bits.
"""
from __future__ import annotations

import math

import torch

import paper_2111_09714_amd as Y

D = 64


def listed():
    return [
        # one sequence of one head: launches and latency (a single request)
        _case("step_1x512", "step", bh=1, n=512),
        # BERT-base at 512 tokens, batch 32: many heads of short sequences
        _case("train_384x512", "train", bh=384, n=512),
        # LRA at 4K tokens, batch 16, two heads: the workload of bench.py
        _case("step_32x4096", "step", bh=32, n=4096),
        # a long sequence whose rows cluster: skewed buckets
        _case("train_32x16384_clustered", "train", bh=32, n=16384, m=16, dist="clustered"),
        # the longest context, 16-bit storage
        _case("train_24x32768_bf16", "train", bh=24, n=32768, tau=9, dtype="bf16"),
        # inference at an odd length, 16-bit storage, with the normalisations around it
        _case("infer_192x1000_bf16", "infer", bh=192, n=1000, dtype="bf16"),
        # cross attention: ragged sides of different length, few hashes
        _case("train_64x1500x1030_bf16", "train", bh=64, n=1500, n_k=1030, m=16, tau=7, dtype="bf16"),
        # *YOSO (the true gradient's estimate) at the LRA text length
        _case("star_16x2000", "star", bh=16, n=2000),
        # YOSO-E at the LRA length, and its training pass on BERT-like lengths in 16 bits
        _case("expect_fwd_32x4096", "expect", bh=32, n=4096, backward=False),
        _case("expect_bwd_96x1000_bf16", "expect", bh=96, n=1000, dtype="bf16", backward=True),
        # one head of medium length in a serving loop that may not allocate
        _case("noalloc_1x2048", "noalloc", bh=1, n=2048),
        # the hash alone: Q and K of a BERT-base batch
        _case("hash_384x512", "hash", bh=384, n=512, fast=False),
    ]


def _case(name, kind, bh, n, n_k=None, m=32, tau=8, dtype="f32", dist="gauss", backward=True, fast=False):
    return {"name": name, "kind": kind, "bh": bh, "n": n, "n_k": n if n_k is None else n_k, "m": m, "tau": tau,
            "dtype": dtype, "dist": dist, "backward": backward, "fast": fast}


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["step", "train", "train", "infer", "star", "expect", "noalloc", "hash"])
    # (rows per side, and pairs, at most those of the largest listed case of the kind)
    top_n, rows, pairs = {"step": (8192, 1 << 17, 1 << 29), "train": (32768, 1 << 19, 1 << 33),
                          "infer": (8192, 1 << 18, 1 << 31), "star": (2048, 1 << 15, 1 << 26),
                          "expect": (4096, 1 << 17, 1 << 28), "noalloc": (3072, 3072, 1 << 24),
                          "hash": (32768, 1 << 18, 1 << 62)}[kind]
    n = _log_int(rng, 100, top_n)
    n_k = n
    if kind in ("step", "train", "noalloc") and rng.random() < 0.3:
        n_k = _log_int(rng, max(100, n // 4), min(top_n, 4 * n))
    most = max(1, min(rows // max(n, n_k), pairs // (n * n_k)))
    bh = 1 if kind == "noalloc" else _log_int(rng, 1, min(most, 384))
    tau = rng.choice([6, 7, 8, 8, 9, 10])
    m = rng.choice([8, 16, 24, 32, 32, 48])
    if kind == "noalloc":
        m = min(m, 32)
    return {"kind": kind, "bh": bh, "n": n, "n_k": n_k, "m": m, "tau": tau, "dtype": rng.choice(["f32", "bf16"]),
            "dist": rng.choice(["gauss", "gauss", "clustered"]), "backward": rng.random() < 0.5,
            "fast": kind == "hash" and rng.random() < 0.5}


# ------------------------------------------------------------------ inputs

def _device():
    return torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")


def _inputs(case, seed):
    """Q, K, V, dY [bh, n, 64], R [64, m tau], the fast hash's signs; `scaled` Q and K rows for the
    chain that normalises them itself."""
    dev = _device()
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    bh, n_q, n_k, m, tau = case["bh"], case["n"], case["n_k"], case["m"], case["tau"]

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=dev)

    def unit(x):
        return x / x.norm(dim=-1, keepdim=True)

    if case["dist"] == "clustered":
        centres = unit(normal(bh, 16, D))

        def rows(n):
            pick = torch.randint(16, (bh, n, 1), generator=g, device=dev).expand(bh, n, D)
            return unit(centres.gather(1, pick) + 0.1 * normal(bh, n, D))
    else:
        def rows(n):
            return unit(normal(bh, n, D))
    q, k = rows(n_q), rows(n_k)
    if case["kind"] == "infer":
        q, k = 8.0 * q, 8.0 * k  # projections as a layer gives them, not yet normalised
    inp = {"q": q.to(dt), "k": k.to(dt), "v": normal(bh, n_k, D).to(dt), "dy": normal(bh, n_q, D).to(dt),
           "R": normal(D, m * tau)}
    nrot = (m * tau + 63) // 64
    inp["signs"] = torch.randint(-2**63, 2**63 - 1, (nrot, 3), generator=g, device=dev, dtype=torch.int64)
    return inp


def _codes64(x, R, m, tau):
    """The codes of the rows of x under R, [bh, n, m] int16, signs of projections taken in 64 bits."""
    bh, n, _ = x.shape
    out = torch.empty(bh, n, m, dtype=torch.int16, device=x.device)
    R64 = R.double()
    weights = (2 ** torch.arange(tau, device=x.device)).to(torch.int64)
    flat, res = x.reshape(-1, D), out.view(-1, m)
    for i in range(0, flat.shape[0], 1 << 17):
        bits = (flat[i:i + (1 << 17)].double() @ R64) > 0
        res[i:i + (1 << 17)] = (bits.view(-1, m, tau).long() * weights).sum(-1).to(torch.int16)
    return out


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    kind, m, tau = case["kind"], case["m"], case["tau"]
    if kind in ("train", "star", "noalloc"):
        s["qc"], s["kc"] = _codes64(s["q"], s["R"], m, tau), _codes64(s["k"], s["R"], m, tau)
    if kind == "expect":
        s["out"] = [torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])]
    if kind == "noalloc":
        s["out"] = [torch.empty_like(s["q"]), torch.empty_like(s["k"]), torch.empty_like(s["v"])]
    return s


def run(s):
    c = s["case"]
    kind, m, tau = c["kind"], c["m"], c["tau"]
    if kind == "hash":
        if c["fast"]:
            return Y.fast_hash_qk(s["q"], s["k"], s["signs"], m, tau)
        return Y.hash_qk(s["q"], s["k"], s["R"], m, tau)
    if kind == "infer":
        q, k = torch.empty_like(s["q"]), torch.empty_like(s["k"])
        Y.yoso_l2_normalize(s["q"], q)
        Y.yoso_l2_normalize(s["k"], k)
        qc, kc = Y.hash_qk(q, k, s["R"], m, tau)
        y = Y.forward(qc, kc, s["v"], m, tau)
        out = torch.empty_like(y)
        Y.yoso_l2_normalize(y, out)
        return out
    if kind == "expect":
        dq, dk, dv = s["out"]
        if c["backward"]:
            Y.yoso_expectation_backward(s["q"], s["k"], s["v"], s["dy"], tau, dq, dk, dv)
            return dq, dk, dv
        Y.yoso_expectation_forward(s["q"], s["k"], s["v"], tau, dq)
        return dq
    if kind == "star":
        return Y.backward_star(s["qc"], s["kc"], s["q"], s["k"], s["v"], s["dy"], m, tau)
    if kind == "noalloc":
        dq, dk, dv = s["out"]
        Y.yoso_backward_noalloc(s["qc"], s["kc"], s["q"], s["k"], s["v"], s["dy"], m, tau, dq, dk, dv)
        return dq, dk, dv
    if kind == "step":
        qc, kc = Y.hash_qk(s["q"], s["k"], s["R"], m, tau)
        y = Y.forward(qc, kc, s["v"], m, tau)
        return (qc, kc, y) + tuple(Y.backward(qc, kc, s["q"], s["k"], s["v"], s["dy"], m, tau))
    y = Y.forward(s["qc"], s["kc"], s["v"], m, tau)
    return (y,) + tuple(Y.backward(s["qc"], s["kc"], s["q"], s["k"], s["v"], s["dy"], m, tau))


# ------------------------------------------------------------------ work

def work(case):
    """Bytes: inputs read once, outputs written once.  Operations: the products named in the
    comments, over the (query, key) pairs that collide (at most all of them; buckets of uniform
    codes) or, where that is less, over each row's bucket matrix."""
    bh, nq, nk, m, tau = case["bh"], case["n"], case["n_k"], case["m"], case["tau"]
    e = 2 if case["dtype"] == "bf16" else 4
    rq, rk = bh * nq, bh * nk
    codes = 2 * m * (rq + rk)
    hash_bytes = e * D * (rq + rk) + 4 * D * m * tau
    hash_flops = (3 * 6 * 64 * ((m * tau + 63) // 64) if case["fast"] else 2 * D * m * tau) * (rq + rk)
    fwd_bytes, fwd_flops = e * D * (rq + rk), m * D * (rq + rk)
    # dQ, dK: a scalar product and two row sums per pair, or 2 d^2 multiply-adds per row and hash; dV as the forward
    pairs = min(bh * nq * nk, m * bh * nq * nk / 2**tau)
    bwd_bytes = e * D * (3 * rq + 4 * rk)
    bwd_flops = min(6 * D * pairs, 4 * D * D * m * (rq + rk)) + fwd_flops
    kind = case["kind"]
    if kind == "hash":
        return {"bytes": hash_bytes + codes, "flops": hash_flops}
    if kind == "infer":
        return {"bytes": hash_bytes + fwd_bytes, "flops": hash_flops + fwd_flops + 4 * D * (2 * rq + rk)}
    if kind == "expect":
        if case["backward"]:  # two scalar products and three row sums per pair
            return {"bytes": bwd_bytes, "flops": 10 * D * bh * nq * nk}
        return {"bytes": e * D * (2 * rq + 2 * rk), "flops": 4 * D * bh * nq * nk}
    if kind == "star":  # two scalar products, two row sums per pair of codes at most one bit apart
        near = min(bh * nq * nk, m * (tau + 1) * bh * nq * nk / 2**tau)
        return {"bytes": bwd_bytes + codes, "flops": 8 * D * near + fwd_flops}
    if kind == "noalloc":
        return {"bytes": bwd_bytes + codes, "flops": bwd_flops}
    if kind == "step":  # Q, K, V, dY in; codes, Y, dQ, dK, dV out
        return {"bytes": hash_bytes + codes + e * D * (3 * rq + 3 * rk), "flops": hash_flops + fwd_flops + bwd_flops}
    return {"bytes": codes + e * D * (4 * rq + 4 * rk), "flops": fwd_flops + bwd_flops}


# ------------------------------------------------------------------ tolerance and exact values

def tolerance(case):
    """About four times what a comparison with `exact` showed at the listed sizes."""
    kind, bf16 = case["kind"], case["dtype"] == "bf16"
    if kind == "hash":
        # signs of projections near zero (1e-6 of the codes)
        return {"rel": 0.0, "differ": 1e-5}
    if kind in ("infer", "step"):
        # whole calls: a sign that flips in the hash moves one of the m samples of a row (1e-3
        # of the result, and 2.6e-3 with the rounding to bf16)
        return {"rel": 1.1e-2 if bf16 else 4.5e-3, "max": 0.9, "differ": 1e-5}
    # rounding to bf16 (1.7e-3, at most 4.2e-3); fp32: 1e-7 to 1.2e-6, at most 1.3e-5
    return {"rel": 7e-3, "max": 2e-2} if bf16 else {"rel": 5e-6, "max": 6e-5}


def exact(case, seed):
    kind, bh, nq, nk = case["kind"], case["bh"], case["n"], case["n_k"]
    m, tau = case["m"], case["tau"]
    if bh * nq * nk * (m if kind != "expect" else 8) > (1 << 40) or (not torch.cuda.is_available() and bh * nq * nk > 1 << 22):
        return None
    s = _inputs(case, seed)
    if kind == "hash":
        if case["fast"]:
            return None, None
        return _codes64(s["q"], s["R"], m, tau), _codes64(s["k"], s["R"], m, tau)
    q64, k64 = s["q"].double(), s["k"].double()
    if kind == "infer":
        q64, k64 = (x / x.norm(dim=-1, keepdim=True) for x in (q64, k64))
        # (the chain stores the normalised rows in the case's type and hashes those)
        qc, kc = (_codes64(x.to(s["q"].dtype), s["R"], m, tau) for x in (q64, k64))
    elif kind != "expect":
        qc, kc = _codes64(s["q"], s["R"], m, tau), _codes64(s["k"], s["R"], m, tau)
    v64, dy64 = s["v"].double(), s["dy"].double()
    y, dq = torch.zeros_like(dy64), torch.zeros_like(q64)
    dk, dv = torch.zeros_like(k64), torch.zeros_like(v64)
    grads = kind in ("step", "train", "star", "noalloc") or (kind == "expect" and case["backward"])
    rows = max(1, (1 << 27) // nk)
    for b in range(bh):
        for i in range(0, nq, rows):
            sl = slice(i, min(nq, i + rows))
            if kind == "expect":
                qn, kn = (x / x.norm(dim=-1, keepdim=True) for x in (q64[b, sl], k64[b]))
                P = (1 - torch.acos((qn @ kn.T).clamp(-1, 1)) / math.pi) ** tau
                W = (tau / 2) * P
            else:
                C = torch.zeros(sl.stop - i, nk, dtype=torch.int16, device=q64.device)
                near = torch.zeros_like(C) if kind == "star" else None
                for h in range(m):
                    a, c = qc[b, sl, h, None], kc[b, None, :, h]
                    C += a == c
                    if kind == "star":
                        x = a ^ c
                        near += (x & (x - 1)) == 0  # equal, or one bit apart
                P = C.double() / m
                if kind == "star":
                    x = q64[b, sl] @ k64[b].T
                    W = (near + (tau - 1) * C).double() / m / (math.pi * (1 - x * x).clamp(min=1 / 64).sqrt())
                else:
                    W = (tau / 2) * P
            y[b, sl] = P @ v64[b]
            if grads:
                G = (dy64[b, sl] @ v64[b].T) * W
                dq[b, sl] = G @ k64[b]
                dk[b] += G.T @ q64[b, sl]
                dv[b] += P.T @ dy64[b, sl]
    if kind == "infer":
        return y / y.norm(dim=-1, keepdim=True).clamp(min=1e-300)
    if kind == "expect" and not case["backward"]:
        return y
    if kind in ("star", "noalloc", "expect"):
        return dq, dk, dv
    if kind == "step":
        return qc, kc, y, dq, dk, dv
    return y, dq, dk, dv
