"""The work users have this framework do, as cases that can be timed and checked.

A case is a dict of plain values; its "kind" says which public calls it makes:

  prefill     eva.prefill: chunk summaries and the fused window + summary
              attention of whole prompts.  With "cache" the prompt also fills a
              decode cache and the first generated token runs through
              eva.append_decode, as a server does.  With "rf" the summaries are
              the stochastic ones (eva.build_summaries_rf, then
              eva.prefill_attention)
  train       eva.prefill_forward keeping the output's rounding residual, then
              eva.prefill_backward: one attention layer of a training step
  decode      eva.append_decode: one token for every sequence of a batch
  generate    eva.generate on a ragged cache: "steps" tokens for every sequence

All inputs are i.i.d. N(0, 1) (queries and keys of unit root mean square, as
after a normalisation), as in the package's own seeded workloads.
"""
import math

import numpy as np
import torch

from paper_2511_00576_amd import _lib, eva

WINDOWS = {"sliding": _lib.EVA_WINDOW_SLIDING, "chunk_aligned": _lib.EVA_WINDOW_CHUNK_ALIGNED,
           "blocked": _lib.EVA_WINDOW_BLOCKED, "noncausal": _lib.EVA_WINDOW_NONCAUSAL}
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
RF_LAMBDA = 0.1


def _case(name, kind, B, H, Hkv, L, d, W, C, dtype="bf16", window="sliding", **more):
    return dict(name=name, kind=kind, B=B, H=H, Hkv=Hkv, L=L, d=d, W=W, C=C, dtype=dtype, window=window, **more)


def listed():
    return [
        # a single user's prompt of odd length that ends in a cache, and its
        # first token: launches and latency count
        _case("prefill_chat", "prefill", 1, 32, 8, 777, 128, 256, 64, cache=True),
        # a batch of 4k prompts of a multi-head model, served: the framework's
        # headline workload (prefill into the cache, first token)
        _case("prefill_llm", "prefill", 8, 32, 32, 4096, 128, 256, 64, cache=True),
        # grouped-query model, 8k prompts
        _case("prefill_gqa", "prefill", 4, 32, 8, 8192, 128, 512, 128, cache=False),
        # one document of 32k tokens
        _case("prefill_long", "prefill", 1, 32, 8, 32768, 128, 1024, 256, cache=False),
        # a small-head model with everything off the round numbers: three query
        # heads per kv head, 24-token chunks, the chunk-aligned window and the
        # stochastic summaries
        _case("prefill_odd_rf", "prefill", 3, 12, 4, 2999, 64, 200, 24, window="chunk_aligned", rf=True),
        # fp32 evaluation of a mid-sized batch
        _case("prefill_f32", "prefill", 2, 16, 4, 2048, 128, 256, 64, dtype="f32", cache=False),
        # training steps: the headline shape, a grouped-query model at 8k, and
        # a small non-causal encoder at an odd length
        _case("train_llm", "train", 8, 32, 32, 4096, 128, 256, 64),
        _case("train_gqa", "train", 4, 32, 8, 8192, 128, 512, 128),
        _case("train_encoder", "train", 4, 12, 12, 1500, 64, 128, 32, window="noncausal"),
        # decode: one user (latency), and a full serving batch at 8k context
        _case("decode_single", "decode", 1, 32, 8, 8000, 128, 512, 128),
        _case("decode_batch", "decode", 64, 32, 8, 8192, 128, 512, 128),
        # batched generation after prompts of different lengths (up to L): 16
        # tokens for each of 32 sequences; every chunk completes once meanwhile
        _case("generate_ragged", "generate", 32, 32, 8, 3072, 128, 256, 16, steps=16),
    ]


# ---- sizes ----------------------------------------------------------------
def _bounds(n, L, W, C, window):
    """First and last exact key of rows n, and the counts of summaries before and from where they lie after."""
    if window == "sliding":
        lo = np.maximum(0, n - W + 1)
    elif window == "chunk_aligned":
        lo = np.maximum(0, n - W + 1) // C * C
    else:
        lo = n // W * W
    hi = np.minimum(L, lo + W) - 1 if window == "noncausal" else n
    after = np.minimum(hi // C + 1, L // C) if window == "noncausal" else np.full_like(n, L // C)
    return lo, hi, lo // C, after


def _pairs(c):
    """(row, key or summary) pairs of one head of one sequence's prefill."""
    lo, hi, s, after = _bounds(np.arange(c["L"], dtype=np.int64), c["L"], c["W"], c["C"], c["window"])
    return int((hi - lo + 1 + s + (c["L"] // c["C"] - after)).sum())


def _lens(c):
    """Prompt lengths of a generation case: spread over the upper two thirds of [1, L], the longest first."""
    B, L = c["B"], c["L"]
    return [max(1, L - (2 * L // 3) * i // max(1, B - 1) - (i * 7) % 13 * (i > 0)) for i in range(B)]


def work(c):
    e = 4 if c["dtype"] == "f32" else 2
    B, H, Hkv, L, d, W, C = (c[k] for k in ("B", "H", "Hkv", "L", "d", "W", "C"))
    if c["kind"] in ("prefill", "train"):
        pairs = B * H * _pairs(c)
        q, k, s = B * H * L * d * e, B * Hkv * L * d * e, B * Hkv * (L // C) * d * e
        if c["kind"] == "train":
            # read Q, K, V, dO; write O, lse, dQ, dK, dV; five products in the
            # backward (scores once more, dP, dQ, dK, dV) beside the forward's two
            return {"bytes": 4 * q + 4 * k + B * H * L * 4, "flops": pairs * d * (4 + 10)}
        n = 2 * q + 2 * k + 2 * s
        if c.get("cache"):
            n += 2 * B * Hkv * (min(W + C, L) + L // C) * d * e
        if c.get("rf"):
            n += B * Hkv * (L // C) * d * 4
        return {"bytes": n, "flops": pairs * d * 4}

    def row(p):  # keys and summaries of the row at position p
        lo, hi, s, _ = _bounds(np.asarray([p]), p + 1, W, C, c["window"])
        return int(hi[0] - lo[0] + 1 + s[0])

    if c["kind"] == "decode":
        rows, toks = B * row(L), B
    else:
        rows, toks = sum(row(n + t) for n in _lens(c) for t in range(c["steps"])), B * c["steps"]
    return {"bytes": (rows * Hkv * d * 2 + toks * (2 * H + 2 * Hkv) * d) * e, "flops": rows * H * d * 4}


def _cost(c):
    w = work(c)
    return w["bytes"] / 5e12 + w["flops"] / (5e13 if c["dtype"] == "f32" else 5e14)


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["prefill", "prefill", "train", "train", "decode", "generate"])
        Hkv = rng.choice([1, 2, 4, 8, 8, 12, 16, 32])
        H = Hkv * rng.choice([1, 1, 2, 3, 4, 4, 8])
        d = rng.choice([64, 128, 128])
        W = rng.choice([128, 256, 512, 1024, log(32, 1024)])
        C = rng.choice([16, 32, 64, 128, 256, log(8, 256)])
        c = dict(kind=kind, H=H, Hkv=Hkv, d=d, W=W, C=C)
        if H > 64:
            continue
        if kind == "prefill":
            c.update(B=log(1, 8), L=log(200, 32768), dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                     window=rng.choice(["sliding", "sliding", "sliding", "chunk_aligned", "blocked", "noncausal"]))
            c["rf"] = rng.random() < 0.2
            c["cache"] = not c["rf"] and c["window"] != "noncausal" and rng.random() < 0.4
        elif kind == "train":
            c.update(B=log(1, 8), L=log(200, 16384), dtype="bf16",
                     window=rng.choice(["sliding", "sliding", "sliding", "chunk_aligned", "blocked", "noncausal"]))
        elif kind == "decode":
            c.update(B=log(1, 64), L=log(200, 16384), dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                     window=rng.choice(["sliding", "sliding", "chunk_aligned", "blocked"]))
        else:
            c.update(B=log(2, 48), L=log(200, 4096), dtype="bf16", window=rng.choice(["sliding", "chunk_aligned"]),
                     steps=rng.choice([4, 8, 16]))
        # no more than the largest listed case, in time and in memory
        history = c["B"] * c["Hkv"] * c["L"] * d * (2 if c["dtype"] == "bf16" else 4)
        if _cost(c) <= most and history <= 2 ** 30 and c["B"] * H * c["L"] * d <= 2 ** 28:
            return c


# ---- inputs ---------------------------------------------------------------
def _inputs(c, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = DTYPES[c["dtype"]]

    def normal(*shape, dtype=dt):
        return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)

    B, H, Hkv, L, d, C = (c[k] for k in ("B", "H", "Hkv", "L", "d", "C"))
    x = {"K": normal(B, Hkv, L, d), "V": normal(B, Hkv, L, d)}
    if c["kind"] in ("prefill", "train"):
        x["Q"] = normal(B, H, L, d)
    if c["kind"] == "train":
        x["dO"] = normal(B, H, L, d)
    if c.get("rf"):
        x["eps"] = normal(B, Hkv, L // C, d, dtype=torch.float32)
    steps = c["steps"] if c["kind"] == "generate" else 1 if c["kind"] == "decode" or c.get("cache") else 0
    if steps:
        x["q"], x["k"], x["v"] = normal(steps, B, H, d), normal(steps, B, Hkv, d), normal(steps, B, Hkv, d)
    return x


def prepare(c, seed):
    x = _inputs(c, seed)
    s = {"case": c, "window": WINDOWS[c["window"]], **x}
    if c["kind"] in ("decode", "generate") or c.get("cache"):
        ragged = c["kind"] == "generate"
        make = eva.RaggedCache if ragged else eva.Cache
        s["cache"] = make(c["B"], c["H"], c["Hkv"], c["d"], c["W"], c["C"],
                          max_tokens=c["L"] + c.get("steps", 1) + 64, dtype=DTYPES[c["dtype"]], fill=0.0,
                          window=s["window"])
        if c["kind"] != "prefill":
            # the prompt's history, in the cache before the first token
            Ks, Vs = eva.build_summaries(x["K"], x["V"], c["C"])
            if ragged:
                s["lens"] = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
                eva.rcache_fill(s["cache"], x["K"], x["V"], Ks, Vs, s["lens"])
            else:
                eva.cache_fill(s["cache"], x["K"], x["V"], Ks, Vs)
            del s["K"], s["V"]
    return s


# ---- one pass -------------------------------------------------------------
def _arrays(cache):
    return [cache.k_ring, cache.vt_ring, cache.k_sum, cache.vt_sum]


def run(s):
    c = s["case"]
    W, C = c["W"], c["C"]
    if c["kind"] == "prefill":
        if c.get("rf"):
            Ks, Vs = eva.build_summaries_rf(s["K"], s["V"], s["eps"], C, RF_LAMBDA)
            return [eva.prefill_attention(s["Q"], s["K"], s["V"], Ks, Vs, W, C, window=s["window"]), Ks, Vs]
        if not c.get("cache"):
            return list(eva.prefill(s["Q"], s["K"], s["V"], W, C, return_summaries=True, window=s["window"]))
        out = eva.prefill(s["Q"], s["K"], s["V"], W, C, cache=s["cache"], return_summaries=True, window=s["window"])
        o = eva.append_decode(s["cache"], s["q"][0], s["k"][0], s["v"][0])
        return [*out, o, *_arrays(s["cache"])]
    if c["kind"] == "train":
        # the residual O_lo is the forward's message to the backward (what O's
        # rounding lost); a training step keeps O, lse and the gradients
        O, lse, Ks, Vs, O_lo = eva.prefill_forward(s["Q"], s["K"], s["V"], W, C, residual=True, window=s["window"])
        dQ, dK, dV = eva.prefill_backward(s["Q"], s["K"], s["V"], Ks, Vs, O, lse, s["dO"], W, C, O_lo=O_lo,
                                          window=s["window"])
        return [O, lse, dQ, dK, dV]
    if c["kind"] == "decode":
        # the token is rolled back before each pass (as a speculative decoder
        # rolls back a rejected one), so that every pass serves the same position
        s["cache"].struct.n_tok = c["L"]
        return [eva.append_decode(s["cache"], s["q"][0], s["k"][0], s["v"][0]), *_arrays(s["cache"])]
    s["cache"].n_tok.copy_(s["lens"])
    return [eva.generate(s["cache"], s["q"], s["k"], s["v"]), s["cache"].n_tok, *_arrays(s["cache"])]


def tolerance(c):
    # About four times the largest relative error of any output against 64 bits
    # over these cases and draws: 4.5e-7 for fp32 (fp32 sums and exponentials),
    # 2.6e-3 for bf16 outputs, softmax weights, score gradients and gradients
    return {"rel": 2e-6} if c["dtype"] == "f32" else {"rel": 1e-2}


# ---- the same in 64 bits --------------------------------------------------
def _summaries64(K, V, C, eps=None):
    """[..., L, d] -> the complete chunks' summary keys and values [..., L // C, d]."""
    d = K.shape[-1]
    n = K.shape[-2] // C
    k = K[..., :n * C, :].reshape(*K.shape[:-2], n, C, d)
    v = V[..., :n * C, :].reshape(*V.shape[:-2], n, C, d)
    kh = k.mean(-2)
    if eps is None:
        a = (k * kh.unsqueeze(-2)).sum(-1) / math.sqrt(d)
    else:
        # omega . x - |x|^2 / 2 with x = k / d^(1/4), omega = mean(x) + lambda clip(eps)
        x = k / d ** 0.25
        om = kh / d ** 0.25 + RF_LAMBDA * eps.clamp(-1, 1)
        a = (x * om.unsqueeze(-2)).sum(-1) - 0.5 * (x * x).sum(-1)
    return kh, (torch.softmax(a, -1).unsqueeze(-1) * v).sum(-2)


def _attend64(c, Q, K, V, Ks, Vs, rows=256):
    """One sequence: Q [H, L, d], K, V [Hkv, L, d], summaries [Hkv, n, d] -> O [H, L, d], lse [H, L]."""
    H, L, d = Q.shape
    Hkv, W, C, window = K.shape[0], c["W"], c["C"], c["window"]
    G = H // Hkv
    n_chunks = Ks.shape[1]
    Q = Q.reshape(Hkv, G, L, d)
    outs, lses = [], []
    for r0 in range(0, L, rows):
        n = np.arange(r0, min(L, r0 + rows), dtype=np.int64)
        lo, hi, s, after = _bounds(n, L, W, C, window)
        k0, k1, s1 = int(lo.min()), int(hi.max()) + 1, int(s.max())
        if window == "noncausal":
            s1 = n_chunks
        dev = [torch.from_numpy(x).to(Q.device).unsqueeze(1) for x in (lo, hi, s, after)]
        keys = torch.arange(k0, k1, device=Q.device)
        sums = torch.arange(s1, device=Q.device)
        ok = torch.cat([(keys >= dev[0]) & (keys <= dev[1]), (sums < dev[2]) | (sums >= dev[3])], 1)
        kk = torch.cat([K[:, k0:k1], Ks[:, :s1]], 1)
        vv = torch.cat([V[:, k0:k1], Vs[:, :s1]], 1)
        bias = torch.zeros(k1 - k0 + s1, dtype=Q.dtype, device=Q.device)
        bias[k1 - k0:] = math.log(C)
        q = Q[:, :, r0:r0 + len(n)].reshape(Hkv, G * len(n), d)
        x = torch.matmul(q, kk.transpose(1, 2).contiguous()).reshape(Hkv, G, len(n), -1) / math.sqrt(d) + bias
        x = x.masked_fill(~ok, -math.inf)
        lse = torch.logsumexp(x, -1)
        p = torch.exp(x - lse.unsqueeze(-1)).reshape(Hkv, G * len(n), -1)
        outs.append(torch.matmul(p, vv).reshape(Hkv, G, len(n), d))
        lses.append(lse)
    return torch.cat(outs, 2).reshape(H, L, d), torch.cat(lses, 2).reshape(H, L)


def _row64(c, q, K, V, Ks, Vs, p):
    """The row at position p of one sequence: q [H, d] -> [H, d]."""
    H, d = q.shape
    Hkv = K.shape[0]
    lo, _, s, _ = _bounds(np.asarray([p]), p + 1, c["W"], c["C"], c["window"])
    lo, s = int(lo[0]), int(s[0])
    kk = torch.cat([K[:, lo:p + 1], Ks[:, :s]], 1)
    vv = torch.cat([V[:, lo:p + 1], Vs[:, :s]], 1)
    x = torch.matmul(q.reshape(Hkv, H // Hkv, d), kk.transpose(1, 2).contiguous()) / math.sqrt(d)
    x[..., p + 1 - lo:] += math.log(c["C"])
    return torch.matmul(torch.softmax(x, -1), vv).reshape(H, d)


def _arrays64(c, cap, R, K, V, Ks, Vs, kept):
    """The cache arrays of one sequence: ring of the `kept` last tokens, all summaries."""
    Hkv, n, d = K.shape
    kr, vr = K.new_zeros(Hkv, R, d), K.new_zeros(Hkv, R, d)
    pos = torch.arange(max(0, n - kept), n, device=K.device)
    kr[:, pos % R], vr[:, pos % R] = K[:, pos], V[:, pos]
    ks, vs = K.new_zeros(Hkv, cap, d), K.new_zeros(Hkv, cap, d)
    ks[:, :Ks.shape[1]], vs[:, :Vs.shape[1]] = Ks, Vs

    def tiled(v):
        return v.reshape(Hkv, -1, 8, d).transpose(-1, -2).contiguous()

    return kr, tiled(vr), ks, tiled(vs)


def _capacity(c):
    C = c["C"]
    tokens = c["L"] + c.get("steps", 1) + 64
    return max(32, -(-(tokens // C + 1) // 32) * 32), -(-(c["W"] + C - 1) // 32) * 32


def exact(c, seed):
    x = {k: v.double() for k, v in _inputs(c, seed).items()} if c["kind"] != "train" else _inputs(c, seed)
    B, C = c["B"], c["C"]
    out = []
    for b in range(B):
        if c["kind"] == "train":
            Q, K, V = (x[k][b].double().requires_grad_() for k in ("Q", "K", "V"))
            O, lse = _attend64(c, Q, K, V, *_summaries64(K, V, C))
            O.backward(x["dO"][b].double())
            out.append([t.detach().cpu() for t in (O, lse, Q.grad, K.grad, V.grad)])
            continue
        K, V = x["K"][b], x["V"][b]
        if c["kind"] == "prefill":
            Ks, Vs = _summaries64(K, V, C, x["eps"][b] if c.get("rf") else None)
            got = [_attend64(c, x["Q"][b], K, V, Ks, Vs)[0], Ks, Vs]
            if not c.get("cache"):
                out.append([t.cpu() for t in got])
                continue
        else:
            got = []
        cap, R = _capacity(c)
        if c["kind"] == "generate":
            n = _lens(c)[b]
            K, V = K[:, :n], V[:, :n]
        first = K.shape[1]
        steps = x["q"].shape[0]
        K = torch.cat([K, x["k"][:, b].transpose(0, 1)], 1)
        V = torch.cat([V, x["v"][:, b].transpose(0, 1)], 1)
        Ks, Vs = _summaries64(K, V, C)
        o = [_row64(c, x["q"][t, b], K[:, :first + t + 1], V[:, :first + t + 1], Ks, Vs, first + t)
             for t in range(steps)]
        arrays = _arrays64(c, cap, R, K, V, Ks, Vs, min(R, K.shape[1]))
        if c["kind"] == "generate":
            got += [torch.stack(o), torch.tensor(float(first + steps), dtype=torch.float64), *arrays]
        else:
            got += [o[0], *arrays]
        out.append([t.cpu() for t in got])
    res = [torch.stack([o[i] for o in out], 1 if c["kind"] == "generate" and i == 0 else 0) for i in range(len(out[0]))]
    if c["kind"] == "generate":
        res[1] = None  # token counts: whole numbers
    return res
