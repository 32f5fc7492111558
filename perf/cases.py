"""Work that a program has this library do, through its public entry points.

The listed cases cover the range of calls: fp32, fp16 and bf16; multi-head,
grouped-query and multi-query attention; a whole prompt, a chunk of a prompt
against a cache, and one new token against a contiguous or a paged cache; head
sizes 64 and 128 and others; and the Q8_0 matrix-vector products of a decode
step.  Head counts are those of the workloads in paper_2608_18656_amd.inputs
(32/4, 32/8, 16/2, 16/16 and 16/1 query / key-value heads).

A case is a dict with a "kind" and the sizes of that kind:
  attention  q [B, Nq, Hq, D] against k, v [B, Nk, Hkv, D]   (fwd)
  cache      the same with a valid length per sequence, the K/V cache either
             contiguous or in shuffled pages                  (fwd_kvcache, fwd_kvcache_paged)
  q8         Q8_0 products y = W x, one after the other       (q8_0_gemv)
"""
from __future__ import annotations

import math

import torch

import paper_2608_18656_amd as fa
from paper_2608_18656_amd.inputs import DTYPES

HEADS = ((32, 4), (32, 8), (16, 2), (16, 16), (16, 1))


def _attention(name, dtype, B, Hq, Hkv, Nq, Nk, D, causal):
    return {"name": name, "kind": "attention", "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "Nq": Nq, "Nk": Nk,
            "D": D, "causal": causal}


def _cache(name, dtype, B, Hq, Hkv, Nq, Nk, D, shortest, page):
    """Valid lengths run evenly from Nk down to ``shortest`` over the batch; page 0 is a contiguous cache."""
    return {"name": name, "kind": "cache", "dtype": dtype, "B": B, "Hq": Hq, "Hkv": Hkv, "Nq": Nq, "Nk": Nk, "D": D,
            "shortest": shortest, "page": page}


def _q8(name, dtype, matrices):
    """matrices: "MxK,MxK,..." in the order in which a layer applies them."""
    return {"name": name, "kind": "q8", "dtype": dtype, "matrices": matrices}


def listed():
    return [
        # the smallest call: a toy model, or a unit test of a user's program; latency decides
        _attention("mha_f32_128", "f32", 1, 2, 2, 128, 128, 64, False),
        # a prompt in full precision (reference runs, small models), a length that divides nothing
        _attention("mha_prefill_f32_777", "f32", 1, 16, 16, 777, 777, 64, True),
        # a few short prompts batched together
        _attention("gqa_prefill_bf16_333", "bf16", 4, 16, 2, 333, 333, 128, True),
        # an ordinary prompt of a small language model: the headline workload
        _attention("gqa_prefill_bf16_2048", "bf16", 1, 32, 8, 2048, 2048, 64, True),
        # long prompts of a larger model
        _attention("gqa_prefill_f16_4096", "f16", 2, 32, 8, 4096, 4096, 128, True),
        # a very long context on one key/value head: the largest call
        _attention("mqa_prefill_f16_16384", "f16", 1, 16, 1, 16384, 16384, 64, True),
        # a head size other than 64 and 128
        _attention("gqa_prefill_d96_bf16_1111", "bf16", 1, 16, 2, 1111, 1111, 96, True),
        # a serving step that continues prompts: 512 new tokens a sequence, caches of different lengths
        _cache("chunked_prefill_bf16", "bf16", 4, 32, 8, 512, 4096, 64, 1024, 0),
        # a serving step of a large batch with long caches: one token a sequence
        _attention("gqa_decode_bf16_8192", "bf16", 16, 32, 8, 1, 8192, 128, False),
        # one user's next token, a short context: latency decides
        _attention("gqa_decode_f16_1537", "f16", 1, 32, 4, 1, 1537, 64, False),
        # a serving step on a paged cache, every sequence at its own length
        _cache("paged_decode_bf16", "bf16", 12, 16, 2, 1, 6144, 128, 700, 256),
        # the linear layers of one decoder layer for one token (hidden size 2048, feed-forward size 5632)
        _q8("q8_layer_bf16", "bf16", "2560x2048,2048x2048,11264x2048,2048x5632"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(("prefill", "prefill", "prefill", "f32", "head", "chunk", "decode", "decode", "paged", "q8"))
    Hq, Hkv = rng.choice(HEADS)
    half = rng.choice(("f16", "bf16"))
    D = rng.choice((64, 128))
    if kind == "prefill":
        N, B = _log_int(rng, 64, 16384), rng.randint(1, 4)
        while B > 1 and B * N * N * Hq * D > 1.3e11:
            B -= 1
        N = min(N, int(math.sqrt(1.3e11 / (B * Hq * D))))
        c = _attention("", half, B, Hq, Hkv, N, N, D, rng.random() < 0.8)
    elif kind == "f32":
        N = _log_int(rng, 64, 1024)
        c = _attention("", "f32", 1, Hq, Hkv, N, N, rng.choice((64, 128)), rng.random() < 0.8)
    elif kind == "head":
        N = _log_int(rng, 64, 1536)
        c = _attention("", half, 1, 16, rng.choice((2, 16)), N if rng.random() < 0.8 else 1, N,
                       8 * rng.choice([i for i in range(4, 33) if i not in (8, 16)]), True)
    elif kind == "chunk":
        Nk = _log_int(rng, 512, 8192)
        Nq = _log_int(rng, 16, min(1024, Nk))
        c = _cache("", half, rng.randint(1, 6), Hq, Hkv, Nq, Nk, D, rng.randint(max(Nq, Nk // 8), Nk),
                   rng.choice((0, 64, 256)))
    elif kind == "decode":
        B, Nk = _log_int(rng, 1, 64), _log_int(rng, 128, 32768)
        B = max(1, min(B, int(5.3e8 / (4 * Nk * Hkv * D))))
        c = _attention("", half, B, Hq, Hkv, 1, Nk, D, False)
    elif kind == "paged":
        Nk = _log_int(rng, 512, 8192)
        c = _cache("", half, rng.randint(2, 16), Hq, Hkv, 1, Nk, D, rng.randint(Nk // 8, Nk), rng.choice((64, 256)))
    else:
        c = _q8("", rng.choice(("f16", "bf16", "f32")),
                "%dx%d" % (_log_int(rng, 512, 32768), 32 * _log_int(rng, 16, 512)))
    del c["name"]
    return c


def _lengths(case):
    B, Nk, lo = case["B"], case["Nk"], case["shortest"]
    return [Nk - (Nk - lo) * b // max(1, B - 1) for b in range(B)]


def _q8_shapes(case):
    return [tuple(int(n) for n in m.split("x")) for m in case["matrices"].split(",")]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt = DTYPES[case["dtype"]]

    def normal(*shape):
        return torch.randn(shape, generator=gen, dtype=torch.float32, device="cuda").to(dt)

    if case["kind"] == "q8":
        weights, xs = [], []
        for M, K in _q8_shapes(case):
            # the stored form, drawn directly: int8 values with one of +-127
            # in each block, binary16 scales (weights of deviation about 0.02)
            nb = K // 32
            q = torch.randn((M, nb, 32), generator=gen, device="cuda").mul_(40.0).round_().clamp_(-127.0, 127.0)
            at = torch.randint(0, 32, (M, nb, 1), generator=gen, device="cuda")
            sign = torch.randint(0, 2, (M, nb, 1), generator=gen, device="cuda").float().mul_(254.0).sub_(127.0)
            q.scatter_(2, at, sign)
            d = torch.randn((M, nb), generator=gen, device="cuda").abs_().mul_(2e-4).add_(1e-4)
            w = torch.empty((M, nb, 34), dtype=torch.uint8, device="cuda")
            w[:, :, :2] = d.half().view(torch.uint8).reshape(M, nb, 2)
            w[:, :, 2:] = q.to(torch.int8).view(torch.uint8)
            weights.append(w)
            xs.append(normal(K))
        return {"kind": "q8", "w": weights, "x": xs}
    B, Hq, Hkv, Nq, Nk, D = (case[k] for k in ("B", "Hq", "Hkv", "Nq", "Nk", "D"))
    s = {"kind": case["kind"], "q": normal(B, Nq, Hq, D), "k": normal(B, Nk, Hkv, D), "v": normal(B, Nk, Hkv, D)}
    if case["kind"] == "attention":
        s["causal"] = case["causal"]
        return s
    s["lengths"] = torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")
    s["page"] = case["page"]
    if case["page"]:
        # every sequence's pages scattered over the pool
        P = case["page"]
        n = -(-Nk // P)
        order = torch.randperm(B * n, generator=gen, device="cuda")
        for name in ("k", "v"):
            rows = torch.zeros((B, n * P, Hkv, D), dtype=dt, device="cuda")
            rows[:, :Nk] = s[name]
            pool = torch.empty((B * n, P, Hkv, D), dtype=dt, device="cuda")
            pool[order] = rows.view(B * n, P, Hkv, D)
            s[name] = pool
        s["table"] = order.to(torch.int32).view(B, n).contiguous()
    return s


def run(state):
    if state["kind"] == "q8":
        return [fa.q8_0_gemv(w, x) for w, x in zip(state["w"], state["x"])]
    if state["kind"] == "attention":
        return fa.fwd(state["q"], state["k"], state["v"], causal=state["causal"])
    if state["page"]:
        return fa.fwd_kvcache_paged(state["q"], state["k"], state["v"], state["table"], state["lengths"], causal=True)
    return fa.fwd_kvcache(state["q"], state["k"], state["v"], state["lengths"], causal=True)


def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "q8":
        shapes = _q8_shapes(case)
        return {"bytes": sum(M * (K // 32) * 34 + (M + K) * e for M, K in shapes),
                "flops": sum(2 * M * K for M, K in shapes)}
    B, Hq, Hkv, Nq, Nk, D = (case[k] for k in ("B", "Hq", "Hkv", "Nq", "Nk", "D"))
    lengths = _lengths(case) if case["kind"] == "cache" else [Nk] * B
    causal = case.get("causal", True)
    pairs = sum(Nq * n - (Nq * (Nq - 1) // 2 if causal else 0) for n in lengths)
    return {"bytes": 2 * B * Nq * Hq * D * e + 4 * B * Hq * Nq + 2 * sum(lengths) * Hkv * D * e,
            "flops": 4 * Hq * D * pairs}


def tolerance(case):
    # fp32 sums in another order; outputs rounded to the input type otherwise
    return {"rel": {"f32": 1e-5, "f16": 2e-3, "bf16": 1e-2}[case["dtype"]]}


def _exact_attention(q, k, v, causal):
    """One sequence in 64 bits: q [Nq, Hq, D], k and v [Nk, Hkv, D]."""
    Nq, Hq, D = q.shape
    Nk, Hkv, _ = k.shape
    o = torch.empty((Nq, Hq, D), dtype=torch.float64, device=q.device)
    lse = torch.empty((Hq, Nq), dtype=torch.float64, device=q.device)
    keys = torch.arange(Nk, device=q.device)
    for g in range(Hkv):
        kg, vg = k[:, g].double().t().contiguous(), v[:, g].double().contiguous()
        for h in range(g * (Hq // Hkv), (g + 1) * (Hq // Hkv)):
            for i0 in range(0, Nq, 2048):
                i1 = min(Nq, i0 + 2048)
                end = min(Nk, i1 + Nk - Nq) if causal else Nk
                s = (q[i0:i1, h].double() @ kg[:, :end].contiguous()).mul_(1.0 / math.sqrt(D))
                if causal:
                    rows = torch.arange(i0, i1, device=q.device)
                    s.masked_fill_(keys[None, :end] > (rows + Nk - Nq)[:, None], -math.inf)
                lse[h, i0:i1] = torch.logsumexp(s, 1)
                o[i0:i1, h] = s.sub_(lse[h, i0:i1, None]).exp_() @ vg[:end]
    return o, lse


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "q8":
        ys = []
        for w, x in zip(s["w"], s["x"]):
            M, nb, _ = w.shape
            d = w[:, :, :2].contiguous().view(torch.float16).double()
            ys.append((w[:, :, 2:].contiguous().view(torch.int8).double() * d).view(M, nb * 32) @ x.double())
        return ys
    B, Nk = case["B"], case["Nk"]
    if case["kind"] == "attention":
        per = [_exact_attention(s["q"][b], s["k"][b], s["v"][b], case["causal"]) for b in range(B)]
    else:
        per = []
        for b, n in enumerate(_lengths(case)):
            k, v = s["k"], s["v"]
            if case["page"]:
                pages = s["table"][b].long()
                k, v = (t[pages].reshape(-1, *t.shape[2:]) for t in (k, v))
            else:
                k, v = k[b], v[b]
            per.append(_exact_attention(s["q"][b], k[:n], v[:n], True))
    return tuple(torch.stack(t) for t in zip(*per))
