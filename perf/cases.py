"""Performance cases of the Flash-ABFT attention forward: the calls that a
program makes, from one short encoder layer to a 32,768-token prefill, through
the package's public entry points.

A case has a kind:

* ``prefill``: one checked forward (``attn_fwd``, or ``attn_fwd_twopass``).
  ``check`` is ``sum`` (the output checksum, the default of the package),
  ``off``, ``weighted``, ``scores`` or ``twopass``;
* ``decode``: few query rows over a long cache (``attn_fwd_splitkv`` with its
  own choice of splits);
* ``guarded``: what a layer that recovers from faults runs: the checked
  forward, the recompute of flagged heads and the global check of the heads.

Inputs are the repository's stand-ins for a layer's Q, K and V: seeded N(0, 1)
in bfloat16, and in the ``peaked`` cases 1% of the keys of each head scaled by
8 (attention sinks: the running max then jumps late in a row).

The outputs are O, the row flags and the verdicts. The row residuals are not
among them: without a fault they are only the rounding of the sums (the exact
value of every one is 0), so there is nothing to compare; the flags state the
outcome of comparing them with the threshold.
"""
from __future__ import annotations

import math

import torch

import paper_2507_16676_amd as F

HEADS = (1, 2, 3, 5, 7, 8, 12, 16, 32)
DIMS = (64, 96, 128, 256)
# the largest listed case, in flops of the attention (see work)
MOST_FLOPS = 4.0 * 128 * 32 * (32768 * 32769 // 2)
MOST_BYTES = 4 << 30


def _case(name, kind, B, H, Lq, Lk, d, causal, check="sum", peaked=False):
    c = dict(kind=kind, B=B, H=H, Lq=Lq, Lk=Lk, d=d, causal=causal, check=check, peaked=peaked)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one encoder layer on one short text: 12 heads, launch and latency
        _case("enc_l128", "prefill", 1, 12, 128, 128, 64, False),
        # the same encoder on a batch of 512-token texts
        _case("enc_l512_b32", "prefill", 32, 12, 512, 512, 64, False),
        # a short decoder prompt: 32 heads of 96 over 256 tokens
        _case("dec_l256_d96", "prefill", 1, 32, 256, 256, 96, True),
        # the same decoder's ordinary prompt batch
        _case("dec_l2048_d96", "prefill", 2, 32, 2048, 2048, 96, True),
        # the benchmark workload: decoder prefill, 4 x 32 heads of 128
        _case("dec_l4096", "prefill", 4, 32, 4096, 4096, 128, True),
        # long-context prefill with peaked keys
        _case("long_l32768", "prefill", 1, 32, 32768, 32768, 128, True, peaked=True),
        # a decoder with 256-wide heads
        _case("dec_l4096_d256", "prefill", 1, 16, 4096, 4096, 256, True),
        # prefill with the score check, a ragged length
        _case("scores_l1999", "prefill", 2, 32, 1999, 1999, 128, True, check="scores"),
        # a protected layer: forward, recompute of flagged heads, global check
        _case("guarded_l2048", "guarded", 1, 32, 2048, 2048, 128, True),
        # decode: one new token per sequence over a long cache
        _case("decode_k32768", "decode", 4, 32, 1, 32768, 128, True),
        # decode of one sequence over an ordinary cache, odd length
        _case("decode_k4097", "decode", 1, 32, 1, 4097, 128, True),
        # the next 64 tokens of a prompt over a cache (chunked prefill)
        _case("chunk_q64_k8192", "decode", 8, 8, 64, 8192, 128, True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another call of the same kinds: lengths spread over the logarithm of
    their range and mostly odd, all head dimensions, checks and masks."""
    while True:
        kind = rng.choice(("prefill", "prefill", "prefill", "decode", "guarded"))
        B, H, d = _log_int(rng, 1, 32), rng.choice(HEADS), rng.choice(DIMS)
        causal = rng.random() < 0.6
        check = "sum"
        if kind == "decode":
            Lk = _log_int(rng, 512, 131072)
            Lq = rng.choice((1, 1, 2, 4, 5, 16, _log_int(rng, 6, 200)))
        else:
            Lk = _log_int(rng, 100, 16384)
            # a whole prompt, or one that continues a cache
            Lq = Lk if rng.random() < 0.7 else max(64, int(Lk * rng.uniform(0.1, 0.9)))
            Lq = min(Lq, Lk)
            if kind == "prefill":
                check = rng.choice(("sum", "sum", "off", "weighted", "scores", "twopass"))
                if d == 256 and check == "scores":
                    continue    # the score check is not built for d = 256
        c = _case("", kind, B, H, Lq, Lk, d, causal, check, rng.random() < 0.3)
        w = work(c)
        if w["flops"] <= MOST_FLOPS / 4 and w["bytes"] <= MOST_BYTES and w["bytes"] >= 1 << 18:
            return c


def prepare(case, seed):
    B, H, Lq, Lk, d = (case[k] for k in ("B", "H", "Lq", "Lk", "d"))
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    q, k, v = (torch.randn((B, H, L, d), generator=g, device="cuda", dtype=torch.bfloat16)
               for L in (Lq, Lk, Lk))
    if case["peaked"]:
        n = max(1, round(0.01 * Lk))
        rows = torch.rand((B, H, Lk), generator=g, device="cuda").topk(n, dim=-1).indices
        at = rows.unsqueeze(-1).expand(B, H, n, d)
        k.scatter_(2, at, k.gather(2, at) * 8)     # exact: a power of two
    s = {"case": case, "q": q, "k": k, "v": v}
    if case["check"] == "scores":
        # the score check's workspace, which a program keeps
        s["ws"] = torch.empty(F.score_check_workspace_bytes(B, H, Lk, d), dtype=torch.uint8,
                              device="cuda")
    return s


def run(state):
    case, q, k, v = state["case"], state["q"], state["k"], state["v"]
    kind, check, causal = case["kind"], case["check"], case["causal"]
    if kind == "decode":
        o, resid, flags = F.attn_fwd_splitkv(q, k, v, causal=causal)
        return {"o": o, "flags": flags}
    if kind == "guarded":
        o, resid, flags = F.attn_fwd(q, k, v, causal=causal)
        recovered, persistent = F.recompute_flagged(q, k, v, o, resid, flags, causal=causal)
        gsum, gflags = F.global_check(o, resid)
        return {"o": o, "flags": flags, "gflags": gflags, "recovered": recovered,
                "persistent": persistent}
    if check == "off":
        return {"o": F.attn_fwd(q, k, v, causal=causal, check=False)}
    if check == "twopass":
        o, resid, flags = F.attn_fwd_twopass(q, k, v, causal=causal)
    elif check == "weighted":
        F.set_weighted_check(True)
        try:
            o, resid, flags = F.attn_fwd(q, k, v, causal=causal)
        finally:
            F.set_weighted_check(False)
    elif check == "scores":
        F.set_score_check(state["ws"])
        try:
            o, resid, flags = F.attn_fwd(q, k, v, causal=causal)
        finally:
            F.set_score_check(None)
    else:
        o, resid, flags = F.attn_fwd(q, k, v, causal=causal)
    return {"o": o, "flags": flags}


def _visible_pairs(Lq, Lk, causal):
    """Pairs of one head; causal: key k of query i iff k <= i + Lk - Lq
    (every drawn and listed case has Lq <= Lk)."""
    if not causal or Lq > Lk:
        return Lq * Lk
    return Lq * (Lk - Lq) + Lq * (Lq + 1) // 2


def work(case):
    B, H, Lq, Lk, d = (case[k] for k in ("B", "H", "Lq", "Lk", "d"))
    rows = B * H * Lq
    n = 2 * d * (2 * rows + 2 * B * H * Lk)      # q, o, k, v once, 2 bytes each
    if case["check"] != "off":
        n += 5 * rows                            # resid, flags
    if case["kind"] == "guarded":
        n += 9 * B * H                           # the global sums and flags
    return {"bytes": float(n), "flops": 4.0 * d * B * H * _visible_pairs(Lq, Lk, case["causal"])}


def tolerance(case):
    """O is rounded to bfloat16 (1.6e-3 in norm, 3.9e-3 at most per value) from
    products whose weights are bfloat16 too: against 64 bits the norm of the
    error is 2.0e-3 to 2.3e-3 and the largest 4.3e-2 (of the larger of the root
    mean square and the value), most of it where a row sees few keys. Decode of
    up to four rows keeps its weights in 32 bits: 1.7e-3 and 3.9e-3. Four times
    that. The flags and verdicts are whole values and agree."""
    if case["kind"] == "decode" and case["Lq"] <= 4:
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 1e-2, "max": 0.17}


def exact(case, seed):
    """O in 64 bits, a block of rows of one head at a time."""
    B, H, Lq, Lk, d = (case[k] for k in ("B", "H", "Lq", "Lk", "d"))
    s = prepare(case, seed)
    out = torch.empty((B, H, Lq, d), dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // Lk)
    keys = torch.arange(Lk, device="cuda")
    for b in range(B):
        for h in range(H):
            k, v = s["k"][b, h].double(), s["v"][b, h].double()
            kt = k.t().contiguous()
            for r in range(0, Lq, step):
                e = min(Lq, r + step)
                x = (s["q"][b, h, r:e].double() @ kt) * (1.0 / math.sqrt(d))
                if case["causal"]:
                    rows = torch.arange(r, e, device="cuda").unsqueeze(1) + (Lk - Lq)
                    x = x.masked_fill(keys > rows, -math.inf)
                out[b, h, r:e] = torch.softmax(x, dim=-1) @ v
    return {"o": out, "flags": None, "gflags": None, "recovered": None, "persistent": None}
