"""Timed cases of the library's entry points: decode steps, prompt ingestion, the prefill scorer, prompt attention.

`listed()` is the fixed list, `draw()` gives further cases of the same ranges, `prepare()` makes what a caller has in
hand before a call, `run()` is one pass through the public entry points (paper_2603_08727_amd.binding), `work()` says
what a pass cannot do without, `exact()` is the same result in 64 bits from plain torch, without the library.

Kinds:
  decode   one token through `layers` committed layers, one call per layer (a generated token of a served model);
           successive passes are successive tokens, so score updates and tailors come at their natural cadence
  ingest   a prompt of one layer: forget the previous request, score, commit, first decode step
  score    the prefill scorer of one layer alone (prompt attention computed elsewhere); `lse`: with that attention's
           log-sum-exp of the window rows
  attend   causal attention of the last `tq` positions of a prompt (tq = t: the whole prompt; less: one chunk of a
           chunked prefill); `stats`: with the scorer fused
"""
from __future__ import annotations

import math

import torch

from paper_2603_08727_amd import binding as A
from paper_2603_08727_amd import synth

STEPS = 32            # distinct tokens a decode state cycles through


def _case(name, kind, **kw):
    c = dict(kind=kind, layers=1, batch=1, hq=32, hkv=8, d=128, t=8192, n=2048, window=32, alpha=0.75, bits=4, rho=0.6,
             policy=0, bytes_mode=0, call="step", tq=0, stats=False, lse=False, temp=1.0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call there is: one layer of a small model, a cache of 128 tokens; launches and host work count,
        # and every 24th step tailors
        _case("decode_small", "decode", hq=8, hkv=2, d=64, t=512, n=128, rho=0.5),
        # one token of a single 8K-context request (8B-class model, grouped heads), through the entry point that
        # never allocates
        _case("decode_8k", "decode", layers=8, t=8192, n=2048, call="static"),
        # the headline shape: four 32K-context requests, a quarter of the cache kept, part of it as 4-bit rows; the
        # layers' pools exceed the last-level cache, as they do in a 36-layer model
        _case("decode_32k_b4", "decode", layers=4, batch=4, t=32768, n=8192),
        # one 128K-context request, an eighth of the cache kept, half of that as 2-bit rows
        _case("decode_128k_2bit", "decode", layers=8, t=131072, n=16384, bits=2, rho=0.5),
        # 64 query heads on 8 kv-heads, the fp8 rows and the byte budget, three requests of an odd length
        _case("decode_g8_fp8", "decode", layers=4, batch=3, hq=64, t=10007, n=2503, bits=8, rho=0.4, bytes_mode=1),
        # requests that still fit their cache: every row bf16, the longest streams
        _case("decode_full_cache", "decode", layers=2, batch=4, t=16384, n=20000),
        # the policy without slack: the cache stays full and every step ends with a tailor
        _case("decode_tailor_each", "decode", layers=4, batch=4, t=16384, n=8192, policy=1),
        # scorer stress: 512 query rows per kv-head against 16K keys
        _case("score_16k_w128", "score", batch=8, t=16384, n=4096, window=128),
        # a prompt of the headline shape on its way into the cache, up to the first generated token
        _case("ingest_32k_b4", "ingest", batch=4, t=32768, n=8192),
        # a whole 32K prompt's attention with the scorer fused
        _case("prefill_32k", "attend", t=32768, n=8192, tq=32768, stats=True),
        # a 512-token chunk of a chunked prefill late in a prompt whose length is no multiple of anything
        _case("prefill_chunk", "attend", t=16411, n=4096, tq=512),
        # a short prompt of a small model without grouped heads
        _case("prefill_mha_2k", "attend", batch=2, hq=16, hkv=16, d=64, t=2003, n=512, tq=2003),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes over the whole range (odd ones included), every head grouping, row format and option."""
    kind = rng.choice(["decode", "decode", "decode", "ingest", "score", "attend", "attend"])
    hkv = rng.choice([2, 4, 8])
    g = rng.choice([1, 2, 4, 4, 8])
    d = rng.choice([64, 128, 128])
    batch = rng.choice([1, 1, 2, 3, 4])
    window = rng.choice([16, 32, 32, 32, 48])
    t = _log_int(rng, 300, 32768)
    if kind in ("score", "attend"):
        t = _log_int(rng, 100, 11000)
    n = max(window + 16, int(t * rng.choice([0.125, 0.25, 0.25, 0.5])) + rng.randrange(7))
    if kind == "decode" and rng.random() < 0.2:
        n = t + 1200                                   # fits its cache
    policy = 1 if kind == "decode" and n < t and rng.random() < 0.15 else 0
    tq = 0
    if kind == "attend":
        tq = t if rng.random() < 0.5 else max(window, min(t, _log_int(rng, 32, 2048)))
    return _case(None, kind, layers=rng.choice([1, 2, 3]) if kind == "decode" else 1, batch=batch, hq=hkv * g, hkv=hkv, d=d,
                 t=t, n=n, window=window, bits=rng.choice([2, 4, 4, 8]), rho=round(rng.uniform(0.0, 1.0), 3), policy=policy,
                 bytes_mode=1 if rng.random() < 0.2 else 0, call=rng.choice(["step", "step", "static"]), tq=tq,
                 stats=kind == "attend" and rng.random() < 0.5, lse=kind == "score" and rng.random() < 0.3,
                 temp=rng.choice([0.5, 1.0, 2.0]))


# ---- inputs ------------------------------------------------------------------------------------------------------

def _workload(c, seed):
    return synth.Workload("case", c["layers"], c["batch"], c["hq"], c["hkv"], c["d"], c["t"], STEPS, 0.25, bits=c["bits"],
                          window=c["window"], alpha=c["alpha"], seed=(seed % 1000003) * 100003)


def _scale(c):
    return 1.0 / (math.sqrt(c["d"]) * c["temp"])


def _config(c):
    return A.arkv_config_default(n_layers=c["layers"], batch=c["batch"], n_q_heads=c["hq"], n_kv_heads=c["hkv"],
                                 head_dim=c["d"], capacity_tokens=c["n"], window=c["window"], alpha=c["alpha"],
                                 quant_bits=c["bits"], tailor_policy=c["policy"], budget_mode=c["bytes_mode"])


def _queries(c, seed):
    """bf16 queries of the last tq positions; the keys and values are synth's."""
    g = torch.Generator(device="cuda")
    g.manual_seed((seed % 1000003) * 100003 + 11)
    q = torch.randn((c["batch"], c["hq"], c["tq"], c["d"]), generator=g, device="cuda", dtype=torch.float32)
    return q.to(torch.bfloat16)


def _lse(qw, k, scale):
    """Natural log-sum-exp of the window rows' causal logits, fp32 [B][Hq][W], as an attention kernel returns it."""
    B, hq, W, d = qw.shape
    hkv, T = k.shape[1], k.shape[2]
    out = torch.empty((B, hq, W), device="cuda", dtype=torch.float32)
    see = torch.arange(T, device="cuda")[None, :] <= torch.arange(T - W, T, device="cuda")[:, None]
    for b in range(B):
        for h in range(hq):
            x = (qw[b, h].float() @ k[b, h // (hq // hkv)].float().t()) * scale
            out[b, h] = torch.logsumexp(x.masked_fill(~see, float("-inf")), dim=1)
    return out


class _Cache:
    """Owns a cache handle."""

    def __init__(self, c):
        self.handle = A.arkv_cache_create(_config(c))

    def __del__(self):
        if getattr(self, "handle", None) is not None:
            A.arkv_cache_destroy(self.handle)
            self.handle = None


def _rho(c):
    return [c["rho"]] * c["batch"]


def prepare(case, seed):
    c = case
    wl, scale = _workload(c, seed), _scale(c)
    cache = _Cache(c)
    s = dict(case=c, cache=cache, handle=cache.handle, scale=scale, at=0)
    stats = torch.zeros((c["batch"], 3), dtype=torch.float32, device="cuda")
    if c["kind"] == "decode":
        # every layer's prompt is scored and committed; the prompt's tensors are not needed any more after that
        for l in range(c["layers"]):
            k, v, qw = synth.prefill_inputs(wl, l, device="cuda")
            A.arkv_prefill_stats(cache.handle, l, qw, k, c["t"], scale, stats)
            A.arkv_prefill_commit(cache.handle, l, k, v, c["t"], _rho(c))
            del k, v, qw
        out = torch.zeros((c["layers"], c["batch"], c["hq"], c["d"]), dtype=torch.bfloat16, device="cuda")
        per_layer = [synth.decode_inputs(wl, l, STEPS, device="cuda") for l in range(c["layers"])]
        s["tokens"] = [[(l, q[i], kn[i], vn[i], out[l]) for l, (q, kn, vn) in enumerate(per_layer)] for i in range(STEPS)]
        s["out"] = out
        return s
    k, v, qw = synth.prefill_inputs(wl, 0, device="cuda")
    s.update(k=k, v=v, qw=qw, stats=stats)
    if c["kind"] == "score" and c["lse"]:
        s["lse"] = _lse(qw, k, scale)
    if c["kind"] == "attend":
        q = _queries(c, seed)
        s["q"], s["out"] = q, torch.zeros_like(q)
    if c["kind"] == "ingest":
        q, kn, vn = synth.decode_inputs(wl, 0, 1, device="cuda")
        s["token"] = (q[0], kn[0], vn[0])
        s["out"] = torch.zeros((c["batch"], c["hq"], c["d"]), dtype=torch.bfloat16, device="cuda")
    return s


def _named(stats):
    return {"entropy": stats[:, 0], "variance": stats[:, 1], "kurtosis": stats[:, 2]}


def run(state):
    s, c = state, state["case"]
    h, scale = s["handle"], s["scale"]
    if c["kind"] == "decode":
        step = A.arkv_decode_step_static if c["call"] == "static" else A.arkv_decode_step
        token = s["tokens"][s["at"]]
        s["at"] = (s["at"] + 1) % STEPS
        for l, q, kn, vn, out in token:
            step(h, l, q, kn, vn, scale, out)
        return s["out"]
    if c["kind"] == "score":
        if c["lse"]:
            A.arkv_prefill_stats_lse(h, 0, s["qw"], s["k"], c["t"], scale, s["lse"], s["stats"])
        else:
            A.arkv_prefill_stats(h, 0, s["qw"], s["k"], c["t"], scale, s["stats"])
        return _named(s["stats"])
    if c["kind"] == "ingest":
        A.arkv_cache_reset(h, 0)
        A.arkv_prefill_stats(h, 0, s["qw"], s["k"], c["t"], scale, s["stats"])
        A.arkv_prefill_commit(h, 0, s["k"], s["v"], c["t"], _rho(c))
        q, kn, vn = s["token"]
        step = A.arkv_decode_step_static if c["call"] == "static" else A.arkv_decode_step
        step(h, 0, q, kn, vn, scale, s["out"])
        return dict(_named(s["stats"]), out=s["out"])
    A.arkv_prefill_attention(h, 0, s["q"], s["k"], s["v"], c["tq"], c["t"], scale, s["out"], s["stats"] if c["stats"] else None)
    return dict(_named(s["stats"]), out=s["out"]) if c["stats"] else s["out"]


# ---- what a pass cannot do without -------------------------------------------------------------------------------

def _row_bytes(c):
    d, bits = c["d"], c["bits"]
    return 4 * d, (2 * (d + 2) if bits == 8 else 2 * (d * bits // 8 + 4 * (d // 32)))


def _kept(c):
    """(Original, Quantized) tokens per kv-head after the commit of the prompt."""
    n, w, t = c["n"], c["window"], c["t"]
    if t < n:
        return t, 0
    b = n - w - 1 if c["policy"] == 1 else min(int(math.floor(_f32(c["alpha"]) * (n - w))), n - w - 1)
    no = min(int(math.floor(_f32(c["rho"]) * (n - w))), b)
    nq = b - no
    if c["bytes_mode"] == 1:
        co, cq = _row_bytes(c)
        nq = nq * co // cq
    no = min(no, t - w)
    return w + no, min(nq, t - w - no)


def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def work(case):
    c = case
    units, g, d, t = c["batch"] * c["hkv"], c["hq"] // c["hkv"], c["d"], c["t"]
    co, cq = _row_bytes(c)
    o, q = _kept(c)
    token = 4 * g * d + co                                   # query in, output out, new key and value in
    if c["kind"] == "decode":
        # every live row, the new token and its append; a pass that ends with a tailor ranks on every token's two
        # running sums, which therefore are read and written
        per = o * co + q * cq + token + co + (16 * (o + q) if c["policy"] == 1 else 0)
        return {"bytes": c["layers"] * units * per, "flops": c["layers"] * units * 4.0 * g * d * (o + q + 1)}
    keys = units * t * 2 * d
    m = g * c["window"]
    score = {"bytes": keys + units * (2 * m * d + 8 * t), "flops": 2.0 * units * m * d * t}
    if c["kind"] == "score":
        return score
    if c["kind"] == "ingest":
        moved = units * (o * (2 * co) + q * (co + cq))       # kept rows in and out
        read = units * (o * co + q * cq + token + co)
        return {"bytes": score["bytes"] + moved + read, "flops": score["flops"] + units * 4.0 * g * d * (o + q + 1)}
    tq = c["tq"]
    seen = tq * (t - tq) + tq * (tq + 1) // 2
    w = {"bytes": 2 * keys + units * g * tq * 4 * d, "flops": 4.0 * c["batch"] * c["hq"] * d * seen}
    if c["stats"]:
        w = {"bytes": w["bytes"] + units * 8 * t, "flops": w["flops"] + score["flops"]}
    return w


def tolerance(case):
    """Outputs of attention are bf16: their distance to the 64-bit result is the rounding, 0.9e-3 to 1.7e-3 in the 2-norm
    over these ranges (packed rows' products are formed in 16-bit operands, which shows only below that); stated is
    four times the largest.  Statistics are single numbers computed from 32-bit probabilities: up to 6e-7 off, a few
    times more with a caller's 32-bit log-sum-exp."""
    if case["kind"] == "score":
        return {"rel": 5e-6, "max": 1e-5}
    return {"rel": 7e-3, "max": 3e-2}


# ---- the same in 64 bits -----------------------------------------------------------------------------------------

def _window_sums(qw, k, scale):
    """One sequence's window attention in fp64: per (kv-head, key) the sums of a and a^2 over (head, query), and the
    statistics of the aggregated distribution over the keys in front of the window."""
    hq, W, d = qw.shape
    hkv, T, _ = k.shape
    g = hq // hkv
    see = torch.arange(T, device=k.device)[None, :] <= torch.arange(T - W, T, device=k.device)[:, None]
    s1 = torch.zeros((hkv, T), dtype=torch.float64, device=k.device)
    s2 = torch.zeros_like(s1)
    for u in range(hkv):
        kk = k[u].double().t().contiguous()
        for h in range(g):
            x = (qw[u * g + h].double() @ kk) * scale
            a = torch.softmax(x.masked_fill(~see, float("-inf")), dim=1)
            s1[u] += a.sum(0)
            s2[u] += (a * a).sum(0)
    p = s1[:, : T - W].sum(0)
    p = p / p.sum()
    n = T - W
    ent = -(p[p > 0] * p[p > 0].log()).sum()
    dv = p - 1.0 / n
    var = (dv ** 2).mean()
    kurt = (dv ** 4).mean() / var ** 2 if float(var) > 0 else torch.zeros_like(var)
    return s1, s2, torch.stack([ent, var, kurt])


def _half_not_above(z):
    """fp16 of z, one step down where it rounded above."""
    h = z.to(torch.float16)
    return _step(h, h.float() > z, -1)


def _step(h, where, direction):
    """fp16 values moved one representable step down (-1) or up (+1) where asked."""
    bits = h.view(torch.int16).to(torch.int32) & 0xFFFF
    key = torch.where(bits >= 0x8000, 0x8000 - bits, bits)       # order-preserving integers, both zeros at 0
    key = key + direction
    back = torch.where(key < 0, 0x8000 - key, key).to(torch.int32)
    back = torch.where(back >= 0x8000, back - 0x10000, back).to(torch.int16).view(torch.float16)
    return torch.where(where, back, h)


def _packed_value(x, bits):
    """What a Quantized row [rows][d] stands for, in fp64 (the format's arithmetic is fp32 by definition)."""
    x = x.float()
    if bits == 8:
        amax = x.abs().amax(1, keepdim=True)
        s = (amax / 448.0).to(torch.float16)
        s = _step(s, s.float() * 448.0 < amax, +1)
        safe = torch.where(s.float() > 0, s.float(), torch.ones_like(amax))
        return (x / safe).to(torch.float8_e4m3fn).double() * s.double()
    r, d = x.shape
    grp = x.view(r, d // 32, 32)
    qmax = float((1 << bits) - 1)
    mn, mx = grp.amin(2, keepdim=True), grp.amax(2, keepdim=True)
    z = _half_not_above(mn)
    rng = mx - z.float()
    s = (rng / qmax).to(torch.float16)
    s = _step(s, s.float() * qmax < rng, +1)
    safe = torch.where(s.float() > 0, s.float(), torch.ones_like(rng))
    code = torch.round((grp - z.float()) / safe).clamp(0, qmax)
    code = torch.where(rng == 0, torch.zeros_like(code), code)
    return (code.double() * s.double() + z.double()).view(r, d)


def _first_step(c, k, v, s1, s2, q, kn, vn, scale):
    """The first decode step of one sequence in fp64: k, v [hkv][T][d], s1, s2 [hkv][T], q [hq][d], kn, vn [hkv][d]."""
    hkv, T, d = k.shape
    g, W = c["hq"] // hkv, c["window"]
    o, nq = _kept(c)
    out = torch.empty((c["hq"], d), dtype=torch.float64, device=k.device)
    for u in range(hkv):
        if T < c["n"]:
            kk, vv = k[u].double(), v[u].double()
        else:
            cnt = float(g * W)
            mu, ex2 = s1[u, : T - W] / cnt, s2[u, : T - W] / cnt
            S = mu + _f32(263.81) * (ex2 - mu * mu).clamp_min(0)
            rank = torch.sort(S, descending=True, stable=True).indices
            io, iq = rank[: o - W], rank[o - W: o - W + nq]
            kk = torch.cat([k[u, T - W:].double(), k[u, io].double(), _packed_value(k[u, iq], c["bits"])])
            vv = torch.cat([v[u, T - W:].double(), v[u, io].double(), _packed_value(v[u, iq], c["bits"])])
        kk = torch.cat([kk, kn[u].double()[None]])
        vv = torch.cat([vv, vn[u].double()[None]])
        p = torch.softmax((q[u * g:(u + 1) * g].double() @ kk.t().contiguous()) * scale, dim=1)
        out[u * g:(u + 1) * g] = p @ vv
    return out


def _causal(q, k, v, scale, T):
    """Causal attention of one head's last rows in fp64: q [tq][d], k, v [T][d]."""
    tq, d = q.shape
    kt, vv = k.double().t().contiguous(), v.double()
    out = torch.empty((tq, d), dtype=torch.float64, device=q.device)
    for r0 in range(0, tq, 1024):
        r1 = min(tq, r0 + 1024)
        last = T - tq + r1
        x = (q[r0:r1].double() @ kt[:, :last]) * scale
        pos = torch.arange(T - tq + r0, T - tq + r1, device=q.device)[:, None]
        x.masked_fill_(torch.arange(last, device=q.device)[None, :] > pos, float("-inf"))
        out[r0:r1] = torch.softmax(x, dim=1) @ vv[:last]
    return out


def exact(case, seed):
    c = case
    wl, scale = _workload(c, seed), _scale(c)
    if c["kind"] == "decode":
        out = torch.empty((c["layers"], c["batch"], c["hq"], c["d"]), dtype=torch.float64, device="cuda")
        for l in range(c["layers"]):
            k, v, qw = synth.prefill_inputs(wl, l, device="cuda")
            q, kn, vn = synth.decode_inputs(wl, l, STEPS, device="cuda")
            for b in range(c["batch"]):
                s1 = s2 = None
                if c["t"] >= c["n"]:
                    s1, s2, _ = _window_sums(qw[b], k[b], scale)
                out[l, b] = _first_step(c, k[b], v[b], s1, s2, q[0, b], kn[0, b], vn[0, b], scale)
        return out
    k, v, qw = synth.prefill_inputs(wl, 0, device="cuda")
    stats = torch.empty((c["batch"], 3), dtype=torch.float64, device="cuda")
    if c["kind"] == "attend":
        q = _queries(c, seed)
        g = c["hq"] // c["hkv"]
        out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        for b in range(c["batch"]):
            for h in range(c["hq"]):
                out[b, h] = _causal(q[b, h], k[b, h // g], v[b, h // g], scale, c["t"])
            if c["stats"]:
                stats[b] = _window_sums(q[b, :, c["tq"] - c["window"]:], k[b], scale)[2]
        return dict(_named(stats), out=out) if c["stats"] else out
    if c["kind"] == "score":
        for b in range(c["batch"]):
            stats[b] = _window_sums(qw[b], k[b], scale)[2]
        return _named(stats)
    q, kn, vn = synth.decode_inputs(wl, 0, 1, device="cuda")
    out = torch.empty((c["batch"], c["hq"], c["d"]), dtype=torch.float64, device="cuda")
    for b in range(c["batch"]):
        s1, s2, stats[b] = _window_sums(qw[b], k[b], scale)
        out[b] = _first_step(c, k[b], v[b], s1, s2, q[0, b], kn[0, b], vn[0, b], scale)
    return dict(_named(stats), out=out)
