"""The workloads whose speed is watched.

Each case is one call of the library as a serving program makes it: rank the
candidates of one or more users against their cached histories, or encode
histories into the cache.  What such a program keeps from request to request
(the model, the action heads, the workspace) is made in ``prepare``, like the
request's own tokens, offsets and cache; ``run`` is the call.

The cache of a ranking case is drawn directly instead of encoded: ranking
reads a cache that another stage filled, and keys and values of a normalised
row under Xavier weights have unit variance at every layer, so N(0, 1) values
are what the call meets.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2606_00422_amd import upr

# Action set of the heads cases: two rewarded actions and a penalised one.
UTILITY = (1.0, 0.5, -2.0)

_MAX_FLOPS = 4.3e12         # the largest listed case's
_MAX_ROWS = 131072


def _case(kind, dtype, U, n, k, d, H, L, F, lens_seed=0, **more):
    """n and k: (lowest, highest) history rows and candidates of a user."""
    return dict(kind=kind, dtype=dtype, users=U, n_lo=n[0], n_hi=n[1], k_lo=k[0], k_hi=k[1],
                d=d, heads=H, layers=L, d_ff=F, lens_seed=lens_seed, **more)


def listed():
    def named(name, *a, **kw):
        return dict(name=name, **_case(*a, **kw))
    return [
        # the smallest model and call: launches and latency
        named("rank_tiny_f32", "rank", "f32", 1, (64, 64), (128, 128), 64, 2, 1, 256),
        # fp32 model, a small batch of uneven users (a service that checks
        # the bf16 model's scores, or serves without reduced precision)
        named("rank_f32_u4", "rank", "f32", 4, (150, 450), (300, 700), 256, 4, 2, 1024, lens_seed=1),
        # one user's request, the latency of online ranking
        named("rank_user", "rank", "bf16", 1, (1024, 1024), (2000, 2000), 512, 8, 4, 2048),
        # the headline batch
        named("rank_u64", "rank", "bf16", 64, (1024, 1024), (2000, 2000), 512, 8, 4, 2048),
        # the same batch size with uneven users, as real traffic is
        named("rank_ragged_u64", "rank", "bf16", 64, (32, 2048), (200, 3000), 512, 8, 4, 2048, lens_seed=2),
        # lifelong histories: attention over 8192 rows
        named("rank_u8_n8192", "rank", "bf16", 8, (8192, 8192), (4096, 4096), 512, 8, 4, 2048),
        # a wide model, rows past the fused LayerNorm's 512, uneven users
        named("rank_wide", "rank", "bf16", 12, (100, 900), (300, 1700), 768, 12, 2, 3072, lens_seed=3),
        # heads of 32 values, uneven users
        named("rank_head32", "rank", "bf16", 16, (32, 512), (200, 1500), 256, 8, 2, 1024, lens_seed=4),
        # fp8 projections on the headline batch
        named("rank_mxfp8_u64", "rank", "bf16_mxfp8", 64, (1024, 1024), (2000, 2000), 512, 8, 4, 2048),
        # per-action probabilities and utility of a medium batch
        named("actions_u16", "actions", "bf16", 16, (256, 256), (1000, 1000), 256, 4, 2, 1024,
              actions=3, hidden=128),
        # one user's history encoded when the user arrives: latency
        named("encode_user", "encode", "bf16", 1, (1000, 1000), (0, 0), 512, 8, 4, 2048),
        # the headline batch's histories
        named("encode_u64", "encode", "bf16", 64, (1024, 1024), (0, 0), 512, 8, 4, 2048),
    ]


def draw(rng: random.Random):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def span(lo, hi):
        """A range of lengths: one length, or from about a tenth of it up."""
        top = log_int(lo, hi)
        return (top, top) if rng.random() < 0.4 else (max(1, top // rng.choice((2, 4, 10))), top)

    while True:
        what = rng.choices(("rank", "encode", "mxfp8", "actions", "f32", "head32"),
                           (40, 20, 10, 10, 10, 10))[0]
        head = 32 if what == "head32" or (what == "f32" and rng.random() < 0.5) else 64
        d = {"f32": rng.choice((64, 128, 256, 512)),
             "mxfp8": rng.choice((256, 512, 768)),
             "head32": rng.choice((128, 256, 512))}.get(what, rng.choice((128, 256, 384, 512, 512, 768, 1024)))
        F = d * rng.choice((2, 4, 4))
        more = dict(actions=rng.choice((2, 3, 5)), hidden=d // 2) if what == "actions" else {}
        case = _case("actions" if what == "actions" else "encode" if what == "encode" else "rank",
                     {"f32": "f32", "mxfp8": "bf16_mxfp8"}.get(what, "bf16"), log_int(1, 64),
                     span(16, 8192), (0, 0) if what == "encode" else span(32, 4096), d, d // head,
                     rng.randint(1, 4), F, lens_seed=rng.randrange(1 << 20), **more)
        nl, kl = _lens(case)
        rows = sum(nl) if what == "encode" else sum(kl)
        # fp32 models and small heads stay at the sizes of their listed cases
        most = {"f32": 1.5e10, "head32": 1e11}.get(what, _MAX_FLOPS)
        if rows <= _MAX_ROWS and sum(nl) <= _MAX_ROWS and work(case)["flops"] <= most:
            return case


# ---------------------------------------------------------------------------
# Sizes
# ---------------------------------------------------------------------------

def _lens(case):
    r = random.Random(case["lens_seed"])
    n = [r.randint(case["n_lo"], case["n_hi"]) for _ in range(case["users"])]
    k = [r.randint(case["k_lo"], case["k_hi"]) for _ in range(case["users"])]
    return n, k


def work(case):
    n, k = _lens(case)
    d, L, F = case["d"], case["layers"], case["d_ff"]
    size = 4 if case["dtype"] == "f32" else 2
    wsize = 1 if case["dtype"] == "bf16_mxfp8" else size
    kv = 2.0 * L * sum(n) * d * size
    if case["kind"] == "encode":
        T = sum(n)
        pairs = sum(x * (x + 1) // 2 for x in n)
        flops = L * 6.0 * d * d * T + (L - 1) * ((2.0 * d * d + 4.0 * d * F) * T + 4.0 * d * pairs)
        weights = wsize * (L * 3.0 * d * d + (L - 1) * (d * d + 2.0 * d * F))
        return {"bytes": T * d * size + weights + kv, "flops": flops}
    R = sum(k)
    seen = sum(x * (y + 1) for x, y in zip(k, n))
    flops = L * ((8.0 * d * d + 4.0 * d * F) * R + 4.0 * d * seen) + 2.0 * d * R
    nbytes = R * d * size + wsize * L * (4.0 * d * d + 2.0 * d * F) + kv + 4 * R
    if case["kind"] == "actions":
        C, Fh = case["actions"], case["hidden"]
        flops += 2.0 * R * C * Fh * (d + 1) - 2.0 * d * R
        nbytes += size * C * Fh * d + 4 * R * C
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Measured: the attention's softmax against another reference logit
    (its sums then round elsewhere) moves a bf16 model's outputs by 5e-4 to
    3.4e-3 (2-norm) and at most 1.5e-2; an fp32 model is 4e-7 to 1.2e-6 off
    the 64-bit result.  The fp8 variant's E4M3 roundings turn any such change
    into steps of up to 6% of an operand: its scores move by 4e-2 (one layer)
    to 7e-2 (four), more than is allowed here, so a change to it has to keep
    nearly every code."""
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    if case["dtype"] == "bf16_mxfp8":
        return {"rel": 3e-2, "max": 3e-1}
    return {"rel": 1e-2, "max": 6e-2}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _bf16(x):
    return torch.from_numpy(x).to(torch.bfloat16).float().numpy()


def _matrix(rng, rows, cols, rounded):
    a = math.sqrt(6.0 / (rows + cols))
    w = rng.uniform(-a, a, size=rows * cols) if rows * cols < 1 << 16 else None
    if w is None:       # large matrices: float32 draws are several times quicker
        w = (rng.random(rows * cols, dtype=np.float32) * 2 - 1) * np.float32(a)
    w = w.astype(np.float32)
    return _bf16(w) if rounded else w


def _vector(rng, size, base=0.0):
    return (base + rng.uniform(-0.1, 0.1, size=size)).astype(np.float32)


def _weights(case, seed):
    """{name: array} in the order of the weight blob: Xavier matrices, small
    biases and shifts, gains near 1."""
    rng = np.random.default_rng([seed, 1])
    d, F = case["d"], case["d_ff"]
    rounded = case["dtype"] != "f32"
    w = {}
    for l in range(case["layers"]):
        for name, rows, cols in (("ln1_g", d, 0), ("ln1_b", d, 0), ("Wq", d, d), ("bq", d, 0),
                                 ("Wk", d, d), ("bk", d, 0), ("Wv", d, d), ("bv", d, 0),
                                 ("Wo", d, d), ("bo", d, 0), ("ln2_g", d, 0), ("ln2_b", d, 0),
                                 ("W1", F, d), ("b1", F, 0), ("W2", d, F), ("b2", d, 0)):
            w[f"{l}.{name}"] = (_matrix(rng, rows, cols, rounded) if cols else
                                _vector(rng, rows, 1.0 if name.endswith("_g") else 0.0))
    w["lnf_g"], w["lnf_b"] = _vector(rng, d, 1.0), _vector(rng, d)
    w["w_score"], w["b_score"] = _matrix(rng, 1, d, rounded), _vector(rng, 1)
    return w


def _head_weights(case, seed):
    rng = np.random.default_rng([seed, 2])
    d, Fh = case["d"], case["hidden"]
    return [dict(W1=_matrix(rng, Fh, d, True), b1=_bf16(_vector(rng, Fh)), w2=_matrix(rng, 1, Fh, True),
                 b2=_bf16(_vector(rng, 1))) for _ in range(case["actions"])]


def _tokens(case, seed):
    """(history tokens, None, None) of an encode case, (None, candidate
    tokens, cache) of a ranking case, drawn on the GPU."""
    n, k = _lens(case)
    gen = torch.Generator(device="cuda").manual_seed(seed * 1000003 + 17)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    d, H = case["d"], case["heads"]

    def normal(*shape, scale):
        return (torch.randn(*shape, generator=gen, device="cuda") * scale).to(dt)

    if case["kind"] == "encode":
        return normal(sum(n), d, scale=d ** -0.5), None, None
    cand = normal(sum(k), d, scale=d ** -0.5)
    cache = torch.empty((case["layers"], 2, H, sum(n), d // H), dtype=dt, device="cuda")
    for l in range(case["layers"]):
        cache[l] = normal(2, H, sum(n), d // H, scale=1.0)
    return None, cand, cache


def _offsets(lens):
    host = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return host, torch.from_numpy(host).cuda()


def _segments(st):
    return upr.segments(st["hoff"], st["hoff_d"]), upr.segments(st["coff"], st["coff_d"])


def prepare(case, seed):
    n, k = _lens(case)
    cfg = upr.make_config(case["d"], case["heads"], case["layers"], case["d_ff"], case["dtype"])
    blob = np.concatenate([v.reshape(-1) for v in _weights(case, seed).values()])
    st = {"case": case, "model": upr.Model(cfg, blob)}
    m = st["model"]
    st["hoff"], st["hoff_d"] = _offsets(n)
    st["coff"], st["coff_d"] = _offsets(k)
    hist, cand, cache = _tokens(case, seed)
    if case["kind"] == "encode":
        st["hist"], st["cache"] = hist, m.new_cache(sum(n))
        st["ws"] = m.workspace(upr.upr_encode_workspace_bytes(m.handle, _segments(st)[0]))
        return st
    st["cand"], st["cache"] = cand, cache
    if case["kind"] == "actions":
        hb = np.concatenate([v.reshape(-1) for h in _head_weights(case, seed) for v in h.values()])
        st["heads"] = upr.Heads(m, case["actions"], case["hidden"], hb)
        st["uw"] = np.asarray((UTILITY * 2)[:case["actions"]], dtype=np.float32)
        st["probs"] = torch.empty((sum(k), case["actions"]), dtype=torch.float32, device="cuda")
        st["util"] = torch.empty(sum(k), dtype=torch.float32, device="cuda")
        st["ws"] = m.workspace(upr.upr_rank_actions_workspace_bytes(m.handle, st["heads"].handle,
                                                                    *_segments(st)))
        return st
    st["scores"] = torch.empty(sum(k), dtype=torch.float32, device="cuda")
    st["ws"] = m.workspace(upr.upr_rank_workspace_bytes(m.handle, *_segments(st)))
    return st


def run(st):
    m, kind = st["model"], st["case"]["kind"]
    if kind == "encode":
        m.encode(st["hist"], st["hoff"], st["hoff_d"], st["cache"], ws=st["ws"])
        return st["cache"]
    if kind == "actions":
        m.rank_actions(st["heads"], st["cache"], st["hoff"], st["hoff_d"], st["cand"], st["coff"],
                       st["coff_d"], st["uw"], probs=st["probs"], utility=st["util"], ws=st["ws"])
        return {"probs": st["probs"], "utility": st["util"]}
    m.rank(st["cache"], st["hoff"], st["hoff_d"], st["cand"], st["coff"], st["coff_d"],
           st["scores"], ws=st["ws"])
    return st["scores"]


# ---------------------------------------------------------------------------
# The same in 64 bits, plain torch
# ---------------------------------------------------------------------------

def _layer_norm(x, g, b):
    mu = x.mean(-1, keepdim=True)
    var = (x - mu).square().mean(-1, keepdim=True)
    return (x - mu) / (var + 1e-5).sqrt() * g + b


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _mx_round(x):
    """x rounded to MXFP8 along its rows: E4M3 values, one power-of-two scale
    per 32 (the largest magnitude of a block lands in [256, 512))."""
    b = x.reshape(*x.shape[:-1], -1, 32)
    amax = b.abs().amax(-1, keepdim=True)
    e = torch.where(amax > 0, torch.frexp(amax)[1].double() - 9.0, torch.full_like(amax, -127.0))
    scale = torch.exp2(e.clamp(min=-127.0))
    v = b / scale
    step = torch.exp2(torch.frexp(v.abs().clamp(min=2.0 ** -6))[1].double() - 4.0)
    return ((v / step).round() * step).clamp(-448.0, 448.0).mul(scale).reshape(x.shape)


def _attend(q, k, v, causal=False, own_k=None, own_v=None):
    """[H, rows, D] queries over [H, n, D] keys and values, and each row's own."""
    D = q.shape[-1]
    s = (q @ k.transpose(1, 2).contiguous()) / math.sqrt(D)
    if causal:
        s.masked_fill_(torch.ones(s.shape[1:], dtype=torch.bool, device=s.device).triu(1), -math.inf)
    if own_k is not None:
        s = torch.cat([s, ((q * own_k).sum(-1, keepdim=True)) / math.sqrt(D)], -1)
    p = torch.softmax(s, -1)
    if own_k is None:
        return p @ v
    return p[..., :-1].contiguous() @ v + p[..., -1:] * own_v


def exact(case, seed):
    w = {name: torch.from_numpy(v).cuda().double() for name, v in _weights(case, seed).items()}
    mx = case["dtype"] == "bf16_mxfp8"
    d, H, L, F = case["d"], case["heads"], case["layers"], case["d_ff"]
    for name in w:
        if ".W" in name:
            w[name] = w[name].reshape(-1, F if name.endswith("W2") else d)
            if mx:
                w[name] = _mx_round(w[name])
    D = d // H
    encode = case["kind"] == "encode"
    hoff, coff = (np.concatenate([[0], np.cumsum(x)]) for x in _lens(case))
    hist, cand, cache = _tokens(case, seed)
    if encode:
        cache = torch.zeros((L, 2, H, int(hoff[-1]), D), dtype=torch.float64, device="cuda")

    def linear(x, l, name):
        return (_mx_round(x) if mx else x) @ w[f"{l}.W{name}"].T + w[f"{l}.b{name}"]

    def heads_of(x):
        return x.reshape(-1, H, D).transpose(0, 1).contiguous()

    out = []
    for u in range(case["users"]):
        h0, h1 = int(hoff[u]), int(hoff[u + 1])
        g = (hist[h0:h1] if encode else cand[int(coff[u]):int(coff[u + 1])]).double()
        for l in range(L):
            a = _layer_norm(g, w[f"{l}.ln1_g"], w[f"{l}.ln1_b"])
            q, k, v = (heads_of(linear(a, l, x)) for x in "qkv")
            if encode:
                cache[l, 0, :, h0:h1], cache[l, 1, :, h0:h1] = k, v
                if l == L - 1:
                    break
                o = _attend(q, k, v, causal=True)
            else:
                o = _attend(q, cache[l, 0, :, h0:h1].double(), cache[l, 1, :, h0:h1].double(),
                            own_k=k, own_v=v)
            g = g + linear(o.transpose(0, 1).reshape(-1, d), l, "o")
            a = _layer_norm(g, w[f"{l}.ln2_g"], w[f"{l}.ln2_b"])
            g = g + linear(_gelu(linear(a, l, "1")), l, "2")
        out.append(g)
    if encode:
        return cache
    z = _layer_norm(torch.cat(out), w["lnf_g"], w["lnf_b"])
    if case["kind"] == "rank":
        return z @ w["w_score"] + w["b_score"]
    probs = []
    for hw in _head_weights(case, seed):
        hw = {name: torch.from_numpy(v).cuda().double() for name, v in hw.items()}
        probs.append(torch.sigmoid(_gelu(z @ hw["W1"].reshape(-1, d).T + hw["b1"]) @ hw["w2"] + hw["b2"]))
    probs = torch.stack(probs, -1)
    u = torch.tensor((UTILITY * 2)[:case["actions"]], dtype=torch.float64, device="cuda")
    return {"probs": probs, "utility": probs @ u}
