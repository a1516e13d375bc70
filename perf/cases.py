"""The verify step's work, as a program that decodes speculatively calls it.

Four kinds of call, all through the package's public entry points:

  attention  specrouter_verify_attention: the gamma_b + 1 new query rows of every
             sequence over its own bf16 KV cache (gamma = 0 is plain decode);
  accept     specrouter_accept_and_rollback: accept / resample / diverge over the
             verifier's and the draft's logits, with the rollback of the lengths
             (fp32 or bf16 logits; plain, tempered, greedy, top-k, top-p);
  step       one whole verify step of a serving loop: append the new K/V rows,
             attention under the validity mask, accept and roll back;
  compact    specrouter_kv_compact: the holes of a cache in the shared-length
             layout reclaimed.

Lengths and windows of a ragged batch are spread evenly over their range and
dealt to the sequences by the seed, so every seed does the same work. Logits
are N(0, sigma^2) for the verifier and the same plus noise for the draft; draft
tokens are samples of the draft's own (tempered, filtered) distribution.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2505_07680_amd as sr

DEV = "cuda"


# ----------------------------------------------------------------------------
# Cases

def _attention(name, B, Hq, Hkv, D, gamma, ctx, holes=-1.0):
    return {"kind": "attention", "name": name, "B": B, "Hq": Hq, "Hkv": Hkv, "D": D,
            "g_lo": gamma[0], "g_hi": gamma[1], "ctx_lo": ctx[0], "ctx_hi": ctx[1], "holes": holes}


def _accept(name, B, gamma, V, logits, temperature=1.0, top_k=0, top_p=1.0, noise=1.5, ctx=(1024, 1024)):
    return {"kind": "accept", "name": name, "B": B, "V": V, "g_lo": gamma[0], "g_hi": gamma[1], "logits": logits,
            "temperature": temperature, "top_k": top_k, "top_p": top_p, "noise": noise,
            "ctx_lo": ctx[0], "ctx_hi": ctx[1]}


def _step(name, B, Hq, Hkv, D, gamma, ctx, V, logits, temperature=1.0, noise=1.0, holes=0.0):
    return {"kind": "step", "name": name, "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "V": V, "g_lo": gamma[0],
            "g_hi": gamma[1], "ctx_lo": ctx[0], "ctx_hi": ctx[1], "logits": logits, "temperature": temperature,
            "top_k": 0, "top_p": 1.0, "noise": noise, "holes": holes}


def _compact(name, B, Hkv, D, ctx, holes):
    return {"kind": "compact", "name": name, "B": B, "Hkv": Hkv, "D": D, "ctx_lo": ctx[0], "ctx_hi": ctx[1],
            "holes": holes}


def listed():
    return [
        # one user, a small model: the latency of a whole step
        _step("step-tiny-b1", 1, 4, 4, 64, (4, 4), (128, 128), 1000, "f32"),
        # a small service on a multi-head-attention model, odd vocabulary, holed caches, ragged windows
        _step("step-mha-b8-v32001", 8, 32, 32, 128, (2, 6), (301, 1903), 32001, "bf16", 0.8, 1.0, 0.02),
        # an 8B-shaped verifier, 16 users, 2K context
        _attention("attn-b16-ctx2048", 16, 32, 8, 128, (5, 5), (2048, 2048)),
        # a 70B-shaped verifier over long documents
        _attention("attn-b4-ctx32768", 4, 64, 8, 128, (8, 8), (32768, 32768)),
        # a full ragged serving batch under the validity mask
        _attention("attn-b256-ragged", 256, 32, 8, 128, (1, 8), (256, 8192), 0.0),
        # the 1B-shaped drafter's plain decode, one row per sequence
        _attention("attn-decode-b32", 32, 32, 8, 64, (0, 0), (4096, 4096)),
        # accepting at the 16-user batch, fp32 logits, plain sampling
        _accept("accept-b16-f32", 16, (5, 5), 128256, "f32", ctx=(2048, 2048)),
        # accepting at the full ragged batch, bf16 logits, plain sampling
        _accept("accept-b256-bf16", 256, (1, 8), 128256, "bf16", noise=1.75, ctx=(256, 8192)),
        # greedy decoding at the chain's batch
        _accept("accept-greedy-b32-f32", 32, (8, 8), 128256, "f32", 0.0, noise=2.0, ctx=(4096, 4096)),
        # nucleus sampling, fp32 logits
        _accept("accept-topp-b16-f32", 16, (5, 5), 128256, "f32", 0.7, 0, 0.9, ctx=(2048, 2048)),
        # top-k and nucleus sampling together, a ragged bf16 batch
        _accept("accept-topk-topp-b64-bf16", 64, (1, 8), 128256, "bf16", 0.7, 50, 0.9, ctx=(256, 4096)),
        # reclaiming 2% holes of a batch's caches
        _compact("compact-b32-ctx4096", 32, 8, 128, (2048, 4096), 0.02),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(4, 4, 64), (32, 8, 64), (32, 8, 128), (32, 8, 128), (64, 8, 128), (32, 32, 128), (32, 2, 64)]
_VOCABS = [1000, 32000, 32001, 50257, 128256, 128256]
_MAX_KV = 3.0e9       # bytes of K and V read
_MAX_LOGITS = 5.0e8   # bytes of logits read


def draw(rng):
    """A case of the listed kinds with sizes over the whole range."""
    kind = rng.choice(["attention", "attention", "accept", "accept", "accept", "step", "compact"])
    B = _log_int(rng, 1, 256)
    g_hi = rng.randint(1, 8) if rng.random() < 0.9 else rng.randint(9, 16)
    g_lo = g_hi if rng.random() < 0.5 else rng.randint(0, g_hi)
    Hq, Hkv, D = rng.choice(_HEADS)
    if kind in ("attention", "step", "compact"):
        ctx_hi = _log_int(rng, 64, 32768)
        most = _MAX_KV / (3 if kind == "compact" else 1)
        ctx_hi = max(16, min(ctx_hi, int(most / (4.0 * B * Hkv * D))))
        ctx_lo = ctx_hi if rng.random() < 0.5 else max(1, ctx_hi // rng.randint(2, 16))
    if kind == "attention":
        if rng.random() < 0.15:
            g_lo = g_hi = 0
        holes = rng.choice([-1.0, 0.0, 0.02])
        return {k: v for k, v in _attention("", B, Hq, Hkv, D, (g_lo, g_hi), (ctx_lo, ctx_hi), holes).items()
                if k != "name"}
    if kind == "compact":
        return {k: v for k, v in _compact("", B, Hkv, D, (ctx_lo, ctx_hi), rng.choice([0.005, 0.02, 0.1])).items()
                if k != "name"}
    V = rng.choice(_VOCABS) if rng.random() < 0.5 else _log_int(rng, 1000, 160000)
    logits = rng.choice(["f32", "bf16"])
    esz = 4 if logits == "f32" else 2
    noise = round(rng.uniform(0.5, 3.0), 2)
    if kind == "step":
        B = max(1, min(B, int(_MAX_LOGITS / ((2 * g_hi + 1) * V * esz))))
        return {k: v for k, v in _step("", B, Hq, Hkv, D, (g_lo, g_hi), (ctx_lo, ctx_hi), V, logits,
                                       rng.choice([0.0, 0.7, 1.0, 1.0]), noise, rng.choice([0.0, 0.02])).items()
                if k != "name"}
    temperature, top_k, top_p = rng.choice([(1.0, 0, 1.0), (1.0, 0, 1.0), (0.7, 0, 1.0), (0.0, 0, 1.0), (0.6, 0, 0.95),
                                            (0.7, 0, 0.9), (0.7, 20, 1.0), (1.0, 50, 1.0), (0.8, 40, 0.95),
                                            (0.7, 50, 0.9)])
    most = _MAX_LOGITS / (3 if top_k or top_p < 1.0 else 1)
    B = max(1, min(B, int(most / ((2 * g_hi + 1) * V * esz))))
    return {k: v for k, v in _accept("", B, (g_lo, g_hi), V, logits, temperature, top_k, top_p, noise,
                                     (256, 4096)).items() if k != "name"}


# ----------------------------------------------------------------------------
# Inputs (torch only)

def _spread(lo, hi, n):
    """n whole numbers spread evenly over [lo, hi]."""
    return [lo + ((hi - lo + 1) * (2 * i + 1)) // (2 * n) for i in range(n)]


def _lens(case):
    B = case["B"]
    g = _spread(case["g_lo"], case["g_hi"], B) if "g_lo" in case else [0] * B
    c = _spread(case["ctx_lo"], case["ctx_hi"], B)
    return g, c


def _gen(seed, what):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + what) & 0x7FFFFFFFFFFF)
    return g


def _dealt(case, seed):
    """(gamma, ctx) as int32 tensors, dealt to the sequences by the seed."""
    g, c = _lens(case)
    r = np.random.default_rng(seed)
    B = case["B"]
    g = np.asarray(g, np.int32)[r.permutation(B)]
    c = np.asarray(c, np.int32)[r.permutation(B)]
    return torch.from_numpy(g).to(DEV), torch.from_numpy(c).to(DEV)


def _cap(case):
    need = case["ctx_hi"] + case.get("g_hi", 0) + 1
    return (need + 63) // 64 * 64


def _cache(case, seed):
    B, Hkv, D = case["B"], case["Hkv"], case["D"]
    shape = (B, Hkv, _cap(case), D)
    g = _gen(seed, 1)
    k = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=g)
    v = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=g)
    return k, v


def _holed(case, seed, length):
    """u8 [B, cap]: 1 below each sequence's length but for the holes (None: no mask in use)."""
    if case["holes"] < 0:
        return None
    cap = _cap(case)
    keep = torch.arange(cap, device=DEV)[None, :] < length[:, None]
    if case["holes"] > 0:
        keep &= torch.rand((case["B"], cap), device=DEV, generator=_gen(seed, 2)) >= case["holes"]
    return keep.to(torch.uint8)


def _padded(B, rows, V, dtype):
    """[B, rows, V] whose batch stride is a multiple of 16 bytes."""
    per = 8 if dtype == torch.bfloat16 else 4
    n = (max(rows, 1) * V + per - 1) // per * per
    return torch.zeros((B, n), dtype=dtype, device=DEV)[:, : rows * V].unflatten(1, (rows, V))


def _keep(z, top_k, top_p):
    """The entries that top-k, then top-p keep (rows of z in the last dimension, already divided by T)."""
    ok = torch.ones_like(z, dtype=torch.bool)
    if 0 < top_k < z.shape[-1]:
        ok = z >= torch.topk(z, top_k, dim=-1).values[..., -1:]
    if top_p < 1.0:
        w, at = torch.sort(torch.where(ok, z, -math.inf), dim=-1, descending=True)
        e = torch.exp(w - w[..., :1])
        above = torch.cumsum(e, -1) - e
        # an entry stays iff the mass of the strictly larger ones is below p: with ties, that of the first equal one
        first = torch.cat([torch.ones_like(w[..., :1], dtype=torch.bool), w[..., 1:] < w[..., :-1]], -1)
        above = torch.where(first, above, torch.zeros_like(above)).cummax(-1).values
        kept = (above < top_p * e.sum(-1, keepdim=True)) & (e > 0)
        n = kept.sum(-1, keepdim=True)
        low = torch.gather(w, -1, n - 1)
        ok &= z >= low
    return ok


def _logits(case, seed, gamma):
    B, V, G = case["B"], case["V"], case["g_hi"]
    dtype = torch.float32 if case["logits"] == "f32" else torch.bfloat16
    p, q = _padded(B, G + 1, V, dtype), _padded(B, G, V, dtype)
    drafts = torch.zeros((B, G), dtype=torch.int32, device=DEV)
    gen = _gen(seed, 3)
    T = case["temperature"]
    group = max(1, int(3e7 // ((G + 1) * V)))
    for b in range(0, B, group):
        n = min(group, B - b)
        zp = torch.randn((n, G + 1, V), device=DEV, generator=gen) * 3.0
        zq = zp[:, :G] + torch.randn((n, G, V), device=DEV, generator=gen) * case["noise"]
        p[b:b + n].copy_(zp)
        q[b:b + n].copy_(zq)
        z = q[b:b + n].float()
        if T > 0:
            z = z / T
            if case["top_k"] or case["top_p"] < 1.0:
                z = torch.where(_keep(z, case["top_k"], case["top_p"]), z, -math.inf)
            # a sample of softmax(z): the largest of z + Gumbel noise
            z = z - torch.log(torch.empty_like(z).exponential_(generator=gen).clamp_min_(1e-30))
        drafts[b:b + n] = z.argmax(-1).to(torch.int32)
    u_acc = torch.rand((B, G), device=DEV, generator=gen)
    u_res = torch.rand((B, G + 1), device=DEV, generator=gen)
    return {"p": p, "q": q, "drafts": drafts, "u_acc": u_acc, "u_res": u_res}


def _inputs(case, seed):
    gamma, ctx = _dealt(case, seed)
    s = {"gamma": gamma, "ctx": ctx, "kv_len": (ctx + gamma + 1).to(torch.int32)}
    if case["kind"] in ("attention", "step", "compact"):
        s["k"], s["v"] = _cache(case, seed)
    if case["kind"] in ("attention", "step"):
        shape = (case["B"], case["g_hi"] + 1, case["Hq"], case["D"])
        s["q_rows"] = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=_gen(seed, 4))
        s["scale"] = 1.0 / math.sqrt(case["D"])
    if case["kind"] == "attention":
        s["mask"] = _holed(case, seed, s["kv_len"])
    if case["kind"] == "step":
        s["mask"] = _holed(case, seed, ctx)
        shape = (case["B"], case["g_hi"] + 1, case["Hkv"], case["D"])
        g = _gen(seed, 5)
        s["k_new"] = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=g)
        s["v_new"] = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=g)
    if case["kind"] == "compact":
        s["kv_len"] = ctx
        s["mask"] = _holed(case, seed, ctx)
    if case["kind"] in ("accept", "step"):
        s.update(_logits(case, seed, gamma))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    B, G = case["B"], case.get("g_hi", 0)
    s["kind"] = case["kind"]
    s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    if case["kind"] in ("attention", "step"):
        s["out"] = torch.empty((B, G + 1, case["Hq"], case["D"]), dtype=torch.float32, device=DEV)
        s["att_ws"] = sr.attention_workspace(B, G, case["Hq"], case["Hkv"], case["D"], _cap(case), device=DEV)
    if case["kind"] in ("accept", "step"):
        code = sr.SR_F32 if case["logits"] == "f32" else sr.SR_BF16
        s["acc"] = sr.AcceptBuffers(B, G, case["V"], code, device=DEV)
        s["phys"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        s["cache_len"] = s["kv_len"].clone()
        s["cap"] = _cap(case)
        s["sampling"] = {"temperature": case["temperature"], "top_k": case["top_k"], "top_p": case["top_p"]}
    if case["kind"] == "compact":
        s["mask0"], s["len0"] = s["mask"].clone(), s["kv_len"].clone()
    return s


# ----------------------------------------------------------------------------
# One pass

def _run_attention(s):
    return sr.specrouter_verify_attention(s["q_rows"], s["k"], s["v"], s["mask"], s["kv_len"], s["gamma"], s["out"],
                                          s["scale"], s["att_ws"], s["status"])


def _run_accept(s, mask):
    a = s["acc"]
    sr.specrouter_accept_and_rollback(s["p"], s["q"], s["drafts"], s["gamma"], s["u_acc"], s["u_res"], s["kv_len"],
                                      a.accept_len, a.out_tokens, a.new_len, a.accept_prob, a.p_tok, a.q_tok, a.kl,
                                      a.tv, s["cache_len"], mask, s["phys"], a.workspace, s["status"],
                                      L_cap=s["cap"], **s["sampling"])
    return {"accept_len": a.accept_len, "out_tokens": a.out_tokens, "new_len": a.new_len,
            "accept_prob": a.accept_prob, "p_tok": a.p_tok, "q_tok": a.q_tok, "kl": a.kl, "tv": a.tv,
            "cache_len": s["cache_len"], "phys": s["phys"]}


def run(s):
    if s["kind"] == "attention":
        return {"out": _run_attention(s)}
    if s["kind"] == "accept":
        return _run_accept(s, None)
    if s["kind"] == "step":
        s["cache_len"].copy_(s["ctx"])  # the lengths that the step starts from
        sr.specrouter_kv_append(s["k_new"], s["v_new"], s["gamma"], s["k"], s["v"], s["mask"], s["cache_len"],
                                status=s["status"])
        out = _run_attention(s)
        return {"out": out, "mask": s["mask"], **_run_accept(s, s["mask"])}
    s["mask"].copy_(s["mask0"])  # the holes that the steps before left
    s["kv_len"].copy_(s["len0"])
    sr.specrouter_kv_compact(s["k"], s["v"], s["mask"], s["kv_len"], s["status"])
    return {"k": s["k"], "v": s["v"], "mask": s["mask"], "kv_len": s["kv_len"]}


# ----------------------------------------------------------------------------
# What a pass cannot do without, and how exact it is

def work(case):
    g, c = _lens(case)
    B, bytes_, flops = case["B"], 0.0, 0.0
    if case["kind"] in ("attention", "step"):
        Hq, Hkv, D = case["Hq"], case["Hkv"], case["D"]
        keys = sum(x + y + 1 for x, y in zip(g, c))
        rows = sum(x + 1 for x in g)
        bytes_ += keys * Hkv * D * 4 + rows * Hq * D * 6 + (keys if case["holes"] >= 0 else 0)
        flops += 4.0 * Hq * D * sum((x + 1) * (x + y + 1) for x, y in zip(g, c))
        if case["kind"] == "step":
            bytes_ += rows * Hkv * D * 8
    if case["kind"] in ("accept", "step"):
        esz = 4 if case["logits"] == "f32" else 2
        n = sum(2 * x + 1 for x in g) * case["V"]
        bytes_ += n * esz + B * (case["g_hi"] + 1) * 40
        flops += 8.0 * n
    if case["kind"] == "compact":
        # every row from the first hole on is read and written
        bytes_ += sum(max(0.0, x - 1.0 / case["holes"]) * (2 - case["holes"]) for x in c) * case["Hkv"] * case["D"] * 4
        bytes_ += 2 * sum(c) + 1
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] == "compact":
        return "exact"
    if case["kind"] in ("attention", "step"):
        # probabilities and products in bf16, sums in 32 bits (1.0e-3 to 1.7e-3 off the 64-bit result)
        return {"rel": 6.5e-3, "max": 0.1, "differ": 0.005}
    # exponentials and sums in 32 bits (up to 2e-7 off; some terms of a small KL cancel); a token whose uniform lies on
    # a bin's edge may differ
    return {"rel": 2e-6, "max": 1e-4, "differ": 0.005}


# ----------------------------------------------------------------------------
# The same in 64 bits, in plain torch

def _exact_attention(case, s, k, v, mask):
    B, G1, Hq, D = s["q_rows"].shape
    Hkv = case["Hkv"]
    grp = Hq // Hkv
    out = torch.zeros((B, G1, Hq, D), dtype=torch.float64, device=DEV)
    for b in range(B):
        g, L = int(s["gamma"][b]), int(s["kv_len"][b])
        q = s["q_rows"][b, : g + 1].double().reshape(g + 1, Hkv, grp, D).permute(1, 2, 0, 3)
        q = q.reshape(Hkv, grp * (g + 1), D).contiguous()
        kk, vv = k[b, :, :L].double(), v[b, :, :L].double()
        sc = torch.matmul(q, kk.transpose(1, 2).contiguous()) * s["scale"]
        pos = torch.arange(L, device=DEV)
        see = pos[None, :] <= (L - (g + 1) + torch.arange(g + 1, device=DEV))[:, None]
        if mask is not None:
            see = see & (mask[b, :L] != 0)[None, :]
        see = see[None].expand(grp, -1, -1).reshape(1, grp * (g + 1), L)
        sc = torch.where(see, sc, -math.inf)
        m = sc.amax(-1, keepdim=True).clamp_min(-1e300)
        w = torch.exp(sc - m)
        d = w.sum(-1, keepdim=True)
        o = torch.matmul(w, vv) / torch.where(d > 0, d, torch.ones_like(d))
        out[b, : g + 1] = o.reshape(Hkv, grp, g + 1, D).permute(2, 0, 1, 3).reshape(g + 1, Hq, D)
    return out


def _softmax(z, case):
    if case["top_k"] or case["top_p"] < 1.0:
        z = torch.where(_keep(z, case["top_k"], case["top_p"]), z, -math.inf)
    return torch.softmax(z, -1)


def _exact_accept(case, s):
    B, G, V, T = case["B"], case["g_hi"], case["V"], case["temperature"]
    f = dict(dtype=torch.float64, device=DEV)
    o = {n: torch.full((B, G), math.nan, **f) for n in ("accept_prob", "p_tok", "q_tok", "kl", "tv")}
    acc, toks = [], torch.full((B, G + 1), -1, dtype=torch.int32)
    gam, dr = s["gamma"].tolist(), s["drafts"].tolist()
    ua, ur = s["u_acc"].double().cpu(), s["u_res"].double().cpu()
    for b in range(B):
        g = gam[b]
        zp, zq = s["p"][b, : g + 1].double(), s["q"][b, :g].double()
        x = s["drafts"][b, :g].long()
        at = torch.arange(g, device=DEV)
        if T == 0:
            ap, aq = zp.argmax(-1), zq.argmax(-1)
            px, qx = (ap[:g] == x).double(), (aq == x).double()
            a = px
            same = ap[:g] == aq
            kl = torch.where(same, 0.0, math.inf).double()
            tv = (~same).double()
        else:
            p, q = _softmax(zp / T, case), _softmax(zq / T, case)
            px, qx = p[at, x], q[at, x]
            a = torch.where(px >= qx, torch.ones_like(px), px / qx)
            pp = p[:g]
            kl = torch.where(pp > 0, pp * (torch.log(pp) - torch.log(q)), torch.zeros_like(pp)).sum(-1)
            tv = 0.5 * (pp - q).abs().sum(-1)
        for n, t in (("accept_prob", a), ("p_tok", px), ("q_tok", qx), ("kl", kl), ("tv", tv)):
            o[n][b, :g] = t
        al = a.tolist()
        k = next((j for j in range(g) if not (al[j] > 0.5 if T == 0 else float(ua[b, j]) < al[j])), g)
        if T == 0:
            t = int(ap[k])
        else:
            w = p[k]
            if k < g:
                r = (p[k] - q[k]).clamp_min(0)
                w = r if float(r.sum()) > 0 else w
            cdf = torch.cumsum(w, 0)
            t = min(int(torch.searchsorted(cdf, cdf[-1:] * float(ur[b, k]), right=True)), V - 1)
        acc.append(k)
        toks[b, :k] = torch.tensor(dr[b][:k], dtype=torch.int32)
        toks[b, k] = t
    k = torch.tensor(acc, dtype=torch.int32, device=DEV)
    new = s["kv_len"] - s["gamma"] + k
    return {"accept_len": k, "out_tokens": toks, "new_len": new, **o, "cache_len": new.clone(),
            "phys": new.max().reshape(1)}


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "attention":
        return {"out": _exact_attention(case, s, s["k"], s["v"], s["mask"])}
    if case["kind"] == "accept":
        return _exact_accept(case, s)
    if case["kind"] == "step":
        k, v, mask = s["k"], s["v"], s["mask"]
        for b in range(case["B"]):
            n, c = int(s["gamma"][b]) + 1, int(s["ctx"][b])
            k[b, :, c:c + n] = s["k_new"][b, :n].transpose(0, 1)
            v[b, :, c:c + n] = s["v_new"][b, :n].transpose(0, 1)
            mask[b, c:c + n] = 1
        out = _exact_attention(case, s, k, v, mask)
        o = _exact_accept(case, s)
        pos = torch.arange(mask.shape[1], device=DEV)[None, :]
        mask[(pos >= o["new_len"][:, None]) & (pos < s["kv_len"][:, None])] = 0
        return {"out": out, "mask": mask, **o}
    k, v = s["k"].double(), s["v"].double()
    mask, n = s["mask"].clone(), s["kv_len"].clone()
    for b in range(case["B"]):
        L = int(s["kv_len"][b])
        at = torch.nonzero(s["mask"][b, :L]).flatten()
        m = int(at.numel())
        k[b, :, :m], v[b, :, :m] = k[b][:, at], v[b][:, at]
        mask[b, :L] = (torch.arange(L, device=DEV) < m).to(torch.uint8)
        n[b] = m
    return {"k": k, "v": v, "mask": mask, "kv_len": n}
