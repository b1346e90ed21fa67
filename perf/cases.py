"""The calls that this library's performance is judged by.

A case is one pass through the public entry points as a serving program makes
it.  Its `kind`:

  evict   a finished prefill is compressed (score, select, compact) and the
          first generated token attends over the compressed cache;
  score   the scores alone, with any of the options;
  write   the prefill's KV-cache write with the first sweep as its by-product,
          then the scores from the sums it hands over (K read once);
  keep    selection and compaction on scores that are already there;
  decode  one generated token's attention over a compressed cache.

Keys follow the recipe of the synthetic workloads: 75 % near-duplicate visual
tokens in groups of 256, the rest text, all sharing an offset, which the
queries share too; values are N(0, 1).

In `evict` the selected positions themselves are not returned: one exchange
of two keys whose scores agree to the last bits moves every position between
them.  The attention over the kept rows, which does not depend on their order,
stands for them there; `keep` returns positions and rows whole, on given
scores, and they are compared exactly.
"""
import math

import torch

import paper_2609_06663_amd as P
from paper_2609_06663_amd.pipeline import EvictionPass

MODES = {"per_head": P.PER_HEAD, "flat": P.LAYER_FLAT, "heads": P.HEAD_BUDGETS}
TYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
NORMS = {"minmax": P.NORM_MINMAX, "winsor": P.NORM_WINSOR, "mad": P.NORM_MAD}


def listed():
    return [
        # the smallest call: two fp32 heads over 512 tokens; launches and host work are all there is
        {"name": "evict_tiny_f32", "kind": "evict", "dtype": "f32", "layers": 1, "q_heads": 2, "kv_heads": 2, "dim": 128,
         "window": 8, "lens": "512", "mode": "per_head", "keep": 0.25},
        # one layer of a short prompt as soon as the prefill has finished it; 56 window rows
        {"name": "evict_layer_8k", "kind": "evict", "dtype": "bf16", "layers": 1, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 8, "lens": "8192", "mode": "per_head", "keep": 0.2},
        # one layer of a long prompt, called layer by layer
        {"name": "evict_layer_32k", "kind": "evict", "dtype": "bf16", "layers": 1, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": "32768", "mode": "per_head", "keep": 0.2},
        # a batch of packed prompts of ragged lengths whose heads share a layer's budget
        {"name": "evict_packed_flat", "kind": "evict", "dtype": "bf16", "layers": 1, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": "29871,4133,17402,32001,9055,21770,12289,26646", "mode": "flat", "keep": 0.15},
        # every head its own keys (no grouped queries), a very long prompt and a small budget
        {"name": "evict_mha_64k", "kind": "evict", "dtype": "bf16", "layers": 1, "q_heads": 32, "kv_heads": 32, "dim": 128,
         "window": 8, "lens": "65536", "mode": "per_head", "keep": 0.03125},
        # the whole model's cache in one call: the headline benchmark's shape
        {"name": "evict_stack28", "kind": "evict", "dtype": "bf16", "layers": 28, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": "32768", "mode": "per_head", "keep": 0.2},
        # a model with 64-wide heads
        {"name": "score_d64", "kind": "score", "dtype": "bf16", "layers": 12, "q_heads": 16, "kv_heads": 4, "dim": 64,
         "window": 4, "lens": "16384", "norm": "minmax", "vnorm": False, "std": False, "prefix": False, "pool": 5},
        # the method's alternatives together, on ragged odd lengths: value norm, MAD, r_std, prefix centroid
        {"name": "score_options", "kind": "score", "dtype": "bf16", "layers": 4, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": "30001,4099,12345", "norm": "mad", "vnorm": True, "std": True, "prefix": True, "pool": 7},
        # the prefill writes its cache and the pass reads K once
        {"name": "write_score_stack28", "kind": "write", "dtype": "bf16", "layers": 28, "q_heads": 28, "kv_heads": 4,
         "dim": 128, "window": 4, "lens": "32768"},
        # a budget for each (layer, head), falling from the first layer to the last
        {"name": "keep_pyramid28", "kind": "keep", "dtype": "bf16", "layers": 28, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": "32768", "mode": "heads", "keep": 0.2},
        # one generated token in one layer: the call that every token makes in every layer
        {"name": "decode_layer", "kind": "decode", "dtype": "bf16", "layers": 1, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": "32768", "mode": "per_head", "keep": 0.2},
        # the same for a batch of sequences whose heads kept different numbers of rows
        {"name": "decode_batch", "kind": "decode", "dtype": "bf16", "layers": 1, "q_heads": 28, "kv_heads": 4, "dim": 128,
         "window": 4, "lens": ",".join(str(4096 + (7919 * i) % 28673) for i in range(16)), "mode": "flat", "keep": 0.2},
    ]


# (query heads, KV heads) of the drawn cases: grouped 7, 4, 8 and 2 to one, and one to one
HEADS = [(28, 4), (16, 4), (32, 8), (16, 2), (8, 4), (32, 32), (2, 2)]
MOST_KEYS = 28 * 4 * 32768  # (layer, head, token) rows of the largest listed case


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["evict", "evict", "evict", "score", "score", "write", "keep", "decode", "decode"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    dim = rng.choice([128, 128, 128, 64])
    q_heads, kv_heads = rng.choice(HEADS)
    window = rng.choice([w for w in (4, 8, 16) if q_heads // kv_heads * w <= 64])
    most = MOST_KEYS if dtype == "bf16" else MOST_KEYS // 4  # fp32 is for small models and checks
    seqs = rng.choice([1, 1, 1, 2, 3, 5, 8])
    if kind == "decode":
        seqs = rng.choice([1, 2, 4, 8, 16])
    lens = [max(window + 1, _spread(rng, 512, 65536)) for _ in range(seqs)]
    while sum(lens) * kv_heads > most:
        lens = [max(512, n // 2) for n in lens]
    layers = _spread(rng, 1, max(1, min(28, most // (sum(lens) * kv_heads))))
    case = {"kind": kind, "dtype": dtype, "layers": layers, "q_heads": q_heads, "kv_heads": kv_heads, "dim": dim,
            "window": window, "lens": ",".join(map(str, lens))}
    if kind in ("evict", "keep", "decode"):
        case["mode"] = rng.choice(["per_head", "per_head", "flat"] if kind != "keep" else ["per_head", "flat", "heads"])
        case["keep"] = round(math.exp(rng.uniform(math.log(0.05), math.log(0.4))), 4)
    if kind == "score":
        case.update(norm=rng.choice(["minmax", "minmax", "winsor", "mad"]), vnorm=rng.random() < 0.3,
                    std=rng.random() < 0.25, prefix=rng.random() < 0.25, pool=rng.choice([5, 5, 3, 7]))
    return case


# ---------------------------------------------------------------------------

def _lens(case):
    return [int(t) for t in str(case["lens"]).split(",")]


def _shape(case):
    cu = [0]
    for t in _lens(case):
        cu.append(cu[-1] + t)
    return P.Shape(case["layers"], case["q_heads"], case["kv_heads"], case["dim"], case["window"], cu)


def _params(case):
    return P.Params(pool_kernel=case.get("pool", 5), norm_mode=NORMS[case.get("norm", "minmax")],
                    imp_mode=P.IMP_ATTN_VNORM if case.get("vnorm") else P.IMP_ATTN,
                    redundancy=P.RED_STD if case.get("std") else P.RED_EUCLID,
                    centroid_scope=P.CENTROID_PREFIX if case.get("prefix") else P.CENTROID_ALL)


def _budget(case):
    """Tokens kept per head: one number per sequence, or per (layer, head) in a pyramid over the layers."""
    w = case["window"]
    if case["mode"] != "heads":
        return [max(w, int(case["keep"] * t)) for t in _lens(case)]
    mean = case["keep"] * max(_lens(case))
    n = case["layers"]
    layer = [max(w, int(mean * (1.9 - 1.8 * i / (n - 1) if n > 1 else 1.0))) for i in range(n)]
    return [b for b in layer for _ in range(case["kv_heads"])]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype):
    """N(0, 1) made piece by piece: the fp32 draws of a whole stack are not held at once."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 26
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device="cuda")
    return out


def _offsets(case, g):
    """[layers][kv_heads][sequences][dim]: the offset that a head's keys and queries of a sequence share."""
    L, H, B, D = case["layers"], case["kv_heads"], len(_lens(case)), case["dim"]
    u = torch.randn(L, H, B, D, generator=g, device="cuda")
    u /= u.norm(dim=-1, keepdim=True)
    a = 0.5 + 2.5 * torch.rand(L, 1, 1, 1, generator=g, device="cuda") if L > 1 else 1.5
    return u * (a * math.sqrt(D))


def _keys(case, g, off):
    L, H, D, lens = case["layers"], case["kv_heads"], case["dim"], _lens(case)
    K = torch.empty(L, H, sum(lens), D, dtype=TYPES[case["dtype"]], device="cuda")
    for l in range(L):
        at = 0
        for s, T in enumerate(lens):
            k = torch.randn(H, T, D, generator=g, device="cuda")
            nv = (3 * T // 4) // 256
            c = torch.randn(H, nv, 1, D, generator=g, device="cuda")
            k[:, :256 * nv] = (k[:, :256 * nv].view(H, nv, 256, D) * 0.1 + c).view(H, 256 * nv, D)
            K[l, :, at:at + T] = k + off[l, :, s, None, :]
            at += T
    return K


def _queries(case, g, off, rows):
    """[layers][q_heads][sequences][rows][dim]."""
    G = case["q_heads"] // case["kv_heads"]
    q = torch.randn(case["layers"], case["q_heads"], len(_lens(case)), rows, case["dim"], generator=g, device="cuda")
    return (q + off.repeat_interleave(G, dim=1)[:, :, :, None, :]).to(TYPES[case["dtype"]]).contiguous()


def _inputs(case, seed):
    g = _generator(seed)
    off = _offsets(case, g)
    K = _keys(case, g, off)
    return g, off, K, _queries(case, g, off, case["window"])


def _max_count(case):
    """A bound of the rows that one head can keep."""
    w, H = case["window"], case["kv_heads"]
    if case["mode"] == "flat":
        return max(min(t, H * (b - w) + w) for t, b in zip(_lens(case), _budget(case)))
    return max(min(t, b) for t, b in zip(_lens(case), _budget(case)))


def _empty(*shape, dtype=torch.float32):
    return torch.empty(*shape, dtype=dtype, device="cuda")


def _zeros(nbytes):
    return torch.zeros(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def _decode_out(case, s):
    L, Hq, B, D = case["layers"], case["q_heads"], len(_lens(case)), case["dim"]
    s.update(O=_empty(L, Hq, B, D), lse=_empty(L, Hq, B), max_count=_max_count(case))
    s["ws_dec"] = _zeros(P.ecokv_decode_workspace_size(s["shape"], s["max_count"]))


def _kept_counts(case, g):
    """Rows that each (layer, head, sequence) kept: the budget, or a share of the layer's."""
    L, H, w = case["layers"], case["kv_heads"], case["window"]
    b = torch.tensor([min(t, n) for t, n in zip(_lens(case), _budget(case))], device="cuda").view(1, 1, -1)
    T = torch.tensor(_lens(case), device="cuda").view(1, 1, -1)
    if case["mode"] != "flat":
        return b.expand(L, H, -1).contiguous().to(torch.int32)
    share = torch.rand(L, H, b.numel(), generator=g, device="cuda") + 0.2
    n = w + (share / share.sum(dim=1, keepdim=True) * (H * (b - w))).long()
    return torch.minimum(n, T).to(torch.int32).contiguous()


def prepare(case, seed):
    s = {"kind": case["kind"], "shape": _shape(case), "params": _params(case)}
    dtype = TYPES[case["dtype"]]
    L, H, D, lens = case["layers"], case["kv_heads"], case["dim"], _lens(case)
    if case["kind"] == "evict":
        g, off, s["K"], s["Q"] = _inputs(case, seed)
        s["V"] = _normal(g, s["K"].shape, dtype)
        s["Qd"] = _queries(case, g, off, 1)
        s["ep"] = EvictionPass(s["shape"], _budget(case), MODES[case["mode"]], s["params"], dtype)
        _decode_out(case, s)
    elif case["kind"] in ("score", "write"):
        g, off, s["K"], s["Q"] = _inputs(case, seed)
        vals = case["kind"] == "write" or case["vnorm"]
        s["V"] = _normal(g, s["K"].shape, dtype) if vals else None
        U = s["shape"].units
        s.update(scores=_empty(s["shape"].score_numel()), lam=_empty(U), stats=_empty(U, P.NSTATS),
                 ws=_zeros(P.ecokv_workspace_size(s["shape"], s["params"])))
        if case["kind"] == "write":
            R = case["q_heads"] // H * case["window"]
            for n in ("K", "V"):  # the new rows arrive token by token, every head's row of a token together
                s[n + "new"] = s[n].transpose(1, 2).contiguous()
                s[n].zero_()
            s.update(pre=_empty(U, 2 * D + 2 * R), ws_pre=_zeros(P.ecokv_prefill_workspace_size(s["shape"])))
    elif case["kind"] == "keep":
        g = _generator(seed)
        n = s["shape"].score_numel()
        # most scores small and close together, a long tail of large ones, each head on a scale of its own
        x = torch.rand(L, H, n // (L * H), generator=g, device="cuda").pow_(4) + 0.3
        x *= torch.exp(0.2 * torch.randn(L, H, 1, generator=g, device="cuda"))
        s["scores"] = x
        s["K"], s["V"] = (_normal(g, (L, H, sum(lens), D), dtype) for _ in range(2))
        s["ep"] = EvictionPass(s["shape"], _budget(case), MODES[case["mode"]], s["params"], dtype)
        s["ep"].scores = x.view(-1)
    else:
        g = _generator(seed)
        off = _offsets(case, g)
        s["Qd"] = _queries(case, g, off, 1)
        s["counts"] = _kept_counts(case, g)
        c = s["counts"].view(-1).long()
        s["offsets"] = (c.cumsum(0) - c).to(torch.int32).view_as(s["counts"])
        own = torch.repeat_interleave(torch.arange(c.numel(), device="cuda"), c)  # the unit of each kept row
        kc = torch.empty(own.numel(), D, dtype=dtype, device="cuda")
        flat = off.view(-1, D)
        for i in range(0, own.numel(), 1 << 20):
            o = own[i:i + (1 << 20)]
            kc[i:i + (1 << 20)] = torch.randn(o.numel(), D, generator=g, device="cuda") + flat[o]
        s["Kc"], s["Vc"] = kc, _normal(g, (own.numel(), D), dtype)
        _decode_out(case, s)
    return s


def _decode(s, Kc, Vc, counts, offsets):
    P.ecokv_decode(s["Qd"], Kc, Vc, s["shape"], counts, offsets, s["max_count"], s["O"], s["lse"], s["ws_dec"])
    return s["O"], s["lse"]


def run(s):
    if s["kind"] == "evict":
        ep = s["ep"].run(s["K"], s["V"], s["Q"])
        O, lse = _decode(s, ep.Kc, ep.Vc, ep.counts, ep.offsets)
        return {"scores": ep.scores, "lambda": ep.lambda_, "stats": ep.stats.view(-1, P.NSTATS), "O": O, "lse": lse}
    if s["kind"] == "score":
        P.ecokv_score_v(s["K"], s["V"], s["Q"], s["shape"], s["params"], s["scores"], s["lam"], s["stats"], s["ws"])
        return {"scores": s["scores"], "lambda": s["lam"], "stats": s["stats"]}
    if s["kind"] == "write":
        P.ecokv_prefill_write(s["Knew"], s["Vnew"], s["Q"], s["shape"], s["params"], s["K"], s["V"], s["pre"],
                              s["ws_pre"])
        P.ecokv_score_pre(s["K"], None, s["Q"], s["shape"], s["params"], s["pre"], s["scores"], s["lam"], s["stats"],
                          s["ws"])
        return {"K": s["K"], "V": s["V"], "scores": s["scores"], "lambda": s["lam"], "stats": s["stats"]}
    if s["kind"] == "keep":
        ep = s["ep"]
        ep.select()
        ep.compact(s["K"], s["V"])
        return {"idx": ep.idx, "counts": ep.counts, "offsets": ep.offsets, "Kc": ep.Kc, "Vc": ep.Vc}
    O, lse = _decode(s, s["Kc"], s["Vc"], s["counts"], s["offsets"])
    return {"O": O, "lse": lse}


# ---------------------------------------------------------------------------

def _rows(case):
    """(all key rows, kept rows) over every layer and head."""
    LH = case["layers"] * case["kv_heads"]
    kept = 0
    if case.get("mode") == "heads":
        kept = sum(min(b, t) for b in _budget(case) for t in _lens(case))
    elif "mode" in case:
        kept = LH * sum(min(b, t) for b, t in zip(_budget(case), _lens(case)))
    return LH * sum(_lens(case)), kept


def work(case):
    rows, kept = _rows(case)
    D, B, L, H, w = case["dim"], len(_lens(case)), case["layers"], case["kv_heads"], case["window"]
    row = D * (2 if case["dtype"] == "bf16" else 4)
    R = case["q_heads"] // H * w
    queries = L * case["q_heads"] * B * row
    scores = 4 * (rows - L * H * B * w)
    per_key = 2 * R * D + 8 * D  # window logits, then distance, norm, cosine and the key sums
    if case["kind"] == "evict":  # K once, the kept V rows; the kept rows of both and their positions written
        return {"bytes": rows * row + 3 * kept * row + 4 * kept + scores + queries * (w + 1),
                "flops": rows * per_key + 4 * kept * R // w * D}
    if case["kind"] == "score":
        return {"bytes": rows * row * (2 if case["vnorm"] else 1) + scores + queries * w, "flops": rows * per_key}
    if case["kind"] == "write":  # the new rows of both, read and written
        return {"bytes": 4 * rows * row + scores + queries * w, "flops": rows * (per_key + 2 * R * D)}
    if case["kind"] == "keep":
        return {"bytes": scores + 4 * kept + 4 * kept * row, "flops": 0}
    return {"bytes": 2 * kept * row + 2 * queries, "flops": 4 * kept * R // w * D}


def tolerance(case):
    if case["kind"] == "keep":
        return "exact"
    if case["kind"] == "evict":
        # two keys whose scores agree within rounding may change places in the selection
        return {"rel": 2e-3, "max": 0.2}
    return {"rel": 1e-5, "max": 1e-4}


# ---------------------------------------------------------------------------

def _score64(K, V, Q, w, G, par, case):
    """Scores, lambda and statistics of one head's keys K [T][D], window queries Q [R][D], in 64 bits."""
    T, D = K.shape
    N = T - w
    K, Q = K.double(), Q.double()
    x = Q @ K.t() / math.sqrt(D)
    j = torch.arange(Q.shape[0], device=K.device) % w
    x.masked_fill_(torch.arange(T, device=K.device)[None, :] > (N + j)[:, None], -math.inf)
    a = torch.softmax(x, dim=1).mean(dim=0)[:N]
    del x
    half = par.pool_kernel // 2
    imp = torch.nn.functional.avg_pool1d(a[None, None], par.pool_kernel, 1, half)[0, 0]
    if case.get("vnorm"):
        imp = imp * V[:N].double().norm(dim=1)
    kbar = (K[:N] if case.get("prefix") else K).mean(dim=0)
    khat = K / K.norm(dim=1, keepdim=True).clamp_min(1e-12)
    mu = khat.mean(dim=0)
    d = (K - kbar).norm(dim=1)
    c = khat[:N] @ mu
    eps, tau, f32 = float(par.eps), math.sqrt(D), lambda v: float(torch.tensor(v, dtype=torch.float32))
    alpha, beta = f32(par.alpha), f32(par.beta)
    DE, dN = d.mean(), d[:N]
    if case.get("std"):
        rE = 1 - torch.sigmoid(d.square().mean().sqrt() / tau)
    else:
        rE = 2 - 2 * torch.sigmoid(DE / tau)
    mu2 = mu.square().sum()
    rC = (T * mu2 - 1) / (T - 1)
    lam = beta * rE + (1 - beta) * rC

    def quantile(v, q):
        v = v.sort().values
        h = q * (v.numel() - 1)
        lo = int(math.floor(h))
        hi = min(lo + 1, v.numel() - 1)
        return v[lo] + (h - lo) * (v[hi] - v[lo])

    norm = case.get("norm", "minmax")
    if norm == "minmax":
        sE = (dN - dN.min()) / (dN.max() - dN.min() + eps)
    elif norm == "winsor":
        q = float(par.winsor_q)
        lo, hi = quantile(dN, q), quantile(dN, 1 - q)
        sE = (dN.clamp(lo, hi) - lo) / (hi - lo + eps)
    else:
        med = quantile(dN, 0.5)
        sE = torch.sigmoid((dN - med) / (float(par.mad_tau) * quantile((dN - med).abs(), 0.5) + eps))
    sdiv = alpha * sE + (1 - alpha) * (1 - c) / 2
    sbar = (sdiv - sdiv.min()) / (sdiv.max() - sdiv.min() + eps)
    scale = imp.mean() / (sbar.mean() + eps)
    S = lam * sbar * scale + (1 - lam) * imp
    st = torch.stack([lam, rC, rE, DE, dN.min(), dN.max(), sdiv.min(), sdiv.max(), imp.mean(), sbar.mean(), mu2, scale])
    return S, st


def exact(case, seed):
    if case["kind"] == "keep":
        return None
    L, H, w, D = case["layers"], case["kv_heads"], case["window"], case["dim"]
    G, lens = case["q_heads"] // H, _lens(case)
    s = prepare(case, seed)
    if case["kind"] == "decode":
        O, lse = s["O"].double(), s["lse"].double()
        for l in range(L):
            for h in range(H):
                for b in range(len(lens)):
                    n, o = int(s["counts"][l, h, b]), int(s["offsets"][l, h, b])
                    q = s["Qd"][l, h * G:(h + 1) * G, b, 0].double()
                    x = q @ s["Kc"][o:o + n].double().t() / math.sqrt(D)
                    O[l, h * G:(h + 1) * G, b] = torch.softmax(x, dim=1) @ s["Vc"][o:o + n].double()
                    lse[l, h * G:(h + 1) * G, b] = torch.logsumexp(x, dim=1)
        return {"O": O, "lse": lse}
    if case["kind"] == "write":  # the cache layout, from the new rows
        for n in ("K", "V"):
            s[n].copy_(s[n + "new"].transpose(1, 2))
    scores = torch.empty(L, H, sum(lens) - w * len(lens), dtype=torch.float64, device="cuda")
    stats = torch.empty(L, H, len(lens), P.NSTATS, dtype=torch.float64, device="cuda")
    for l in range(L):
        for h in range(H):
            at = 0
            for b, T in enumerate(lens):
                q = s["Q"][l, h * G:(h + 1) * G, b].reshape(G * w, D)
                v = s["V"][l, h, at:at + T] if s["V"] is not None else None
                S, stats[l, h, b] = _score64(s["K"][l, h, at:at + T], v, q, w, G, s["params"], case)
                scores[l, h, at - b * w:at - b * w + T - w] = S
                at += T
    out = {"scores": scores.view(-1), "lambda": stats[..., 0].reshape(-1), "stats": stats.view(-1, P.NSTATS)}
    if case["kind"] == "write":
        out.update(K=s["K"].double(), V=s["V"].double())
    return {**out, "O": None, "lse": None} if case["kind"] == "evict" else out
