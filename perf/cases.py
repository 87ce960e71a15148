"""The work that a program has this library do, as timed cases.

A prefill hands its K/V cache to `evict`, layer by layer or a whole stack of layers at once, and then decodes on the
compacted cache; tuning and evaluation programs call the stages (`score`, `smooth`, `select`, `compact`) by
themselves. Every case is one call, or the two calls of a prefill's last layer and its first decoding step, through
the package's public functions with the buffers that such a program keeps (workspace, outputs, prefix sums).

A case is a dict of plain values:
  do                      evict (one layer) | serve (evict, then one decoding step) | score | smooth | select | compact | decode
  items, shortest, longest, lengths_seed   sequences or layers, and their lengths (equal, or spread over the range)
  q_heads, kv_heads, dim, window           attention geometry
  layout                  head ([H][L][d] per item) or token ([L][H][d])
  ratio, cutoff, mode     kept share of the tokens; cutoff of the smoothing and its mode (fraction | energy)
  scope                   global (one budget pool) or item
  lse                     whether the prefill kernel's log-sum-exp of the window rows is at hand
"""
import math
import random

import numpy as np
import torch

import paper_2604_06694_amd as A

FLOOR_FRAC, POOL, ALPHA = 0.1, 7, 1.0
ENERGY = 0.9          # share of the spectral energy (DC bin apart) that the energy-adaptive cutoff keeps

# query heads, KV heads, head_dim, window: the geometries of the synthetic workloads and of the tests' shapes
GEOMETRIES = [(28, 4, 128, 32), (28, 4, 128, 64), (32, 4, 128, 32), (8, 2, 256, 32), (8, 2, 64, 16), (32, 4, 128, 16)]


def _case(name, do, geometry, items, shortest, longest=None, **more):
    q_heads, kv_heads, dim, window = geometry
    case = {"name": name, "do": do, "items": items, "shortest": shortest, "longest": longest or shortest,
            "lengths_seed": 0, "q_heads": q_heads, "kv_heads": kv_heads, "dim": dim, "window": window,
            "layout": "head", "ratio": 0.4, "cutoff": 0.125, "mode": "fraction", "scope": "global", "lse": False}
    case.update(more)
    return case


def listed():
    return [
        # one layer of a short clip: the smallest call
        _case("evict_1x2048", "evict", (28, 4, 128, 32), 1, 2048),
        # layer-wise eviction during the prefill of long audio, wide window
        _case("evict_1x32768_w64", "evict", (28, 4, 128, 64), 1, 32768),
        # the same for a prompt as long as it happens to be (lengths of real prompts are no powers of two)
        _case("evict_1x13577", "evict", (32, 4, 128, 32), 1, 13577),
        # all layers of a 7B model at once, then the first decoding step
        _case("serve_28x8192", "serve", (28, 4, 128, 32), 28, 8192),
        # all layers, long audio, wide window: the largest call
        _case("serve_28x32768_w64", "serve", (28, 4, 128, 64), 28, 32768),
        # a serving batch of eight requests of different lengths, budgets per request, wide heads
        _case("serve_8xragged_d256", "serve", (8, 2, 256, 32), 8, 2048, 32768, lengths_seed=3, ratio=0.3, scope="item"),
        # scoring alone, all layers of a 30B model, keys in the [L][H][d] order in which a projection leaves them
        _case("score_48x16384_token", "score", (32, 4, 128, 32), 48, 16384, layout="token"),
        # smoothing alone: sequences of a sweep over the cutoff, ragged
        _case("smooth_24xragged", "smooth", (8, 2, 128, 32), 24, 1500, 30000, lengths_seed=5),
        # the energy-adaptive cutoff, one layer
        _case("smooth_energy_1x8192", "smooth", (28, 4, 128, 32), 1, 8192, mode="energy"),
        # top-k alone, all layers
        _case("select_28x16384", "select", (28, 4, 128, 32), 28, 16384),
        # the gather alone: an eviction policy of the program's own, ragged batch
        _case("compact_8xragged", "compact", (28, 4, 128, 32), 8, 2000, 20000, lengths_seed=7, scope="item"),
        # a decoding step of one layer over a batch of 16 short compacted caches
        _case("decode_16x4096", "decode", (28, 4, 128, 32), 16, 4096),
    ]


def _lengths(case):
    lo, hi, n = case["shortest"], case["longest"], case["items"]
    if lo == hi:
        return [lo] * n
    r = random.Random(case["lengths_seed"])
    return [int(math.exp(r.uniform(math.log(lo), math.log(hi)))) for _ in range(n)]


def _spread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["evict", "evict", "serve", "serve", "score", "smooth", "select", "compact", "decode"])
    geometry = rng.choice(GEOMETRIES)
    q_heads, kv_heads, dim, window = geometry
    length = _spread(rng, 400, 32768)
    if rng.random() < 0.25:
        length = 1 << int(round(math.log2(length)))
    # items: from one layer to as many as stay well below the largest listed case
    room = 28 * 32768 * 28 * 64 * 128 / 2
    cap = min(48, int(room / (length * q_heads * window * dim)), int(300e6 / (length * kv_heads * dim)))
    items = 1 if do == "evict" else max(1, _spread(rng, 2, max(2, cap)))
    ragged = items > 1 and rng.random() < 0.4
    shortest = max(400, length // rng.choice([2, 4, 16])) if ragged else length
    if shortest >= length:
        ragged, shortest = False, length
    mode = "energy" if do == "smooth" and rng.random() < 0.25 else "fraction"
    case = _case("", do, geometry, items, shortest, length, lengths_seed=rng.randrange(1 << 20),
                 layout=rng.choice(["head", "head", "token"]), ratio=round(rng.uniform(0.15, 0.8), 3),
                 cutoff=rng.choice([0.0625, 0.125, 0.25]), mode=mode,
                 scope="item" if ragged else rng.choice(["global", "item"]),
                 lse=do in ("evict", "serve", "score") and rng.random() < 0.25)
    del case["name"]
    return case


# ---- inputs --------------------------------------------------------------------------------------------------------

def _gen(seed, part):
    return torch.Generator(device="cuda").manual_seed(seed * 16 + part)


def _continuous(x, rho):
    """First-order autoregression along dim 1 of white noise x [heads, L, ...]: acoustic frames change slowly."""
    step, decay = 1, rho
    while step < x.shape[1] and decay > 1e-3:
        head = x[:, :step]
        x = torch.cat([head, x[:, step:] + decay * x[:, :-step]], dim=1)
        step, decay = 2 * step, decay * decay
    return x


def _rows(case, lens, gen, keys):
    """Packed bf16 rows of all items: slowly varying with a few spikes for keys, white noise for values."""
    heads, dim = case["kv_heads"], case["dim"]
    out = torch.empty(sum(lens) * heads * dim, dtype=torch.bfloat16, device="cuda")
    at = 0
    for L in lens:
        x = torch.randn((heads, L, dim), generator=gen, device="cuda")
        if keys:
            x = _continuous(x, 0.95)
            spikes = torch.randint(0, max(1, L - case["window"]), (16,), generator=gen, device="cuda")
            x[:, spikes] *= 2.0
        if case["layout"] == "token":
            x = x.transpose(0, 1)
        n = heads * L * dim
        out[at:at + n] = x.reshape(-1).to(torch.bfloat16)
        at += n
    return out


def _sequences(case, lens, gen, smoothed):
    """Packed fp32 score sequences: positive, slowly varying, heavy upper tail; smoothed ones are averaged as well."""
    parts = []
    for L in lens:
        x = _continuous(torch.randn((case["kv_heads"], L), generator=gen, device="cuda"), 0.9) / 2.3
        x = torch.exp(1.2 * x) * (case["q_heads"] // case["kv_heads"] * case["window"] / (2.0 * L))
        if smoothed:
            x = torch.nn.functional.avg_pool1d(x[None], 15, 1, 7)[0]
        parts.append(x.reshape(-1))
    return torch.cat(parts).contiguous()


def _params(case):
    return A.Params(case["q_heads"], case["kv_heads"], case["dim"], case["window"], pool_kernel=POOL,
                    floor_frac=FLOOR_FRAC, kv_layout=A.LAYOUT_TOKEN_MAJOR if case["layout"] == "token" else A.LAYOUT_HEAD_MAJOR,
                    cutoff_mode=A.CUTOFF_ENERGY_NO_DC if case["mode"] == "energy" else A.CUTOFF_FRACTION)


def _cutoff(case):
    return ENERGY if case["mode"] == "energy" else case["cutoff"]


def _item(s, flat, i):
    """Item i of a packed K or V buffer as [H][L][d]."""
    c, lens = s["case"], s["lens"]
    a, n = sum(lens[:i]) * c["kv_heads"] * c["dim"], lens[i] * c["kv_heads"] * c["dim"]
    x = flat[a:a + n]
    if c["layout"] == "token":
        return x.view(lens[i], c["kv_heads"], c["dim"]).transpose(0, 1)
    return x.view(c["kv_heads"], lens[i], c["dim"])


def _logits(s, i, h, dtype):
    """Scaled window logits of head h of item i, invisible keys at -inf: [G * W, L]."""
    c, L = s["case"], s["lens"][i]
    g, W, d = c["q_heads"] // c["kv_heads"], c["window"], c["dim"]
    q = s["q"].view(c["items"], c["q_heads"], W, d)[i, h * g:(h + 1) * g].reshape(g * W, d).to(dtype)
    z = q @ _item(s, s["k"], i)[h].to(dtype).t().contiguous() / math.sqrt(d)
    last = (L - W + torch.arange(W, device="cuda")).repeat(g)
    return z.masked_fill(torch.arange(L, device="cuda")[None] > last[:, None], -math.inf)


def prepare(case, seed):
    lens, p, do = _lengths(case), _params(case), case["do"]
    n, heads, dim = case["items"], case["items"] * case["kv_heads"], case["dim"]
    s = {"case": case, "p": p, "lens": lens}
    s["cu"] = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device="cuda")
    if do != "decode":
        s["ws"] = torch.empty(max(256, A.workspace_bytes(p, lens)), dtype=torch.uint8, device="cuda")
    if do in ("evict", "serve", "select", "compact", "decode"):
        # criticality of the heads: exponential draws, which normalised are a Dirichlet(1)
        w = torch.empty(heads, device="cuda").exponential_(generator=_gen(seed, 0))
        s["w"] = w / w.sum()
        s["rows"] = A.total_kept(p, lens, case["ratio"])
    if do in ("evict", "serve", "score", "compact"):
        s["k"] = _rows(case, lens, _gen(seed, 1), True)
    if do in ("evict", "serve", "compact"):
        s["v"] = _rows(case, lens, _gen(seed, 2), False)
    if do in ("evict", "serve", "score"):
        s["q"] = torch.randn(n * case["q_heads"] * case["window"] * dim, generator=_gen(seed, 3), device="cuda").to(torch.bfloat16)
        if case["lse"]:
            s["lse"] = torch.stack([torch.logsumexp(_logits(s, i, h, torch.float32), dim=1)
                                    for i in range(n) for h in range(case["kv_heads"])]).reshape(-1).contiguous()
    if do in ("evict", "serve"):
        s["outs"] = {"k_out": torch.empty((s["rows"], dim), dtype=torch.bfloat16, device="cuda"),
                     "v_out": torch.empty((s["rows"], dim), dtype=torch.bfloat16, device="cuda"),
                     "indices": torch.empty(s["rows"], dtype=torch.int32, device="cuda"),
                     "budgets": torch.empty(heads, dtype=torch.int32, device="cuda"),
                     "cu_budgets": torch.empty(heads + 1, dtype=torch.int32, device="cuda")}
    if do in ("score", "smooth", "select"):
        if do != "score":
            s["scores"] = _sequences(case, lens, _gen(seed, 4), do == "select")
        s["out"] = torch.empty(sum(lens) * case["kv_heads"], device="cuda")
    if do in ("select", "compact", "decode"):
        if case["scope"] == "global":
            s["budgets"], s["cu_b"] = A.allocate(p, s["w"], 1, heads, lens[:1], case["ratio"])
        else:
            s["budgets"], s["cu_b"] = A.allocate(p, s["w"], n, case["kv_heads"], lens, case["ratio"], cu_seqlens=s["cu"])
    if do == "compact":
        # what the gather gets from a selection: clusters of neighbouring tokens, ascending
        scores = _sequences(case, lens, _gen(seed, 4), True)
        s["indices"] = A.select(p, scores, s["budgets"], s["cu_b"], lens, s["rows"], cu_seqlens=s["cu"])
    if do == "decode":
        one = dict(case, kv_heads=1, layout="head")
        s["outs"] = {"k_out": _rows(one, [s["rows"]], _gen(seed, 1), True), "v_out": _rows(one, [s["rows"]], _gen(seed, 2), False)}
    if do in ("serve", "decode"):
        s["q1"] = torch.randn(n * case["q_heads"] * dim, generator=_gen(seed, 5), device="cuda").to(torch.bfloat16)
        s["attended"] = torch.empty((n, case["q_heads"], dim), device="cuda")
        s["ws1"] = torch.empty(max(256, A.decode_workspace_bytes(p, n, s["rows"])), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    c, p, lens = s["case"], s["p"], s["lens"]
    do = c["do"]
    if do in ("evict", "serve"):
        o = A.evict(p, s["q"], s["k"], s["v"], s["w"], lens, c["ratio"], c["cutoff"], ALPHA,
                    alloc_scope=A.SCOPE_GLOBAL if c["scope"] == "global" else A.SCOPE_ITEM, cu_seqlens=s["cu"],
                    workspace=s["ws"], outputs=s["outs"], lse=s.get("lse"))
        if do == "evict":
            return {name: o[name] for name in ("k_out", "v_out", "indices", "budgets", "cu_budgets")}
        # Over the hundreds of heads of a stack, two tokens whose scores agree to the last bits of fp32 may now and then
        # change places at the threshold, which moves every row between them by one: what the program goes on with
        # is attention over the rows, which does not depend on their order and shows a wrong row or a lost one.
        out = A.decode_attend(p, s["q1"], o["k_out"], o["v_out"], o["cu_budgets"], c["items"], s["rows"],
                              out=s["attended"], workspace=s["ws1"])
        return {"attended": out, "budgets": o["budgets"], "cu_budgets": o["cu_budgets"]}
    if do == "score":
        return {"scores": A.score(p, s["q"], s["k"], lens, cu_seqlens=s["cu"], out=s["out"], workspace=s["ws"], lse=s.get("lse"))}
    if do == "smooth":
        return {"smoothed": A.smooth(p, s["scores"], lens, _cutoff(c), ALPHA, cu_seqlens=s["cu"], out=s["out"], workspace=s["ws"])}
    if do == "select":
        return {"indices": A.select(p, s["scores"], s["budgets"], s["cu_b"], lens, s["rows"], cu_seqlens=s["cu"])}
    if do == "compact":
        k, v = A.compact(p, s["k"], s["v"], s["indices"], s["cu_b"], lens, s["rows"], cu_seqlens=s["cu"])
        return {"k": k, "v": v}
    return {"attended": A.decode_attend(p, s["q1"], s["outs"]["k_out"], s["outs"]["v_out"], s["cu_b"], c["items"], s["rows"],
                                        out=s["attended"], workspace=s["ws1"])}


# ---- what a pass cannot do without, and how exact it is ------------------------------------------------------------

def work(case):
    lens, do = _lengths(case), case["do"]
    row = case["dim"] * 2
    keys = sum(lens) * case["kv_heads"]
    kept = sum(A.n_keep(case["ratio"], L) for L in lens) * case["kv_heads"]
    gather, step = 4 * kept * row + 4 * kept, 2 * kept * row
    rows = case["q_heads"] * case["window"]
    q = case["items"] * rows * row
    # two multiply-adds' worth per (window row, key, channel), once; a decoding step: logits and weighted sum
    window = 2.0 * rows * sum(lens) * case["dim"]
    decode = 4.0 * kept * case["dim"] * (case["q_heads"] // case["kv_heads"])
    # a real transform forward and back: 2.5 n log2 n each
    smooth = sum(5.0 * L * math.log2(L) for L in lens) * case["kv_heads"]
    return {"evict": {"bytes": q + keys * row + gather, "flops": window + smooth},
            "serve": {"bytes": q + keys * row + gather + step, "flops": window + smooth + decode},
            "score": {"bytes": q + keys * row + 4 * keys, "flops": window},
            "smooth": {"bytes": 8 * keys, "flops": smooth},
            "select": {"bytes": 4 * keys + 4 * kept, "flops": keys},
            "compact": {"bytes": gather, "flops": 0},
            "decode": {"bytes": step, "flops": decode}}[do]


def tolerance(case):
    if case["do"] in ("evict", "select", "compact"):
        # indices are whole numbers and rows are copied; the selections of 700 heads of the listed cases were those
        # that scores in 64 bits give, so for the few heads of one layer nothing need be allowed
        return "exact"
    if case["do"] == "serve":
        # 5e-7 from attention over rows selected in 64 bits; room for one token that ties with the threshold to fp32
        # rounding and is replaced by the one it ties with (a share of about 1 / sqrt(rows kept) of one head's output)
        return {"rel": 5e-3, "max": 0.2, "differ": 0.0}
    if case["do"] == "smooth" and case["mode"] == "energy":
        # fp32 transforms; the cutoff is a whole number of bins that rounding can move by one
        return {"rel": 1e-3, "max": 1e-2}
    if case["do"] == "smooth":
        return {"rel": 5e-6, "max": 1e-4}
    # fp32 accumulation and exponentials of logits up to about a hundred: 4e-7 to 7e-7 seen
    return {"rel": 5e-6, "max": 1e-4}


# ---- the same in 64 bits, without the package's kernels --------------------------------------------------------------

def _exact_scores(s):
    c, parts = s["case"], []
    for i, L in enumerate(s["lens"]):
        for h in range(c["kv_heads"]):
            raw = torch.softmax(_logits(s, i, h, torch.float64), dim=1).sum(dim=0)
            sums = torch.nn.functional.pad(raw, (POOL // 2 + 1, POOL // 2)).cumsum(0)
            parts.append((sums[POOL:] - sums[:L]) / POOL)
    return torch.cat(parts)


def _exact_smoothed(s):
    c, x, parts, at = s["case"], s["scores"].cpu().numpy().astype(np.float64), [], 0
    for L in s["lens"]:
        f = np.fft.rfft(x[at:at + c["kv_heads"] * L].reshape(c["kv_heads"], L), axis=1)
        at += c["kv_heads"] * L
        if c["mode"] == "energy":
            e = np.cumsum(np.abs(f[:, 1:]) ** 2, axis=1)
            top = 1 + np.argmax(e >= ENERGY * e[:, -1:], axis=1)
        else:
            top = np.full(c["kv_heads"], math.floor(c["cutoff"] * (L // 2)))
        f[np.arange(f.shape[1])[None] > top[:, None]] = 0
        parts.append(np.fft.irfft(f, n=L, axis=1).reshape(-1))
    return np.concatenate(parts)


def _exact_attended(s):
    c, cu = s["case"], s["cu_b"].cpu().tolist()
    g, d = c["q_heads"] // c["kv_heads"], c["dim"]
    k, v = (s["outs"][x].view(-1, d) for x in ("k_out", "v_out"))
    q = s["q1"].view(-1, g, d)
    out = torch.empty((c["items"] * c["kv_heads"], g, d), dtype=torch.float64, device="cuda")
    for i in range(len(cu) - 1):
        z = q[i].double() @ k[cu[i]:cu[i + 1]].double().t().contiguous() / math.sqrt(d)
        out[i] = torch.softmax(z, dim=1) @ v[cu[i]:cu[i + 1]].double()
    return out.view(c["items"], c["q_heads"], d)


def exact(case, seed):
    do = case["do"]
    if do in ("evict", "serve", "select"):
        # whole numbers, and rows chosen by them: a choice among equals has no value to be near to
        return None
    s = prepare(case, seed)
    if do == "score":
        return {"scores": _exact_scores(s)}
    if do == "smooth":
        return {"smoothed": _exact_smoothed(s)}
    if do == "decode":
        return {"attended": _exact_attended(s)}
    counts, cu = s["budgets"].cpu().tolist(), s["cu_b"].cpu().tolist()
    got = {}
    for name in ("k", "v"):
        got[name] = torch.cat([_item(s, s[name], n // case["kv_heads"])[n % case["kv_heads"]][s["indices"][cu[n]:cu[n] + b].long()]
                               for n, b in enumerate(counts)])
    return got
