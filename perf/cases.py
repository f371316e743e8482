"""Performance cases: the calls an act-first rollout and its OPD update make.

Each case is one call (or one captured decode step) through the package's
public entry points: the decode step over contiguous and paged caches, the
causal prefill of appended tokens, and the OPD token loss with and without the
logits gradient.  `listed()` holds twelve fixed ones, `draw()` gives others of
the same ranges.  Context lengths come from a case's own `lens_seed`; queries,
keys, values, logits and placements come from the seed given to `prepare`.
"""
import math
import random

import torch

HEAD_DIM = 128
SCALE = 1.0 / math.sqrt(HEAD_DIM)
LOG_CLIP, DELTA, KAPPA, EPS = 20.0, 0.2, 3.0, 1e-8  # the OPD loss's default constants
PEAKY_FRAC, PEAKY_GAIN = 0.05, 4.0


def listed():
    return [
        # one decode step of a small student with a few short contexts in flight (early turns, the end
        # of a batch): 28 layers in a HIP graph, bound by launches and latency
        dict(name="decode_step_graph", path="decode", layers=28, hq=16, hkv=8, batch=4, lo=256, hi=1024,
             dist="uniform", page=0, out="f32", peaky=False, lens_seed=1),
        # the last request of a batch still decoding, on a long context: one sequence over the whole chip
        dict(name="decode_single_long", path="decode", layers=1, hq=32, hkv=8, batch=1, lo=30001, hi=30001,
             dist="uniform", page=0, out="f32", peaky=False, lens_seed=2),
        # 0.6B / 1.7B student, early-turn contexts
        dict(name="decode_student_1p7b", path="decode", layers=1, hq=16, hkv=8, batch=64, lo=1024, hi=4096,
             dist="uniform", page=0, out="f32", peaky=False, lens_seed=3),
        # long-horizon ragged batch, the headline workload
        dict(name="decode_long_ragged", path="decode", layers=1, hq=32, hkv=8, batch=32, lo=512, hi=32768,
             dist="log", page=0, out="f32", peaky=False, lens_seed=4),
        # act-first short-action burst: the largest batch, peaky keys, 16-bit outputs
        dict(name="decode_burst", path="decode", layers=1, hq=32, hkv=8, batch=256, lo=4224, hi=12800,
             dist="uniform", page=0, out="bf16", peaky=True, lens_seed=5),
        # 4B student on a serving engine's 16-token pages, the new token appended by the call
        dict(name="decode_paged_append", path="decode", layers=1, hq=32, hkv=8, batch=64, lo=2048, hi=8192,
             dist="uniform", page=16, out="bf16", peaky=False, lens_seed=6),
        # one request takes in its reference observation (continuous batching admits one at a time)
        dict(name="prefill_single", path="prefill", hq=32, hkv=8, batch=1, hist_lo=8000, hist_hi=8000, new_lo=301,
             new_hi=301, split_p=False, out="bf16", peaky=True, lens_seed=7),
        # a batch of fresh prompts of mixed lengths, 0.6B / 1.7B student, two-term softmax weights
        dict(name="prefill_prompts", path="prefill", hq=16, hkv=8, batch=12, hist_lo=0, hist_hi=0, new_lo=200,
             new_hi=2000, split_p=True, out="f32", peaky=False, lens_seed=8),
        # the reference observations of a whole act-first burst
        dict(name="prefill_burst", path="prefill", hq=32, hkv=8, batch=256, hist_lo=4096, hist_hi=12288, new_lo=128,
             new_hi=512, split_p=False, out="f32", peaky=True, lens_seed=9),
        # a small update: a few short responses, a small odd vocabulary in padded rows
        dict(name="opd_small", path="opd", responses=6, lo=0, hi=48, vocab=1003, pad=5, grad=True, lens_seed=10),
        # the loss alone (no gradient) of some responses, the Qwen3 vocabulary
        dict(name="opd_loss_only", path="opd", responses=16, lo=64, hi=512, vocab=151936, pad=0, grad=False,
             lens_seed=11),
        # a full optimization batch: loss and logits gradient of 64 responses
        dict(name="opd_batch", path="opd", responses=64, lo=64, hi=512, vocab=151936, pad=0, grad=True, lens_seed=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "opd", "opd"])
    case = _draw_one(rng, kind)
    while _cost(case) > 1.0:
        case = _draw_one(rng, kind)
    return case


def _cost(case):
    """Work relative to the largest listed case of the path."""
    w = work(case)
    if case["path"] == "prefill":
        return w["flops"] * (1.5 if case["split_p"] else 1.0) / 9.0e12
    return w["bytes"] / {"decode": 9.0e9, "opd": 10.0e9}[case["path"]]


def _draw_one(rng, kind):
    lens_seed = rng.randrange(1 << 30)
    if kind == "decode":
        hq, hkv = rng.choice([(16, 8), (32, 8), (32, 8), (64, 8), (16, 16), (28, 4), (32, 4), (12, 2), (16, 1)])
        lo = _log_int(rng, 64, 16384)
        hi = min(32768, int(lo * rng.uniform(1.0, 16.0)))
        graph = rng.random() < 0.2
        return dict(path="decode", layers=rng.randrange(4, 13) if graph else 1, hq=hq, hkv=hkv,
                    batch=_log_int(rng, 1, 16 if graph else 256), lo=min(lo, 2048) if graph else lo,
                    hi=max(min(lo, 2048), min(hi, 4096)) if graph else hi, dist=rng.choice(["uniform", "log"]),
                    page=rng.choice([0, 0, 16, 32, 64]), out=rng.choice(["f32", "bf16"]), peaky=rng.random() < 0.3,
                    lens_seed=lens_seed)
    if kind == "prefill":
        hq, hkv = rng.choice([(16, 8), (32, 8), (32, 8), (64, 8), (16, 16), (28, 4), (12, 2)])
        hist_lo = 0 if rng.random() < 0.3 else _log_int(rng, 128, 12288)
        new_lo = _log_int(rng, 16, 1024)
        return dict(path="prefill", hq=hq, hkv=hkv, batch=_log_int(rng, 1, 256), hist_lo=hist_lo,
                    hist_hi=int(hist_lo * rng.uniform(1.0, 2.0)), new_lo=new_lo,
                    new_hi=int(new_lo * rng.uniform(1.0, 4.0)), split_p=rng.random() < 0.3,
                    out=rng.choice(["f32", "bf16"]), peaky=rng.random() < 0.3, lens_seed=lens_seed)
    vocab = rng.choice([151936, 151936, 65536, 50257, 32000, _log_int(rng, 1000, 155000)])
    lo = _log_int(rng, 8, 256)
    return dict(path="opd", responses=_log_int(rng, 2, 64), lo=lo, hi=min(512, int(lo * rng.uniform(1.0, 8.0))),
                vocab=vocab, pad=rng.choice([0, 0, 64]) + -vocab % 8, grad=rng.random() < 0.7, lens_seed=lens_seed)


# ------------------------------------------------------------------ shapes of a case (no seed)

def _lengths(case):
    """Cached tokens (and, for a prefill, new tokens) of every sequence, or tokens of every response."""
    rng = random.Random(case["lens_seed"])
    if case["path"] == "decode":
        if case["dist"] == "log":
            a, b = math.log(case["lo"]), math.log(case["hi"])
            return [max(case["lo"], min(case["hi"], int(math.exp(rng.uniform(a, b))))) for _ in range(case["batch"])]
        return [rng.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]
    if case["path"] == "prefill":
        hist = [rng.randint(case["hist_lo"], case["hist_hi"]) for _ in range(case["batch"])]
        new = [rng.randint(case["new_lo"], case["new_hi"]) for _ in range(case["batch"])]
        return [h + n for h, n in zip(hist, new)], new
    return [rng.randint(case["lo"], case["hi"]) for _ in range(case["responses"])]


def _inserted(case):
    """(start, length) of every response's unsupervised span; about half of the responses have one of 8 tokens."""
    rng = random.Random(case["lens_seed"] + 1)
    spans = []
    for n in _lengths(case):
        if n > 8 and rng.random() < 0.5:
            spans.append((rng.randint(0, n - 8), 8))
        else:
            spans.append((0, 0))
    return spans


def work(case):
    if case["path"] == "decode":
        tokens, layers = sum(_lengths(case)), case["layers"]
        out = 4 if case["out"] == "f32" else 2
        per_layer = tokens * case["hkv"] * HEAD_DIM * 2 * 2 + case["batch"] * (case["hq"] * HEAD_DIM * (2 + out) + 8)
        if case["page"]:
            per_layer += case["batch"] * case["hkv"] * HEAD_DIM * 2 * 2 * 2 + tokens // case["page"] * 4
        return {"bytes": layers * per_layer, "flops": layers * tokens * 4 * HEAD_DIM * case["hq"]}
    if case["path"] == "prefill":
        lens, new = _lengths(case)
        positions = sum(n * (length - n) + n * (n + 1) // 2 for length, n in zip(lens, new))
        out = 4 if case["out"] == "f32" else 2
        return {"bytes": sum(lens) * case["hkv"] * HEAD_DIM * 2 * 2 + sum(new) * case["hq"] * HEAD_DIM * (2 + out),
                "flops": positions * 4 * HEAD_DIM * case["hq"]}
    rows = sum(_lengths(case))
    live = rows - sum(n for _, n in _inserted(case))
    return {"bytes": live * case["vocab"] * 2 + (rows * case["vocab"] * 2 if case["grad"] else 0) + rows * 25,
            "flops": live * case["vocab"] * 4}


def tolerance(case):
    # About four times the errors against 64 bits seen on an MI355X: fp32 decode 2.5e-6, two-term prefill 3.9e-6,
    # 16-bit outputs and gradients 1.7e-3, 16-bit softmax weights 2.3e-3, fp32 OPD values 1.3e-6 (2e-5 stated: the
    # batch loss sums terms of both signs).
    if case["path"] == "decode":
        return {"rel": 1e-5, "max": 2e-4} if case["out"] == "f32" else {"rel": 7e-3, "max": 3e-2}
    if case["path"] == "prefill":
        if case["split_p"] and case["out"] == "f32":
            return {"rel": 1.6e-5, "max": 1e-3}
        return {"rel": 1e-2, "max": 8e-2}
    return {"rel": 7e-3, "max": 3e-2} if case["grad"] else {"rel": 2e-5, "max": 1e-4}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _i32(values):
    return torch.tensor(values, dtype=torch.int32, device="cuda")


def _normal(g, shape, std=1.0):
    """bf16 N(0, std^2)."""
    t = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    flat = t.view(-1)
    for s in range(0, flat.numel(), 1 << 28):
        flat[s:s + (1 << 28)].normal_(0.0, std, generator=g)
    return t


def _cache(g, case, rows):
    k = _normal(g, (rows, case["hkv"], HEAD_DIM))
    v = _normal(g, (rows, case["hkv"], HEAD_DIM))
    if case["peaky"]:
        gain = torch.ones(rows, dtype=torch.bfloat16, device="cuda")
        gain.masked_fill_(torch.rand(rows, generator=g, device="cuda") < PEAKY_FRAC, PEAKY_GAIN)
        k.mul_(gain[:, None, None])
    return k, v


def _offsets(rng, lens, reserve):
    """First rows of regions of len + reserve rows, placed in a shuffled order; and the total."""
    order = list(range(len(lens)))
    rng.shuffle(order)
    offs, row = [0] * len(lens), 0
    for b in order:
        offs[b] = row
        row += lens[b] + reserve
    return offs, row


def _decode_inputs(case, seed):
    rng, g = random.Random(seed), _gen(seed)
    lens, batch = _lengths(case), case["batch"]
    s = {"case": case, "lens": _i32(lens)}
    if case["page"]:
        pages = [-(-n // case["page"]) for n in lens]
        perm = list(range(sum(pages) + 8))
        rng.shuffle(perm)
        table, at = [], 0
        for n in pages:
            table.append(perm[at:at + n] + [0] * (max(pages) - n))
            at += n
        s["table"] = _i32(table)
        rows = len(perm) * case["page"]
    else:
        offs, rows = _offsets(rng, lens, 8)
        s["offs"] = _i32(offs)
    for name in ("q", "k", "v", "k_new", "v_new"):
        s[name] = []
    for _ in range(case["layers"]):
        s["q"].append(_normal(g, (batch, case["hq"], HEAD_DIM)))
        k, v = _cache(g, case, rows)
        if case["page"]:
            shape = (-1, case["page"], case["hkv"], HEAD_DIM)
            k, v = k.view(shape), v.view(shape)
            s["k_new"].append(_normal(g, (batch, case["hkv"], HEAD_DIM)))
            s["v_new"].append(_normal(g, (batch, case["hkv"], HEAD_DIM)))
        s["k"].append(k)
        s["v"].append(v)
    return s


def _prefill_inputs(case, seed):
    rng, g = random.Random(seed), _gen(seed)
    lens, new = _lengths(case)
    offs, rows = _offsets(rng, lens, 8)
    starts = [0] * len(new)
    for b in range(1, len(new)):
        starts[b] = starts[b - 1] + new[b - 1]
    q = _normal(g, (sum(new), case["hq"], HEAD_DIM))
    k, v = _cache(g, case, rows)
    return {"case": case, "q": q, "k": k, "v": v, "offs": _i32(offs), "lens": _i32(lens), "starts": _i32(starts),
            "new": _i32(new), "max_new": max(new)}


def _opd_inputs(case, seed):
    g = _gen(seed)
    lens = _lengths(case)
    n, vocab = sum(lens), case["vocab"]
    starts = [0]
    for m in lens:
        starts.append(starts[-1] + m)
    mask = torch.ones(n, dtype=torch.uint8, device="cuda")
    for b, (at, m) in enumerate(_inserted(case)):
        mask[starts[b] + at:starts[b] + at + m] = 0
    z = _normal(g, (n, vocab + case["pad"]), 2.0)
    tokens = torch.randint(0, vocab, (n,), generator=g, device="cuda", dtype=torch.int32)
    # the sampled token's log-probability is about -Exp(1)
    target = -torch.empty(n, device="cuda").exponential_(1.0, generator=g)
    rows = torch.arange(n, device="cuda")
    z[rows, tokens.long()] = (target + (math.log(vocab) + 2.0)).to(torch.bfloat16)
    lp = torch.empty(n, dtype=torch.float64, device="cuda")
    for s in range(0, n, 2048):
        lp[s:s + 2048] = -torch.logsumexp(z[s:s + 2048, :vocab].float(), 1).double()
    lp += z[rows, tokens.long()].double()
    # stored by the sampler a little earlier in training (3% much earlier), never within rounding of a clip
    gap = 0.1 * torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    stale = torch.rand(n, generator=g, device="cuda") < 0.03
    far = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 29 + 1
    gap = torch.where(stale, gap + far * torch.where(torch.rand(n, generator=g, device="cuda") < 0.5, -1.0, 1.0), gap)
    for kink in (math.log(1 - DELTA), math.log(1 + DELTA), math.log(KAPPA), -LOG_CLIP, LOG_CLIP):
        gap = torch.where((gap - kink).abs() < 1e-3, kink + 2e-3, gap)
    old = (lp - gap).float()
    teacher = old + torch.randn(n, generator=g, device="cuda")
    return {"case": case, "z": z, "tokens": tokens, "old": old, "teacher": teacher, "mask": mask,
            "starts": _i32(starts)}


def _inputs(case, seed):
    return {"decode": _decode_inputs, "prefill": _prefill_inputs, "opd": _opd_inputs}[case["path"]](case, seed)


# ------------------------------------------------------------------ the framework's calls

def _decode(s, layer):
    case, out = s["case"], s["out"][layer]
    if case["page"]:
        s["attn"].run_paged(s["q"][layer], s["k"][layer], s["v"][layer], s["table"], s["lens"], SCALE, out,
                            k_new=s["k_new"][layer], v_new=s["v_new"][layer])
    else:
        s["attn"].run(s["q"][layer], s["k"][layer], s["v"][layer], s["offs"], s["lens"], SCALE, out)


def prepare(case, seed):
    from paper_2609_36608_amd import DecodeAttention

    s = _inputs(case, seed)
    if case["path"] == "opd":
        return s
    dtype = torch.float32 if case["out"] == "f32" else torch.bfloat16
    if case["path"] == "prefill":
        lens, _ = _lengths(case)
        s["attn"] = DecodeAttention(case["hq"], case["hkv"], case["batch"], max(lens), out_dtype=dtype)
        s["out"] = torch.empty(s["q"].shape, dtype=dtype, device="cuda")
        return s
    s["attn"] = DecodeAttention(case["hq"], case["hkv"], case["batch"], max(_lengths(case)), out_dtype=dtype,
                                page_tokens=case["page"])
    s["out"] = torch.empty((case["layers"], case["batch"], case["hq"], HEAD_DIM), dtype=dtype, device="cuda")
    if case["layers"] > 1:  # a decode step over the layers is captured once and replayed
        _decode(s, 0)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for layer in range(case["layers"]):
                _decode(s, layer)
    return s


def run(s):
    from paper_2609_36608_amd import opd_loss

    case = s["case"]
    if case["path"] == "opd":
        out = {"vocab": case["vocab"]} if case["pad"] else None
        return opd_loss(s["z"], s["tokens"], s["old"], s["teacher"], s["mask"], s["starts"], grad=case["grad"],
                        out=out)
    if case["path"] == "prefill":
        s["attn"].prefill(s["q"], s["k"], s["v"], s["offs"], s["lens"], s["starts"], s["new"], s["max_new"], SCALE,
                          s["out"], split_p=case["split_p"])
        return s["out"]
    if "graph" in s:
        s["graph"].replay()
    else:
        _decode(s, 0)
    if case["page"]:  # the caches hold the appended tokens
        return {"out": s["out"], "k": s["k"], "v": s["v"]}
    return {"out": s["out"]}


# ------------------------------------------------------------------ 64-bit results

def _attend(q, k, v, visible=None):
    """q [m, 128], k / v [t, 128] in 64 bits; visible [m, t] or None for all."""
    s = (q @ k.t().contiguous()) * SCALE
    if visible is not None:
        s.masked_fill_(~visible, -math.inf)
    return torch.softmax(s, 1) @ v


def _exact_decode(case, seed):
    s = _decode_inputs(case, seed)
    lens, g = _lengths(case), case["hq"] // case["hkv"]
    out = torch.empty((case["layers"], case["batch"], case["hq"], HEAD_DIM), dtype=torch.float64, device="cuda")
    for layer in range(case["layers"]):
        k, v = s["k"][layer], s["v"][layer]
        if case["page"]:
            for b, n in enumerate(lens):
                page = int(s["table"][b, (n - 1) // case["page"]])
                k[page, (n - 1) % case["page"]] = s["k_new"][layer][b]
                v[page, (n - 1) % case["page"]] = s["v_new"][layer][b]
        for b, n in enumerate(lens):
            if case["page"]:
                pages = s["table"][b, :-(-n // case["page"])].long()
                kb, vb = k[pages].flatten(0, 1)[:n], v[pages].flatten(0, 1)[:n]
            else:
                at = int(s["offs"][b])
                kb, vb = k[at:at + n], v[at:at + n]
            for h in range(case["hkv"]):
                out[layer, b, h * g:(h + 1) * g] = _attend(s["q"][layer][b, h * g:(h + 1) * g].double(),
                                                           kb[:, h].double().contiguous(),
                                                           vb[:, h].double().contiguous())
    if case["page"]:
        return {"out": out, "k": None, "v": None}
    return {"out": out}


def _exact_prefill(case, seed):
    s = _prefill_inputs(case, seed)
    lens, new = _lengths(case)
    g = case["hq"] // case["hkv"]
    out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
    offs, starts = s["offs"].tolist(), s["starts"].tolist()
    for b, (n, m) in enumerate(zip(lens, new)):
        seen = torch.arange(n, device="cuda")[None] <= (n - m + torch.arange(m, device="cuda"))[:, None]
        seen = seen.repeat_interleave(g, 0)
        for h in range(case["hkv"]):
            q = s["q"][starts[b]:starts[b] + m, h * g:(h + 1) * g].double().reshape(m * g, HEAD_DIM)
            kb = s["k"][offs[b]:offs[b] + n, h].double().contiguous()
            vb = s["v"][offs[b]:offs[b] + n, h].double().contiguous()
            out[starts[b]:starts[b] + m, h * g:(h + 1) * g] = _attend(q, kb, vb, seen).view(m, g, HEAD_DIM)
    return out


def _exact_opd(case, seed):
    s = _opd_inputs(case, seed)
    lens, vocab = _lengths(case), case["vocab"]
    n = sum(lens)
    on = s["mask"].bool()
    lp, scale = torch.empty(n, dtype=torch.float64, device="cuda"), None
    weight = torch.zeros(n, dtype=torch.float64, device="cuda")
    at = 0
    for m in lens:
        part = s["mask"][at:at + m].double()
        weight[at:at + m] = part / (len(lens) * (part.sum() + EPS))
        at += m
    rows, tok = torch.arange(n, device="cuda"), s["tokens"].long()
    for i in range(0, n, 1024):
        lp[i:i + 1024] = s["z"][rows[i:i + 1024], tok[i:i + 1024]].double() - torch.logsumexp(
            s["z"][i:i + 1024, :vocab].double(), 1)
    old = s["old"].double()
    a = s["teacher"].double() - old
    rho = torch.exp((lp - old).clamp(-LOG_CLIP, LOG_CLIP))
    inside = (lp - old).abs() < LOG_CLIP
    clipped = rho.clamp(1 - DELTA, 1 + DELTA)
    free = rho * a <= clipped * a
    loss = torch.where(free, -rho * a, -clipped * a)
    slope = torch.where(free | ((rho > 1 - DELTA) & (rho < 1 + DELTA)), -a, torch.zeros_like(a))
    dual = (a < 0) & (-KAPPA * a < loss)
    loss = torch.where(dual, -KAPPA * a, loss)
    slope = torch.where(dual, torch.zeros_like(a), slope)
    zero = torch.zeros_like(loss)
    loss = torch.where(on, loss, zero)
    scale = torch.where(on & inside, weight * slope * rho, zero)
    res = {"loss": (weight * loss).sum()[None], "token_logp": torch.where(on, lp, zero), "token_weight": weight,
           "token_loss": loss}
    if case["grad"]:
        grad = torch.empty((n, vocab), dtype=torch.float64, device="cuda")
        for i in range(0, n, 1024):
            p = torch.softmax(s["z"][i:i + 1024, :vocab].double(), 1).mul_(-scale[i:i + 1024, None])
            p[torch.arange(p.shape[0], device="cuda"), tok[i:i + 1024]] += scale[i:i + 1024]
            grad[i:i + 1024] = p
        res["grad_logits"] = grad
    return res


def exact(case, seed):
    return {"decode": _exact_decode, "prefill": _exact_prefill, "opd": _exact_opd}[case["path"]](case, seed)
