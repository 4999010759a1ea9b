"""Workloads of this library's entry points, for timing them and comparing their outputs.

Every case is one call, or one step, of a program that serves or calibrates a decoder with an
evicted KV cache (head dimension 128, bf16): the prompt compression of a routed plan
(`evict_prefill`), the hand-off to decoding (`decode_init_from_prefill`), a decode step of every
layer (`decode_step`) and the entropy profile that allocates capacities (`entropy_profile`).

`listed()` holds the workloads of `synth/workloads.py` and `bench.py` (one layer at 1K, the
32-layer route at 8K alone and at batch 8, 32K prompts, the H2O / TOVA composition, decode steps,
full-span H2O, the entropy profile) and ragged ones of the same ranges; `draw(rng)` draws others.
Inputs are N(0, 1) with a planted sink, heavy hitters and recent keys, the recipe of `synth/`.

Gathered K and V rows are copies, so they come back as their 16-bit patterns.  A prompt
compression also returns its scores by position where a program asks for them.
"""
import math

import torch

import paper_2606_15157_amd as rkv

D = 128
DEVICE = "cuda"
DECODE_TOKENS = 16      # distinct new tokens a decode case cycles through

# cost of the largest listed case: drawn ones stay below it
MAX_BYTES, MAX_FLOPS = 9.5e9, 2.3e12


def listed():
    return [
        # one layer of a short prompt: the smallest call, bound by launches and latency
        {"name": "one_layer_1k", "kind": "prefill", "route": "snapkv", "layers": 1, "batch": 1, "seq": 1024, "hq": 32,
         "hkv": 8, "window": 32, "pool": 7, "budget": 128, "scores": True, "handoff": False},
        # the whole prompt compression of one 8K sequence, every layer in one call (the benchmark)
        {"name": "route_8k", "kind": "prefill", "route": "mixed", "layers": 32, "batch": 1, "seq": 8192, "hq": 32,
         "hkv": 8, "window": 32, "pool": 7, "budget": 512, "scores": False, "handoff": False},
        # the same route over a batch of eight prompts
        {"name": "route_8k_b8", "kind": "prefill", "route": "mixed", "layers": 32, "batch": 8, "seq": 8192, "hq": 32,
         "hkv": 8, "window": 32, "pool": 7, "budget": 512, "scores": False, "handoff": False},
        # long prompts with a wide observation window
        {"name": "long_32k_b4_w64", "kind": "prefill", "route": "mixed", "layers": 32, "batch": 4, "seq": 32768,
         "hq": 32, "hkv": 8, "window": 64, "pool": 7, "budget": 1024, "scores": False, "handoff": False},
        # a prompt of no round length under H2O / TOVA tied in both phases, handed to decoding
        {"name": "composition_20k", "kind": "prefill", "route": "h2o_tova", "layers": 32, "batch": 1, "seq": 20011,
         "hq": 32, "hkv": 8, "window": 32, "pool": 7, "budget": 512, "scores": False, "handoff": True},
        # a ragged batch with two query heads per KV head, an odd window and a narrow pool, scores
        # by position returned (a program that studies routes)
        {"name": "ragged_3k", "kind": "prefill", "route": "mixed", "layers": 7, "batch": 3, "seq": 3331, "hq": 16,
         "hkv": 8, "window": 27, "pool": 5, "budget": 331, "scores": True, "handoff": False},
        # eight query heads per KV head: eight row tiles at an ordinary window
        {"name": "grouped8_12k", "kind": "prefill", "route": "mixed", "layers": 16, "batch": 1, "seq": 12289, "hq": 64,
         "hkv": 8, "window": 32, "pool": 7, "budget": 640, "scores": True, "handoff": False},
        # H2O accumulating over every prompt query
        {"name": "full_span_8k", "kind": "prefill", "route": "h2o_full", "layers": 4, "batch": 1, "seq": 8192, "hq": 32,
         "hkv": 8, "window": 32, "pool": 7, "budget": 512, "scores": True, "handoff": False},
        # one decode step of one sequence (interactive), and of a full batch
        {"name": "decode_b1", "kind": "decode", "route": "h2o_tova", "layers": 32, "batch": 1, "capacity": 512,
         "hq": 32, "hkv": 8},
        {"name": "decode_b64", "kind": "decode", "route": "h2o_tova", "layers": 32, "batch": 64, "capacity": 1024,
         "hq": 32, "hkv": 8},
        # calibration of the capacities: every query of a sequence, and the last ones of a ragged batch
        {"name": "entropy_4k", "kind": "entropy", "layers": 32, "batch": 1, "seq": 4096, "queries": 4096, "hq": 32,
         "hkv": 8},
        {"name": "entropy_tail_9k", "kind": "entropy", "layers": 8, "batch": 2, "seq": 9001, "queries": 515, "hq": 16,
         "hkv": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill"] * 5 + ["full_span", "decode", "decode", "entropy"])
    hq, hkv = rng.choice([(32, 8), (32, 8), (32, 8), (16, 8), (8, 8), (64, 8), (16, 4)])
    g = hq // hkv
    if kind == "decode":
        c = {"kind": "decode", "route": rng.choice(["h2o", "tova", "h2o_tova"]), "layers": rng.randint(8, 32),
             "batch": _log_int(rng, 1, 64), "capacity": _log_int(rng, 64, 2048), "hq": hq, "hkv": hkv}
    elif kind == "entropy":
        seq = _log_int(rng, 500, 16000)
        c = {"kind": "entropy", "layers": rng.randint(1, 32), "batch": rng.randint(1, 4), "seq": seq,
             "queries": min(seq, _log_int(rng, 100, 8000)), "hq": hq, "hkv": hkv}
    else:
        full = kind == "full_span"
        seq = _log_int(rng, 400, 12000) if full else _log_int(rng, 400, 32768)
        window = 32
        while not full and rng.random() < 0.5:
            window = rng.randint(8, 64)
            if g * ((window + 31) // 32) <= 8:
                break
            window = 32
        route = "h2o_full" if full else rng.choice(["mixed", "mixed", "snapkv", "h2o", "h2o_tova"])
        c = {"kind": "prefill", "route": route, "layers": rng.randint(1, 8) if full else rng.randint(4, 32),
             "batch": 1 if full else _log_int(rng, 1, 8), "seq": seq, "hq": hq, "hkv": hkv, "window": window,
             "pool": rng.choice([3, 5, 7, 7, 7, 13]), "budget": min(_log_int(rng, 100, 2048), seq // 3),
             "scores": full or rng.random() < 0.5, "handoff": route == "h2o_tova"}
    while True:
        w = work(c)
        if w["bytes"] <= MAX_BYTES and w["flops"] <= MAX_FLOPS:
            return c
        key = "batch" if c["batch"] > 1 else "layers"
        c[key] = max(1, c[key] // 2)


# ---- plans

def _rules(case):
    n, route = case["layers"], case["route"]
    if route == "mixed":   # StreamingLLM, SnapKV, H2O and SnapKV layers in the shares 2 : 14 : 12 : 4
        a, b, c = round(n / 16), round(n / 2), round(7 * n / 8)
        return [rkv.STREAMING if l < a else rkv.H2O if b <= l < c else rkv.SNAPKV for l in range(n)]
    if route == "h2o_tova":
        return [rkv.H2O if 2 * l < n else rkv.TOVA for l in range(n)]
    return [{"snapkv": rkv.SNAPKV, "h2o": rkv.H2O, "tova": rkv.TOVA, "h2o_full": rkv.H2O_FULL}[route]] * n


def _budgets(case):
    """A linear ramp of capacities over the layers (Eq. 3); equal ones for a tied route."""
    n, avg = case["layers"], case["budget"]
    if n == 1 or case["handoff"]:
        return [avg] * n
    return rkv.allocate_budgets([1024.0 - 896.0 * l / (n - 1) for l in range(n)], n * avg, min(48, avg))


def _plan(case):
    rules, budgets = _rules(case), _budgets(case)
    if case["handoff"]:
        return rkv.Plan.from_scoped_route(rules, [rkv.SCOPE_BOTH] * len(rules), budgets, window=case["window"],
                                          pool_kernel=case["pool"])
    return rkv.Plan(rules, budgets, window=case["window"], pool_kernel=case["pool"])


# ---- inputs

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(seed)


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device=DEVICE, dtype=torch.bfloat16)


def _prompt_layer(g, case, rows):
    """Queries of the last `rows` positions, keys and values of one layer; along the mean of the
    last queries, key 0 is raised by 3 standard deviations of a logit, 16 keys by 2 and the last
    64 by 1."""
    b, seq, hq, hkv = case["batch"], case["seq"], case["hq"], case["hkv"]
    q, k = _normal(g, b, hq, rows, D), _normal(g, b, hkv, seq, D)
    last = q.view(b, hkv, hq // hkv, rows, D)[:, :, :, max(0, rows - 64):].float().mean(dim=(2, 3))
    u = D ** 0.5 * last / (last * last).sum(-1, keepdim=True)
    recent = min(64, seq - 1)
    heavy = torch.rand((b, hkv, seq - recent - 1), generator=g, device=DEVICE)
    heavy = 1 + heavy.topk(min(16, heavy.shape[-1]), dim=-1).indices
    at = heavy.unsqueeze(-1).expand(-1, -1, -1, D)
    k.scatter_(2, at, (k.gather(2, at).float() + 2 * u.unsqueeze(2)).to(k.dtype))
    k[:, :, 0] = (k[:, :, 0].float() + 3 * u).to(k.dtype)
    k[:, :, seq - recent:] = (k[:, :, seq - recent:].float() + u.unsqueeze(2)).to(k.dtype)
    return q, k, _normal(g, b, hkv, seq, D)


def _query_rows(case, rule):
    return case["seq"] if rule == rkv.H2O_FULL else case["window"]


def _arena(shapes, dtype):
    """Tensors of the given shapes side by side in one buffer, and that buffer."""
    sizes = [math.prod(s) for s in shapes]
    flat = torch.zeros(sum(sizes), dtype=dtype, device=DEVICE)
    return [t.view(s) for t, s in zip(flat.split(sizes), shapes)], flat


def _prompt_inputs(case, seed):
    g = _generator(seed)
    rules = _rules(case)
    qkv = [_prompt_layer(g, case, _query_rows(case, r)) for r in rules]
    return [q if r != rkv.STREAMING else None for (q, _, _), r in zip(qkv, rules)], [x[1] for x in qkv], [x[2] for x in qkv]


def _prepare_prefill(case, seed):
    plan = _plan(case)
    b, seq, hq, hkv = case["batch"], case["seq"], case["hq"], case["hkv"]
    q, k, v = _prompt_inputs(case, seed)
    counts = plan.retained_counts(seq)
    rows = [(b, hkv, n, D) for n in counts]
    out, result = {}, {}
    for key, name in (("k_out", "k"), ("v_out", "v")):
        out[key], flat = _arena(rows, torch.bfloat16)
        result[name] = flat.view(torch.int16)
    out["idx"], result["idx"] = _arena([s[:3] for s in rows], torch.int32)
    if case["scores"]:
        out["scores"], result["scores"] = _arena([(b, hkv, seq)] * len(rows), torch.float32)
    state = None
    if case["handoff"]:
        out["acc"], _ = _arena([s[:3] for s in rows], torch.float32)
        state = {}
        for key in ("k_cache", "v_cache"):
            state[key], flat = _arena(rows, torch.bfloat16)
            result[key] = flat.view(torch.int16)
        state["pos"], result["pos"] = _arena([s[:3] for s in rows], torch.int32)
        state["acc"] = [torch.zeros(s[:3], device=DEVICE) if r == rkv.H2O else None
                        for s, r in zip(rows, plan.rules_decode)]
    return {"plan": plan, "q": q, "k": k, "v": v, "out": out, "state": state, "result": result,
            "workspace": rkv.alloc_workspace(plan, b, seq, hq, hkv)}


def _prepare_decode(case, seed):
    """The caches of prompts compressed earlier (slots in position order: spread over the prompt,
    then the recent half) and the new tokens of a few steps."""
    g = _generator(seed)
    b, c, hq, hkv, rules = case["batch"], case["capacity"], case["hq"], case["hkv"], _rules(case)
    prompt, recent = 8 * c, c // 2
    stride = (prompt - recent) // (c - recent)
    spread = torch.arange(c - recent, device=DEVICE, dtype=torch.int32) * stride
    tail = torch.arange(prompt - recent, prompt, device=DEVICE, dtype=torch.int32).expand(b, hkv, recent)
    state = {"k_cache": [], "v_cache": [], "pos": [], "acc": []}
    state["k_cache"], flat_k = _arena([(b, hkv, c, D)] * len(rules), torch.bfloat16)
    state["v_cache"], flat_v = _arena([(b, hkv, c, D)] * len(rules), torch.bfloat16)
    state["pos"], flat_pos = _arena([(b, hkv, c)] * len(rules), torch.int32)
    n_h2o = sum(r == rkv.H2O for r in rules)
    acc, flat_acc = _arena([(b, hkv, c)] * n_h2o, torch.float32)
    for l, r in enumerate(rules):
        state["k_cache"][l].copy_(_normal(g, b, hkv, c, D))
        state["v_cache"][l].copy_(_normal(g, b, hkv, c, D))
        jitter = torch.randint(0, stride, (b, hkv, c - recent), generator=g, device=DEVICE, dtype=torch.int32)
        state["pos"][l].copy_(torch.cat([spread + jitter, tail], dim=-1))
        if r == rkv.H2O:   # accumulated attention: a few large entries, many small ones
            acc[len([a for a in state["acc"] if a is not None])].copy_(
                torch.randn((b, hkv, c), generator=g, device=DEVICE).exp_().mul_(0.02))
            state["acc"].append(acc[len([a for a in state["acc"] if a is not None])])
        else:
            state["acc"].append(None)
    tokens = []
    for heads in (hq, hkv, hkv):
        x = [_normal(g, DECODE_TOKENS, b, heads, D) for _ in rules]
        tokens.append([[t[i] for t in x] for i in range(DECODE_TOKENS)])
    plan = rkv.Plan([rkv.FULL] * len(rules), [0] * len(rules), rules, [c] * len(rules))
    result = {"k_cache": flat_k.view(torch.int16), "v_cache": flat_v.view(torch.int16), "pos": flat_pos}
    if n_h2o:
        result["acc"] = flat_acc
    return {"plan": plan, "state": state, "tokens": tokens, "step": 0, "prompt": prompt, "result": result}


def _prepare_entropy(case, seed):
    q, k = [], []
    g = _generator(seed)
    for _ in range(case["layers"]):
        x = _prompt_layer(g, case, case["queries"])
        q.append(x[0])
        k.append(x[1])
    return {"q": q, "k": k}


def prepare(case, seed):
    kind = case["kind"]
    state = {"prefill": _prepare_prefill, "decode": _prepare_decode, "entropy": _prepare_entropy}[kind](case, seed)
    state["kind"] = kind
    return state


def run(s):
    if s["kind"] == "prefill":
        out = rkv.evict_prefill(s["plan"], s["q"], s["k"], s["v"], out=s["out"], workspace=s["workspace"])
        if s["state"] is not None:
            rkv.decode_init_from_prefill(s["plan"], out, s["state"])
        return s["result"]
    if s["kind"] == "decode":
        i = s["step"] % DECODE_TOKENS
        q, k, v = (t[i] for t in s["tokens"])
        rkv.decode_step(s["plan"], s["state"], q, k, v, s["prompt"] + s["step"])
        s["step"] += 1
        return s["result"]
    out = rkv.entropy_profile(s["q"], s["k"])
    return {"h": out["h"], "rows": out["rows"]}


# ---- what a pass cannot do without

def work(case):
    b, hq, hkv, n = case["batch"], case["hq"], case["hkv"], case["layers"]
    if case["kind"] == "decode":
        c, n_h2o = case["capacity"], sum(r == rkv.H2O for r in _rules(case))
        entries = n * b * hkv * c
        # keys and positions read, accumulated scores read and written, the new token read and stored
        nbytes = entries * (2 * D + 4) + 8 * b * hkv * c * n_h2o + 2 * D * b * n * (hq + 2 * hkv + 2 * hkv)
        return {"bytes": nbytes, "flops": 2 * D * n * b * hq * (c + 1)}
    seq = case["seq"]
    if case["kind"] == "entropy":
        nq = case["queries"]
        seen = nq * (seq - nq) + nq * (nq + 1) // 2
        return {"bytes": n * b * (2 * D * (hkv * seq + hq * nq) + 4 * hq * nq), "flops": 2 * D * n * b * hq * seen}
    nbytes = flops = 0
    for rule, budget in zip(_rules(case), _budgets(case)):
        keep = min(budget, seq)
        if rule != rkv.STREAMING:
            rows = {rkv.TOVA: 1, rkv.H2O_FULL: seq}.get(rule, case["window"])
            nbytes += 2 * D * b * (hkv * seq + hq * rows)
            flops += 2 * D * b * hq * (seq * (seq + 1) // 2 if rule == rkv.H2O_FULL else rows * seq)
        copies = 3 if case["handoff"] else 2     # kept rows read once, written to the output and the decode cache
        nbytes += b * hkv * keep * (2 * 2 * D * copies + 4 * (copies - 1))
        if case["scores"] and rule != rkv.STREAMING:
            nbytes += 4 * b * hkv * seq
    return {"bytes": nbytes, "flops": flops}


# ---- correctness

def tolerance(case):
    if case["kind"] == "decode":
        # a victim may be another one of two entries with equal scores: its slot's values differ
        slots = case["layers"] * case["batch"] * case["hkv"] * case["capacity"]
        return {"rel": 1e-6 + 1.0 / math.sqrt(slots), "max": 0.99, "differ": 0.01}
    if case["kind"] == "entropy":   # 32-bit rows, 7e-8 from the 64-bit ones
        return {"rel": 4e-7, "max": 4e-5}
    # 32-bit sums of exponentials of bf16 products: over a window's rows 6e-8 .. 6e-7 from the 64-bit
    # ones, over every prompt query 6e-7 .. 9e-6 (thousands of terms).  Retained positions whose scores
    # are equal but for rounding may be exchanged, and the kept rows between them then move by one
    rel = 4e-5 if case["route"] == "h2o_full" else 3e-6
    return {"rel": rel, "max": 100 * rel, "differ": 0.01}


def _attention(q, k, first):
    """Causal softmax rows in 64 bits: q [n, D] at positions first .. first + n - 1."""
    z = q.double() @ k.double().t() / D ** 0.5
    at = torch.arange(first, first + q.shape[0], device=q.device).unsqueeze(1)
    return torch.softmax(z.masked_fill_(torch.arange(k.shape[0], device=q.device) > at, -math.inf), dim=1)


def _exact_scores(case, rule, budget, q, k):
    """The ranking scores of one layer [B, Hkv, L], zero past its candidates."""
    b, seq, hkv, w = case["batch"], case["seq"], case["hkv"], case["window"]
    g = case["hq"] // hkv
    end = {rkv.SNAPKV: seq - w if budget > w else 0, rkv.TOVA: seq}.get(rule, seq - budget // 2)
    s = torch.zeros((b, hkv, seq), dtype=torch.float64, device=DEVICE)
    for i in range(b):
        for h in range(hkv):
            for qh in q[i, h * g:(h + 1) * g]:
                if rule == rkv.TOVA:
                    qh = qh[w - 1:]
                a = torch.zeros(seq, dtype=torch.float64, device=DEVICE)
                for r in range(0, qh.shape[0], 4096):
                    rows = qh[r:r + 4096]
                    a += _attention(rows, k[i, h], seq - qh.shape[0] + r).sum(0)
                if rule == rkv.SNAPKV:
                    p = case["pool"] // 2
                    a[:seq - w] = torch.nn.functional.max_pool1d(a[None, None, :seq - w], case["pool"], 1, p)[0, 0]
                s[i, h] += a / g
    s[:, :, end:] = 0
    return s


def exact(case, seed):
    if case["kind"] == "prefill":
        if not case["scores"]:
            return None
        if work(case)["flops"] > 1.2e12:   # the 64-bit logits would take too long
            return None
        q, k, _ = _prompt_inputs(case, seed)
        rules, budgets = _rules(case), _budgets(case)
        scores = [torch.zeros((case["batch"], case["hkv"], case["seq"]), dtype=torch.float64, device=DEVICE)
                  if r == rkv.STREAMING else _exact_scores(case, r, n, qi, ki) for r, n, qi, ki in zip(rules, budgets, q, k)]
        res = {"k": None, "v": None, "idx": None, "scores": torch.cat([t.flatten() for t in scores])}
        if case["handoff"]:
            res.update({"k_cache": None, "v_cache": None, "pos": None})
        return res
    if case["kind"] == "entropy":
        if work(case)["flops"] > 2.3e12:
            return None
        s = _prepare_entropy(case, seed)
        g, seq, nq = case["hq"] // case["hkv"], case["seq"], case["queries"]
        rows = torch.empty((case["layers"], case["batch"], case["hq"], nq), dtype=torch.float64, device=DEVICE)
        for l in range(case["layers"]):
            for i in range(case["batch"]):
                for h in range(case["hq"]):
                    for r in range(0, nq, 4096):
                        x = s["q"][l][i, h, r:r + 4096]
                        p = _attention(x, s["k"][l][i, h // g], seq - nq + r)
                        rows[l, i, h, r:r + 4096] = -torch.xlogy(p, p).sum(1)
        return {"h": rows.mean(dim=(1, 2, 3)), "rows": rows}
    # one decode step: every H2O entry's accumulated score; the new token replaces the smallest one
    # outside the recent half
    s = _prepare_decode(case, seed)
    g, c = case["hq"] // case["hkv"], case["capacity"]
    acc = []
    for l, r in enumerate(_rules(case)):
        if r != rkv.H2O:
            continue
        q, kn = s["tokens"][0][0][l].double(), s["tokens"][1][0][l].double()
        keys = torch.cat([s["state"]["k_cache"][l].double(), kn.unsqueeze(2)], dim=2)       # [B, Hkv, C + 1, D]
        qg = q.view(case["batch"], case["hkv"], g, 1, D)
        z = torch.stack([(qg[:, :, i] * keys).sum(-1) for i in range(g)], dim=2) / D ** 0.5
        total = torch.softmax(z, dim=-1).mean(dim=2)
        total[:, :, :c] += s["state"]["acc"][l].double()
        held = total[:, :, :c].masked_fill(s["state"]["pos"][l] > s["prompt"] - c // 2, math.inf)
        victim = held.argmin(-1, keepdim=True)
        acc.append(total[:, :, :c].scatter(2, victim, total[:, :, c:]).flatten())
    res = {"k_cache": None, "v_cache": None, "pos": None}
    if acc:
        res["acc"] = torch.cat(acc)
    return res
