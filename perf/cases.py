"""The work that a program has this library do, as cases that can be timed and checked.

A serving program holds one cache per layer.  For each layer it calls kivi_prefill once per prompt and
kivi_decode_step (kivi_decode_step_ragged for sequences of different lengths) once per generated token,
so these are the passes measured here: whole decoding steps (append, flush where one is due,
attention) from one short sequence to batches that fill the card, at 2 and 4 bits, with one to 71
query heads per kv-head, group sizes 32 to 128 and both flush policies; and prompt quantisation.

Keys carry a few fixed channels of large magnitude per kv-head, values have none (the pattern of
kv-caches that per-channel key groups are made for); queries are plain normal values.
"""
import math
import random

import torch

from paper_2402_02750_amd import kivi

D = 128
SCALE = 1.0 / math.sqrt(D)


def _step(name, batch, q_heads, kv_heads, tokens, bits=2, group=32, residual=128, policy="window"):
    return {"name": name, "op": "step", "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads,
            "tokens": tokens, "bits": bits, "group": group, "residual": residual, "policy": policy}


def listed():
    """`tokens` is what the cache holds before the pass; a step appends one more."""
    return [
        # the smallest call: one short sequence, four heads (the configuration the smoke test runs)
        _step("step_tiny", 1, 4, 4, 1023, residual=32),
        # one user of a Llama-2-7B-shaped layer in the middle of a chat, a context of odd length
        _step("step_one_user", 1, 32, 32, 3001),
        # the benchmark's configuration: Llama-2-7B-shaped layer, batch 16, context 4096
        _step("step_llama7b", 16, 32, 32, 4095),
        # the streaming configuration (batch 64, prompt 2048) on a step that also flushes a group
        _step("step_stream_flush", 64, 32, 32, 2048 + 127),
        # 4 bits, Llama-2-13B-shaped layer, batch 8, context 8192
        _step("step_llama13b_4bit", 8, 40, 40, 8191, bits=4),
        # grouped-query attention, Mistral-7B-shaped layer, long contexts
        _step("step_mistral_gqa", 4, 32, 8, 32767),
        # eight query heads per kv-head (64 query / 8 kv heads), a medium batch
        _step("step_gqa8", 4, 64, 8, 16384 - 7),
        # multi-query attention, 71 query heads on one kv-head (Falcon-7B-shaped)
        _step("step_mqa", 16, 71, 1, 4095),
        # Algorithm 1's own policy (keys flushed a residual at a time, one value token per step), G = 64
        _step("step_alg1_g64", 8, 32, 32, 4000, group=64, policy="alg1"),
        # a serving batch: 64 sequences of different lengths, grouped-query attention
        {"name": "step_ragged", "op": "ragged", "batch": 64, "q_heads": 32, "kv_heads": 8, "lo": 500, "hi": 8000,
         "lengths": 1, "bits": 2, "group": 32, "residual": 128},
        # prompts of the benchmark's configuration, [b, h, t, d] tensors
        {"name": "prefill_llama7b", "op": "prefill", "batch": 16, "kv_heads": 32, "tokens": 4096, "bits": 2,
         "group": 32, "residual": 128, "policy": "window", "order": "bhtd"},
        # one long prompt of odd length at 4 bits, straight out of a projection ([b, t, h, d])
        {"name": "prefill_4bit_one", "op": "prefill", "batch": 1, "kv_heads": 8, "tokens": 16001, "bits": 4,
         "group": 32, "residual": 128, "policy": "window", "order": "bthd"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "step", "ragged", "prefill"])
    bits = rng.choice([2, 2, 4])
    group = rng.choice([32, 32, 32, 64, 128])
    residual = rng.choice([r for r in (32, 64, 96, 128, 128, 192) if r % group == 0])
    q_heads, kv_heads = rng.choice([(4, 4), (16, 8), (32, 32), (40, 40), (24, 8), (32, 8), (28, 4), (64, 8), (71, 1)])
    if op == "prefill":
        tokens = _log(rng, 100, 32768)
        batch = _log(rng, 1, max(1, min(64, 1500000 // (kv_heads * tokens))))
        return {"op": op, "batch": batch, "kv_heads": kv_heads, "tokens": tokens, "bits": bits, "group": group,
                "residual": residual, "policy": rng.choice(["window", "window", "alg1"]),
                "order": rng.choice(["bhtd", "bthd"])}
    if op == "ragged":
        lo = _log(rng, 50, 4000)
        hi = _log(rng, lo + 1, 16000)
        batch = _log(rng, 4, max(4, min(128, 4200000 // (hi * max(kv_heads, q_heads // 3)))))
        return {"op": op, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "lo": lo, "hi": hi,
                "lengths": rng.randrange(1, 10000), "bits": bits, "group": group, "residual": residual}
    tokens = _log(rng, 200, 32768)
    batch = _log(rng, 1, max(1, min(64, 4200000 // (tokens * max(kv_heads, q_heads // 3)))))
    return {"op": op, "batch": batch, "q_heads": q_heads, "kv_heads": kv_heads, "tokens": tokens, "bits": bits,
            "group": group, "residual": residual, "policy": rng.choice(["window", "window", "window", "alg1"])}


def _lengths(case):
    """Tokens per sequence before the pass."""
    if case["op"] != "ragged":
        return [case["tokens"]] * case["batch"]
    rng = random.Random(case["lengths"])
    return [rng.randint(case["lo"], case["hi"]) for _ in range(case["batch"])]


def _after_prefill(case, tokens):
    """(quantised keys, quantised values) of a sequence after its prompt."""
    g, r = case["group"], case["residual"]
    if case.get("policy", "window") == "window":
        n = max(tokens - r, 0) // g * g
        return n, n
    return tokens - tokens % r, max(tokens - r, 0)


def _after_step(case, tokens):
    """The same after one decoding step."""
    g, r = case["group"], case["residual"]
    nk, nv = _after_prefill(case, tokens)
    total = tokens + 1
    if case.get("policy", "window") == "window":
        while total - nk >= r + g:
            nk += g
        return nk, nk
    if total - nk == r:
        nk += r
    return nk, max(total - r, nv)


def _inputs(case, seed):
    """Prompt keys and values as [b, h, t, d] views, and the step's new rows and queries."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    b, h, t = case["batch"], case["kv_heads"], max(_lengths(case))

    def normal(*shape):
        return torch.randn(*shape, dtype=torch.float16, device="cuda", generator=gen)

    gain = torch.ones(h, D, device="cuda")
    at = torch.rand(h, D, device="cuda", generator=gen).argsort(1)[:, :6]
    gain.scatter_(1, at, 8 + 7 * torch.rand(h, 6, device="cuda", generator=gen))
    gain = gain.half()
    if case.get("order") == "bthd":
        k, v = normal(b, t, h, D).transpose(1, 2), normal(b, t, h, D).transpose(1, 2)
    else:
        k, v = normal(b, h, t, D), normal(b, h, t, D)
    k.mul_(gain[:, None, :])
    if case["op"] == "prefill":
        return k, v, None, None, None
    return k, v, normal(b, h, D) * gain, normal(b, h, D), normal(b, case["q_heads"], D)


def _layout(case):
    g, r = case["group"], case["residual"]
    cap_q = -(-(max(_lengths(case)) + 1) // g) * g
    cap_r = -(-(r + g) // 32) * 32
    return kivi.make_layout(case["batch"], case.get("q_heads", case["kv_heads"]), case["kv_heads"], case["bits"], r,
                            cap_q, cap_r, group=g)


def _policy(case):
    return kivi.KIVI_FLUSH_ALG1 if case.get("policy") == "alg1" else kivi.KIVI_FLUSH_WINDOW


_COUNTERS = ("n_kq", "n_vq", "k_r_start", "n_kr", "v_r_start", "n_vr")


def prepare(case, seed):
    layout = _layout(case)
    cache = kivi.Cache(layout)
    for buf in cache.buffers.values():
        buf.zero_()
    k, v, k_new, v_new, q = _inputs(case, seed)
    if case["op"] == "prefill":
        return {"op": "prefill", "layout": layout, "cache": cache, "k": k, "v": v, "tokens": case["tokens"],
                "policy": _policy(case), "result": {n: cache.view(n) for n in cache.buffers}}
    lens = _lengths(case)
    state = {"op": case["op"], "layout": layout, "cache": cache, "k_new": k_new, "v_new": v_new, "q": q,
             "out": torch.empty(case["batch"], case["q_heads"], D, dtype=torch.float32, device="cuda")}
    result = {"out": state["out"], "k_resid": cache.view("k_resid"), "v_resid": cache.view("v_resid")}
    if case["op"] == "ragged":
        states = kivi.make_states(case["batch"])
        for i, n in enumerate(lens):
            part = kivi.CacheSlice(cache, i, 1, kivi.kivi_seq_state_t())
            kivi.kivi_prefill(part.layout, k[i:i + 1], v[i:i + 1], n, part)
            states[i] = part.state()
        state["states"], state["before"] = states, bytes(states)
    else:
        kivi.kivi_prefill(layout, k, v, lens[0], cache, policy=_policy(case))
        state["before"] = tuple(getattr(cache.c, n) for n in _COUNTERS)
        state["policy"] = _policy(case)
        (k0, v0), (k1, v1) = _after_prefill(case, lens[0]), _after_step(case, lens[0])
        g = case["group"]
        if k1 > k0:     # what a flush adds to the quantised keys and values
            result["k_codes"] = cache.view("k_codes")[:, :, k0 // 32:k1 // 32]
            result["k_scale"] = cache.view("k_scale")[:, :, k0 // g:k1 // g]
            result["k_zero"] = cache.view("k_zero")[:, :, k0 // g:k1 // g]
        if v1 > v0:
            result["v_codes"] = cache.view("v_codes")[:, :, v0 // 32:-(-v1 // 32)]
            result["v_scale"] = cache.view("v_scale")[:, :, v0:v1]
            result["v_zero"] = cache.view("v_zero")[:, :, v0:v1]
    state["result"] = result
    return state


def run(state):
    layout, cache = state["layout"], state["cache"]
    c = cache.c
    if state["op"] == "prefill":
        c.n_kq = c.n_vq = c.k_r_start = c.n_kr = c.v_r_start = c.n_vr = 0     # an empty cache again
        kivi.kivi_prefill(layout, state["k"], state["v"], state["tokens"], cache, policy=state["policy"])
    elif state["op"] == "ragged":
        states = state["states"]
        kivi.ctypes.memmove(states, state["before"], len(state["before"]))    # the same step again
        kivi.kivi_decode_step_ragged(layout, cache, states, state["k_new"], state["v_new"], state["q"], SCALE,
                                     state["out"])
    else:
        c.n_kq, c.n_vq, c.k_r_start, c.n_kr, c.v_r_start, c.n_vr = state["before"]
        kivi.kivi_decode_step(layout, cache, state["k_new"], state["v_new"], state["q"], SCALE, state["out"],
                              policy=state["policy"])
    return state["result"]


def work(case):
    """Every byte of the cache once, inputs once, results once; multiply-adds of logits and outputs."""
    bits, g, h = case["bits"], case["group"], case["kv_heads"]
    packed = D * bits // 8 + D // g * 4           # per token, kv-head and tensor
    total = flops = 0
    if case["op"] == "prefill":
        units = case["batch"] * h
        nk, nv = _after_prefill(case, case["tokens"])
        total = units * (2 * case["tokens"] * 2 * D + (nk + nv) * packed + (2 * case["tokens"] - nk - nv) * 2 * D)
        return {"bytes": total, "flops": units * (nk + nv) * D * 4}
    for n in _lengths(case):
        (k0, v0), (k1, v1) = _after_prefill(case, n), _after_step(case, n)
        total += h * ((k1 + v1) * packed + (2 * (n + 1) - k1 - v1) * 2 * D)       # the attention's reads
        total += h * (2 * 2 * 2 * D + (k1 - k0 + v1 - v0) * (2 * D + packed))     # append, flush
        total += case["q_heads"] * D * (2 + 4)
        flops += 4 * case["q_heads"] * (n + 1) * D
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["op"] == "prefill":
        return "exact"          # codes, scales, zero-points and copied rows are a bit contract
    # four times the distance from the 64-bit result that these cases show (up to 2.1e-4): logits of some
    # hundreds, and zero-points that cancel most of the codes' share, both in fp32 sums
    return {"rel": 8e-4, "max": 1e-2}


def _quantise(x, levels):
    """x fp16 [..., n] in groups along the last axis: code * s + z in 64 bits; the quotient is rounded to
    32 bits before it is rounded to a code, as the quantiser's contract says."""
    lo, hi = x.amin(-1, keepdim=True), x.amax(-1, keepdim=True)
    s = ((hi.double() - lo.double()).float().double() / levels).float().half()
    sd, zd = s.double(), lo.double()
    quotient = ((x.double() - zd).float().double() / torch.where(sd == 0, 1.0, sd)).float()
    code = quotient.round().clamp(0, levels).double() * (sd != 0)
    return code * sd + zd, sd, zd


def exact(case, seed):
    k, v, k_new, v_new, q = _inputs(case, seed)
    g, levels = case["group"], 2 ** case["bits"] - 1
    if case["op"] == "prefill":
        layout = _layout(case)
        b, h, t = case["batch"], case["kv_heads"], case["tokens"]
        nk, nv = _after_prefill(case, t)
        cap = layout.cap_q_tokens
        k_scale = torch.zeros(b, h, cap // g, D, dtype=torch.float64, device="cuda")
        v_scale = torch.zeros(b, h, cap, D // g, dtype=torch.float64, device="cuda")
        k_zero, v_zero = torch.zeros_like(k_scale), torch.zeros_like(v_scale)
        for i in range(b):
            if nk:
                _, s, z = _quantise(k[i, :, :nk].reshape(h, nk // g, g, D).transpose(2, 3), levels)
                k_scale[i, :, :nk // g], k_zero[i, :, :nk // g] = s[..., 0], z[..., 0]
            if nv:
                _, s, z = _quantise(v[i, :, :nv].reshape(h, nv, D // g, g), levels)
                v_scale[i, :, :nv], v_zero[i, :, :nv] = s[..., 0], z[..., 0]
        return {"k_codes": None, "k_scale": k_scale, "k_zero": k_zero, "v_codes": None, "v_scale": v_scale,
                "v_zero": v_zero, "k_resid": None, "v_resid": None}
    h, hq = case["kv_heads"], case["q_heads"]
    out = torch.empty(case["batch"], hq, D, dtype=torch.float64, device="cuda")
    for i, n in enumerate(_lengths(case)):
        nk, nv = _after_step(case, n)
        ki = torch.cat([k[i, :, :n], k_new[i, :, None]], 1)
        vi = torch.cat([v[i, :, :n], v_new[i, :, None]], 1)
        kd, vd = ki.double(), vi.double()
        if nk:
            x, _, _ = _quantise(ki[:, :nk].reshape(h, nk // g, g, D).transpose(2, 3), levels)
            kd[:, :nk] = x.transpose(2, 3).reshape(h, nk, D)
        if nv:
            x, _, _ = _quantise(vi[:, :nv].reshape(h, nv, D // g, g), levels)
            vd[:, :nv] = x.reshape(h, nv, D)
        logits = torch.matmul(q[i].double().reshape(h, hq // h, D), kd.transpose(1, 2).contiguous()) * SCALE
        out[i] = torch.matmul(torch.softmax(logits, -1), vd).reshape(hq, D)
    return {"out": out, "k_resid": None, "v_resid": None}
