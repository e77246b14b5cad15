"""GPU parity of decode_one_kernel (one query head per kv-head) at the sizes where it can go wrong: windows that end inside
a slot, a step or a ring, tiles that do not fill a step, units in one, several and many parts, more units than fit the chip at
once, scales outside the ordinary range."""
import numpy as np
import pytest

import gpu_harness as gh
from paper_2402_02750_amd import kivi, workloads
from paper_2402_02750_amd.workloads import CONFIGS, scaled

pytestmark = pytest.mark.gpu

# (heads, batch, bits, G, residual, prompt tokens, steps, gain of the keys, gain of the values)
CASES = [
    (1, 1, 2, 32, 32, 1, 3, 1, 1),              # nothing quantised, two to four rows
    (2, 1, 4, 32, 32, 63, 2, 1, 1),             # ... a window of two tiles; a flush in the second step
    (3, 1, 2, 32, 32, 32 + 32 * 1, 12, 1, 1),   # one tile; 33 to 44 rows
    (2, 2, 2, 32, 32, 32 + 32 * 8, 17, 1, 1),   # a full step of tiles; rows past 48: a second step of rows
    (2, 2, 4, 32, 64, 64 + 32 * 9, 9, 1, 1),    # ... of the other width, one tile more
    (5, 3, 2, 32, 128, 1000, 40, 1, 1),         # a ring that wraps, two flushes, two parts a unit and more
    (4, 1, 2, 32, 32, 30000, 2, 1, 1),          # many parts
    (4, 1, 4, 32, 32, 30000, 2, 1, 1),
    (2, 1, 2, 32, 1024, 3000, 3, 1, 1),         # a large window: most steps are rows
    (32, 9, 2, 32, 128, 1300, 14, 1, 1),        # one part a unit, not all compute units alike; a flush in the last step but two
    (32, 9, 4, 32, 128, 1300, 14, 1, 1),
    (2, 2, 2, 32, 64, 9599, 3, 1, 1),           # a flush beside parts of many steps
    (32, 26, 4, 32, 32, 900, 2, 1, 1),          # a few more units than fit at once
    (3, 2, 2, 64, 128, 2001, 3, 1, 1),
    (3, 2, 4, 128, 128, 2001, 3, 1, 1),
    (2, 2, 2, 32, 64, 900, 2, 60, 1),           # key scales past 64
    (2, 2, 4, 32, 64, 900, 2, 60, 500),         # large value scales
    (2, 2, 2, 32, 64, 900, 2, 1, 2.0 ** -13),   # value scales among fp16's subnormals
    (2, 2, 4, 32, 64, 900, 2, 2.0 ** -10, 1),   # small key scales
    (2, 2, 2, 32, 64, 900, 2, 2.0 ** -12, 1),
    (2, 2, 4, 64, 64, 900, 2, 2.0 ** -14, 1),   # ... next to fp16's subnormals
]


@pytest.mark.parametrize("heads,batch,bits,group,residual,tokens,steps,kgain,vgain", CASES)
def test_one_head(heads, batch, bits, group, residual, tokens, steps, kgain, vgain):
    """Decoding steps from a prompt, every step against the oracle; the cache after the last, of all heads.  Tolerance: operands are
    rounded to 22 bits; the products of a logit, which cancel in part, sum to up to 150 in magnitude here, so that a logit is off by up to
    150 x 2^-23, and an output by twice that and the fp32 sums' share: 4e-5 of the largest value."""
    run_steps(heads, batch, bits, group, residual, tokens, steps, kgain, vgain, "window", bound=4e-5)


# K and V split at different tokens: a value token quantised in most steps (every position in a tile, both halves of a
# slot's tokens), values of a partly filled tile, key flushes (after which the window has no token with both rows)
UNEVEN_CASES = [
    (1, 1, 2, 32, 32, 1, 70, 1, 1),             # from nothing quantised to two tiles
    (1, 1, 4, 32, 32, 20, 50, 1, 1),
    (3, 2, 2, 64, 128, 2001, 40, 1, 1),         # rows, mixed slots and tiles in several parts
    (3, 2, 4, 128, 128, 2001, 40, 1, 1),
    (2, 2, 2, 32, 96, 959, 36, 1, 1),
    (2, 2, 4, 64, 64, 1000, 36, 1, 1),
    (2, 2, 2, 128, 128, 511, 34, 1, 1),
    (2, 1, 2, 32, 1024, 3000, 3, 1, 1),         # a large window
    (2, 1, 4, 32, 30016, 30100, 3, 1, 1),       # hardly anything but
    (32, 9, 2, 64, 128, 1300, 3, 1, 1),         # one part a unit
    (32, 9, 4, 32, 128, 1300, 3, 1, 1),
    (32, 26, 4, 32, 32, 900, 2, 1, 1),          # a few more units than fit at once
    (4, 1, 2, 32, 32, 30000, 2, 1, 1),
    (2, 2, 2, 32, 64, 900, 2, 60, 1),
    (2, 2, 4, 32, 64, 900, 2, 60, 500),
    (2, 2, 2, 64, 64, 900, 2, 1, 2.0 ** -13),
]


@pytest.mark.parametrize("heads,batch,bits,group,residual,tokens,steps,kgain,vgain", UNEVEN_CASES)
def test_one_head_uneven(heads, batch, bits, group, residual, tokens, steps, kgain, vgain):
    """The same with the policy that flushes keys and values separately; tolerance as above (fp16 value rows are weighted with
    fp32 probabilities)."""
    run_steps(heads, batch, bits, group, residual, tokens, steps, kgain, vgain, "alg1", bound=4e-5)


# (heads, batch, bits, G, residual, policy, prompt tokens)
TIGHT_CASES = [
    (2, 2, 2, 32, 32, "window", 300),
    (2, 1, 4, 32, 64, "window", 200),
    (1, 2, 2, 32, 96, "window", 128),
    (2, 1, 2, 64, 64, "window", 500),           # flushes in a launch of their own
    (2, 2, 2, 32, 32, "alg1", 300),
    (2, 1, 4, 64, 64, "alg1", 200),
]


@pytest.mark.parametrize("heads,batch,bits,group,residual,policy,tokens", TIGHT_CASES)
def test_one_head_tight_ring(heads, batch, bits, group, residual, policy, tokens):
    """Rings with no slot to spare, in which the row that a step writes lies next to those that it flushes, for more than two
    turns of the ring."""
    ring = residual + group
    run_steps(heads, batch, bits, group, residual, tokens, 2 * ring + 5, 1, 1, policy, bound=4e-5, ring=ring)



# (bits, G, policy)
FORMS = [(2, 32, "window"), (4, 32, "window"), (2, 64, "alg1"), (4, 32, "alg1"), (4, 128, "window")]


@pytest.mark.parametrize("ratio,size", [(2.0 ** 12, 2.0 ** -8), (2.0 ** 16, 2.0 ** -8), (2.0 ** 18, 2.0 ** -8), (2.0 ** 23, 2.0 ** -8)])
@pytest.mark.parametrize("bits,group,policy", FORMS)
def test_one_head_query_outliers(bits, group, policy, ratio, size):
    """A channel at which the query looks with `ratio` times the weight, and whose keys are smaller by as much, takes no bits
    from the others.  Tolerance as in test_key_outliers (test_gpu_tiles.py): 2^-20 of the largest value."""
    rng = np.random.default_rng(bits + group)
    tokens = 1500
    k = rng.standard_normal((1, 3, tokens, 128)) / size
    q = rng.standard_normal((1, 3, 128)) * size
    k[..., 5] /= ratio
    q[..., 5] = np.sign(q[..., 5]) * size * ratio
    check_outliers(bits, group, policy, k, rng.standard_normal((1, 3, tokens, 128)), q, 2.0 ** -20)


@pytest.mark.parametrize("large,small", [(1000, 2.0 ** -5), (4000, 2.0 ** -3), (30000, 2.0 ** -3)])
@pytest.mark.parametrize("bits,group,policy", FORMS)
def test_one_head_key_outliers(bits, group, policy, large, small):
    """A key channel 2^15 and more times larger than the others, at which the query hardly looks, takes no bits from them.
    Tolerance as above."""
    rng = np.random.default_rng(bits + group)
    tokens = 1500
    k = rng.standard_normal((1, 3, tokens, 128)) * small
    k[..., 5] = rng.uniform(-1, 1, (1, 3, tokens)) * large
    q = rng.standard_normal((1, 3, 128)) / small
    q[..., 5] *= small / large
    check_outliers(bits, group, policy, k, rng.standard_normal((1, 3, tokens, 128)), q, 2.0 ** -20)


@pytest.mark.parametrize("ratio", [2.0 ** 12, 2.0 ** 16, 2.0 ** 18])
@pytest.mark.parametrize("bits,group,policy", [f for f in FORMS if f[1] < 128])
def test_one_head_value_groups(bits, group, policy, ratio):
    """A channel group whose values are `ratio` times smaller than the others' keeps its bits: the bound, as in test_value_outliers
    (test_gpu_tiles.py) 2^-20 of the largest value, holds for every group with its own largest value."""
    rng = np.random.default_rng(bits + group)
    k, v = (rng.standard_normal((1, 3, 1500, 128)) for _ in range(2))
    v *= 64
    v[..., :group] /= ratio
    check_outliers(bits, group, policy, k, v, rng.standard_normal((1, 3, 128)), 2.0 ** -20)


@pytest.mark.parametrize("outlier,size,every", [(40000, 2.0 ** -4, 5000), (1000, 2.0 ** -8, 5000), (40000, 2.0 ** -4, 32), (1000, 2.0 ** -8, 320)])
@pytest.mark.parametrize("bits,group,policy", FORMS)
def test_one_head_value_outliers(bits, group, policy, outlier, size, every):
    """Tokens with very large values and no probability take no bits from the others: 2^-20 of the largest ordinary value."""
    rng = np.random.default_rng(bits + group)
    tokens = 1500
    k, v = (rng.standard_normal((1, 3, tokens, 128)) for _ in range(2))
    q = np.repeat(rng.standard_normal((1, 1, 128)) * 0.3, 3, axis=1)
    v *= size
    ordinary = float(np.abs(v).max())
    for t in range(7, tokens - 128, every):
        k[:, :, t] = -40 * np.sign(q[0, 0])
        v[:, :, t] = outlier * np.sign(v[:, :, t])
    check_outliers(bits, group, policy, k, v, q, 2.0 ** -20, ordinary)


def check_outliers(bits, group, policy, k, v, q, bound, largest=None):
    """An attention call against the oracle; `bound` is in units of `largest`, by default of every channel group's largest value."""
    gh.require_gpu()
    k, v, q = (x.astype(np.float16) for x in (k, v, q))
    heads = k.shape[1]
    w = scaled(CONFIGS["llama7b"], name="oneoutliers", batch=1, n_q_heads=heads, n_kv_heads=heads, bits=bits, group=group, residual=128, seed=1)
    print(f"case one head outliers B={bits} G={group} {policy}", flush=True)
    at = [(0, h) for h in range(heads)]
    ref = gh.oracle_attention_for_heads(w, gh.oracle_cache_for_heads(w, k, v, at, policy), q, at)
    flush = kivi.KIVI_FLUSH_ALG1 if policy == "alg1" else kivi.KIVI_FLUSH_WINDOW
    layout, cache = gh.gpu_prefill(w, k, v, flush, kivi.KIVI_DECODE_AUTO)
    err = np.abs(gh.pick_heads(gh.gpu_attention(layout, cache, q, w.softmax_scale), w, at) - ref)
    err = err.reshape(-1, 128 // group, group).max((0, 2))
    bounds = bound * (np.abs(v.astype(np.float32)).reshape(-1, 128 // group, group).max((0, 2)) if largest is None else largest)
    assert (err <= bounds).all(), f"{err} against {bounds}"


def run_steps(heads, batch, bits, group, residual, tokens, steps, kgain, vgain, policy, rep=1, bound=1e-4, ring=None):
    torch = gh.require_gpu()
    total = tokens + steps
    flush = kivi.KIVI_FLUSH_ALG1 if policy == "alg1" else kivi.KIVI_FLUSH_WINDOW
    w = scaled(CONFIGS["llama7b"], name="onehead", batch=batch, n_q_heads=heads * rep, n_kv_heads=heads, bits=bits, group=group,
               residual=residual, seed=17 * heads + bits + tokens)
    print(f"case one head {policy} h={heads}x{rep} b={batch} B={bits} G={group} R={residual} L={tokens}+{steps} gains {kgain} {vgain}", flush=True)
    k = (workloads.keys(w, total).astype(np.float32) * kgain).astype(np.float16)
    v = (workloads.values(w, total).astype(np.float32) * vgain).astype(np.float16)
    scale = float(np.abs(v.astype(np.float32)).max())
    at = sorted({(0, 0), (batch - 1, heads - 1), (batch // 2, heads // 2)})
    oc = gh.oracle_cache_for_heads(w, k[:, :, :tokens], v[:, :, :tokens], at, policy)
    layout, cache = gh.gpu_prefill(w, k[:, :, :tokens], v[:, :, :tokens], flush, kivi.KIVI_DECODE_AUTO, extra_q_tokens=steps, ring=ring, zero=True)
    _, other = gh.gpu_prefill(w, k[:, :, :tokens], v[:, :, :tokens], flush, kivi.KIVI_DECODE_VALU, extra_q_tokens=steps, ring=ring, zero=True)
    size = cache.workspace.numel()
    room = torch.full((size + 65536,), 0x5A, dtype=torch.uint8, device="cuda")      # nothing is written past the workspace
    cache.workspace = room[:size].zero_()
    for step in range(steps):
        q = (workloads.queries(w, step).astype(np.float32) / kgain).clip(-60000, 60000).astype(np.float16)     # logits of ordinary size
        new = [np.ascontiguousarray(x[:, :, tokens + step]) for x in (k, v)]
        kn, vn, qt = [torch.from_numpy(x).cuda() for x in (*new, q)]
        out = torch.full((batch, heads * rep, 128), float("nan"), dtype=torch.float32, device="cuda")
        kivi.kivi_decode_step(layout, cache, kn, vn, qt, w.softmax_scale, out, flush)
        oc.append(np.stack([k[b, h, tokens + step] for b, h in at])[:, None], np.stack([v[b, h, tokens + step] for b, h in at])[:, None])
        ref = gh.oracle_attention_for_heads(w, oc, q, at)
        got = out.cpu().numpy()
        err = np.abs(gh.pick_heads(got, w, at) - ref).max()
        assert err <= bound * scale, f"step {step}: {err:.3e} against {bound * scale:.3e}"
        ref_all = torch.empty_like(out)        # all heads: the vector path on a cache of its own
        kivi.kivi_decode_step(other.layout, other, kn, vn, qt, w.softmax_scale, ref_all, flush)
        gh.check_close(got / scale, ref_all.cpu().numpy() / scale, f"step {step}, all heads")
    gh.compare_quantized_state(cache, oc, at)
    for name, buf in cache.buffers.items():            # all heads; the vector path's cache had a flush and an append of its own
        assert torch.equal(buf, other.buffers[name]), name
    assert (room[size:] == 0x5A).all()
