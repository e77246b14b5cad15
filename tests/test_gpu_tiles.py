"""GPU parity of the matrix-core kernel for several query heads per kv-head, at the sizes where its split can
go wrong: every column layout (2, 4 and 8 heads, with idle columns), partial steps, units cut among several
workgroups, one and two launches, rows and values that end inside a tile, scales outside the ordinary range, sequences
of different lengths."""
import numpy as np
import pytest

import gpu_harness as gh
from paper_2402_02750_amd import kivi, workloads
from paper_2402_02750_amd.workloads import CONFIGS, scaled

pytestmark = pytest.mark.gpu

# (query heads, kv-heads, batch, bits, G, policy, tokens, gain of the keys, gain of the values)
W, A = kivi.KIVI_FLUSH_WINDOW, kivi.KIVI_FLUSH_ALG1
CASES = [
    (4, 2, 1, 2, 32, W, 33, 1, 1),          # one tile quantised at most, one step
    (6, 2, 1, 4, 32, W, 128 + 32 * 5, 1, 1),    # 3 of 4 head slots, a step of one tile after a full one
    (10, 2, 1, 2, 32, A, 777, 1, 1),        # 5 of 8 head slots; values end inside a tile
    (9, 1, 2, 4, 64, W, 2000, 1, 1),        # 9 heads: two runs, the second with one head
    (71, 1, 1, 2, 128, W, 1300, 1, 1),      # nine runs of a single kv-head
    (8, 1, 1, 2, 32, W, 9000, 1, 1),        # one unit in many parts
    (8, 2, 5, 4, 32, A, 2500, 1, 1),        # units cut at uneven places, K and V split differently
    (32, 4, 40, 2, 32, W, 3300, 1, 1),      # two launches, eight heads
    (16, 4, 60, 2, 32, W, 4200, 1, 1),      # two launches, four heads
    (16, 4, 130, 2, 32, A, 901, 1, 1),      # split differently, more units than 512: a launch for the tiles that hold rows
    (32, 4, 129, 4, 64, A, 1000, 1, 1),     # ... eight heads
    (8, 2, 2, 2, 32, W, 900, 60, 1),        # key scales past 64
    (16, 2, 2, 4, 32, A, 900, 60, 500),     # large value scales
    (8, 2, 2, 2, 32, W, 900, 1, 2.0 ** -13),    # value scales among fp16's subnormals
    (16, 2, 2, 4, 32, W, 900, 2.0 ** -10, 1),   # small key scales
]


@pytest.mark.parametrize("hq,hkv,batch,bits,group,policy,tokens,kgain,vgain", CASES)
def test_tiles(hq, hkv, batch, bits, group, policy, tokens, kgain, vgain):
    """Against the oracle and against the vector path.  Tolerance: probabilities and operands keep 21 bits or
    more, fp32 sums of a few thousand terms lose at most 2^-24 of their largest term each; the logits (up to
    about 50 here) carry 2^-20 of themselves into the probabilities: below 1e-4 of the largest value
    together.  The vector path is held to the repository's tolerance on the same numbers."""
    gh.require_gpu()
    w = scaled(CONFIGS["mistral_gqa"], name="tiles", batch=batch, n_q_heads=hq, n_kv_heads=hkv, bits=bits, group=group,
               residual=128, seed=31 * hq + bits)
    print(f"case tiles hq={hq} hkv={hkv} B={batch} bits={bits} G={group} policy={policy} L={tokens} gains {kgain} {vgain}", flush=True)
    k = (workloads.keys(w, tokens).astype(np.float32) * kgain).astype(np.float16)
    v = (workloads.values(w, tokens).astype(np.float32) * vgain).astype(np.float16)
    q = (workloads.queries(w).astype(np.float32) / max(1, kgain)).astype(np.float16)
    heads = [(0, 0), (batch - 1, hkv - 1), (batch // 2, hkv // 2)]
    oc = gh.oracle_cache_for_heads(w, k, v, heads, "window" if policy == W else "alg1")
    ref = gh.oracle_attention_for_heads(w, oc, q, heads)
    scale = float(np.abs(v.astype(np.float32)).max())
    outs = {}
    for path in (kivi.KIVI_DECODE_MFMA, kivi.KIVI_DECODE_MFMA_TWO, kivi.KIVI_DECODE_MFMA_ONE, kivi.KIVI_DECODE_VALU):
        layout, cache = gh.gpu_prefill(w, k, v, policy, path)
        outs[path] = gh.gpu_attention(layout, cache, q, w.softmax_scale)
        got = gh.pick_heads(outs[path], w, heads)
        if path == kivi.KIVI_DECODE_VALU or (hq == 2 * hkv and path == kivi.KIVI_DECODE_MFMA_TWO):
            gh.check_close(got / scale, ref / scale, f"path {path}")
        else:
            err = np.abs(got - ref).max()
            assert err <= 1e-4 * scale, f"path {path}: {err:.3e} against {1e-4 * scale:.3e}"
    # all heads, not only the oracle's: the vector path serves the same cache in its own way
    gh.check_close(outs[kivi.KIVI_DECODE_MFMA] / scale, outs[kivi.KIVI_DECODE_VALU] / scale, "all heads")


@pytest.mark.parametrize("hq,hkv,bits,group,policy", [(4, 2, 2, 32, W), (4, 2, 4, 64, W), (8, 2, 2, 32, W), (6, 2, 4, 32, A), (8, 2, 2, 128, W),
                                                     (16, 2, 2, 32, W)])
def test_small_keys(hq, hkv, bits, group, policy):
    """Key zero-points and scales among fp16's subnormals, and queries large enough for the logits to need them.  Tolerance: the query
    enters times 2^-5 here (its largest element below 2^9), a key operand is exact to 2^-25 (half of fp16's smallest number) in each of
    128 channels, times codes of up to 3 or 15; what that adds up to in a logit moves a probability by as much of itself, and the output by
    that times the values' mean deviation, which is less than the largest value."""
    gh.require_gpu()
    tokens = 1200
    w = scaled(CONFIGS["mistral_gqa"], name="smallkeys", batch=1, n_q_heads=hq, n_kv_heads=hkv, bits=bits, group=group, residual=128, seed=9 * hq + bits)
    print(f"case small keys hq={hq} hkv={hkv} bits={bits} G={group} policy={policy}", flush=True)
    rng = np.random.default_rng(hq + bits + group)
    k = (rng.standard_normal((1, hkv, tokens, 128)) * 2.0 ** -16).astype(np.float16)
    q = np.clip(rng.standard_normal((1, hq, 128)) * 2.0 ** 12, -2.0 ** 13, 2.0 ** 13).astype(np.float16)
    v = workloads.values(w, tokens)
    heads = [(0, h) for h in range(hkv)]
    oc = gh.oracle_cache_for_heads(w, k, v, heads, "window" if policy == W else "alg1")
    assert 0 < np.abs(oc.k_zero.astype(np.float32)).max() < 2.0 ** -13
    ref = gh.oracle_attention_for_heads(w, oc, q, heads)
    bound = 2.0 ** 5 * w.softmax_scale * 128 * 2.0 ** -25 * (2 ** bits - 1) * float(np.abs(v.astype(np.float32)).max())
    oc.k_zero = oc.k_zero * np.float16(0)              # (what flushing them to zero would give)
    assert np.abs(gh.oracle_attention_for_heads(w, oc, q, heads) - ref).max() > 4 * bound
    for path in (kivi.KIVI_DECODE_MFMA, kivi.KIVI_DECODE_MFMA_ONE):
        layout, cache = gh.gpu_prefill(w, k, v, policy, path)
        err = np.abs(gh.pick_heads(gh.gpu_attention(layout, cache, q, w.softmax_scale), w, heads) - ref).max()
        assert err <= bound, f"path {path}: {err:.3e} against {bound:.3e}"


# (query heads, kv-heads, bits, tokens of every sequence)
RAGGED_CASES = [
    (32, 8, 2, [20000]),                        # 157 steps per unit, more than there are rows for parts
    (64, 8, 4, [10000]),                        # the same with the smaller limit of eight heads at 4 bits
    (28, 4, 4, [2600, 2600, 2600, 12800]),      # seven heads, a long sequence last: its units meet the shorter intervals
    (8, 2, 2, [25600, 2000, 2000]),             # ... first
    (12, 4, 4, [700, 40, 4000, 1]),             # three heads; sequences without quantised tokens
    (16, 4, 4, [33, 5000, 129]),                # four heads, last steps of one, two and four tiles
    (10, 1, 2, [900, 900, 15000]),              # ten heads of one kv-head: two pairs of launches
]


@pytest.mark.parametrize("hq,hkv,bits,tokens,group", [c + (32,) for c in RAGGED_CASES] + [
    (4, 2, 2, [3000, 95, 700], 32),             # two heads; a flush in the step
    (4, 2, 4, [1300, 200, 4000], 64),
    (2, 2, 2, [3000, 95, 700], 32),             # one head, several workgroups per unit
    (3, 3, 4, [191, 1300, 5000], 64),
    (2, 2, 2, [2000, 1, 383], 128),
    (8, 2, 2, [191, 1300, 5000], 64),           # four heads
    (16, 2, 4, [2000, 255, 1], 128),            # eight
    (12, 1, 2, [900, 191, 400, 1500], 64),      # twelve: two pairs of launches
    (17, 1, 2, [95, 1300, 3000], 32),           # seventeen: runs of eight as units
    (34, 2, 4, [191, 1300, 700], 64),
])
def test_tiles_ragged(hq, hkv, bits, tokens, group):
    """Sequences of different lengths: a decoding step and an attention call against the oracle (tolerance as in
    test_tiles) and, all heads, against the vector path; nothing is written past the workspace."""
    torch = gh.require_gpu()
    batch, total = len(tokens), max(tokens) + 1
    w = scaled(CONFIGS["mistral_gqa"], name="tilesragged", batch=batch, n_q_heads=hq, n_kv_heads=hkv, bits=bits, group=group,
               residual=max(group, 64), seed=77 * hq + bits)
    print(f"case tiles ragged hq={hq} hkv={hkv} bits={bits} G={group} L={tokens}", flush=True)
    k, v = workloads.keys(w, total), workloads.values(w, total)
    kt, vt = torch.from_numpy(k).cuda(), torch.from_numpy(v).cuda()
    heads = sorted({0, hkv // 2, hkv - 1})
    scale = float(np.abs(v.astype(np.float32)).max())
    outs = {}
    for path in (kivi.KIVI_DECODE_MFMA, kivi.KIVI_DECODE_VALU):
        layout = kivi.make_layout(batch, hq, hkv, bits, w.residual, gh.round_up(total, group), max(128, 2 * group), group=group, decode_path=path)
        cache = kivi.Cache(layout)
        size = cache.workspace.numel()
        room = torch.full((size + 65536,), 0x5A, dtype=torch.uint8, device="cuda")
        cache.workspace = room[:size].zero_()
        states = kivi.make_states(batch)
        for b, n in enumerate(tokens):
            part = kivi.CacheSlice(cache, b, 1)
            kivi.kivi_prefill(part.layout, kt[b:b + 1], vt[b:b + 1], n, part)
            states[b] = part.state()
        new = [torch.stack([x[b, :, n] for b, n in enumerate(tokens)]).contiguous() for x in (kt, vt)]
        results = []
        for step in (0, 1):
            out = torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda")
            q = torch.from_numpy(workloads.queries(w, step)).cuda()
            if step == 0:
                kivi.kivi_decode_step_ragged(layout, cache, states, *new, q, w.softmax_scale, out)
            else:
                kivi.kivi_decode_attention_ragged(layout, cache, states, q, w.softmax_scale, out)
            torch.cuda.synchronize()
            results.append(out.cpu().numpy())
        assert (room[size:] == 0x5A).all()
        outs[path] = results
    got, other = outs[kivi.KIVI_DECODE_MFMA], outs[kivi.KIVI_DECODE_VALU]
    for step in (0, 1):
        gh.check_close(got[step] / scale, other[step] / scale, f"step {step}, all heads")
        q = workloads.queries(w, step)
        for b, n in enumerate(tokens):
            at = [(b, h) for h in heads]
            oc = gh.oracle_cache_for_heads(w, k[:, :, :n], v[:, :, :n], at, "window")
            oc.append(np.stack([k[b, h, n] for b, h in at])[:, None], np.stack([v[b, h, n] for b, h in at])[:, None])
            ref = gh.oracle_attention_for_heads(w, oc, q, at)
            err = np.abs(gh.pick_heads(got[step], w, at) - ref).max()
            assert err <= 1e-4 * scale, f"step {step} sequence {b}: {err:.3e} against {1e-4 * scale:.3e}"


@pytest.mark.parametrize("hq,hkv,bits", [(8, 2, 2), (16, 2, 4), (12, 2, 4), (4, 2, 2), (4, 2, 4), (2, 2, 2), (2, 2, 4)])
def test_tiles_ragged_small_workspace(hq, hkv, bits):
    """A ragged step that flushes, with room for few parts per head: served as with the full workspace from as many rows on
    as the longest sequence has splits, refused before anything is launched below; the attention alone needs two.
    (Tolerance: another cut of the same work adds the same terms, 22 bits each, in another order.)"""
    torch = gh.require_gpu()
    tokens, residual = [479, 300, 95], 64           # the first and the last flush in this step
    batch, total = len(tokens), max(tokens) + 1
    w = scaled(CONFIGS["mistral_gqa"], name="tilesws", batch=batch, n_q_heads=hq, n_kv_heads=hkv, bits=bits, residual=residual, seed=hq)
    kt, vt = torch.from_numpy(workloads.keys(w, total)).cuda(), torch.from_numpy(workloads.values(w, total)).cuda()
    q = torch.from_numpy(workloads.queries(w, 0)).cuda()
    new = [torch.stack([x[b, :, n] for b, n in enumerate(tokens)]).contiguous() for x in (kt, vt)]
    layout = kivi.make_layout(batch, hq, hkv, bits, residual, gh.round_up(total, 32), 96)
    row = batch * hq * 130 * 4
    full = kivi.kivi_decode_workspace_bytes(layout)
    base = full - ((layout.cap_q_tokens // 32 + 3) // 4 + layout.cap_r_tokens // 32 + 2) * row
    tiles_per_split = 16 if bits == 2 or hq <= 2 * hkv else 8
    need = -(-((480 - residual) // 32) // tiles_per_split) + 1
    results = {}
    for rows in (None, 4, 3, 2, 1):
        print(f"case tiles workspace hq={hq} hkv={hkv} bits={bits} rows={rows}", flush=True)
        cache = kivi.Cache(layout)
        size = full if rows is None else base + rows * row
        room = torch.full((full + row,), 0x5A, dtype=torch.uint8, device="cuda")
        cache.workspace = room[:size].zero_()
        for buf in cache.buffers.values():
            buf.zero_()
        states = kivi.make_states(batch)
        for b, n in enumerate(tokens):
            part = kivi.CacheSlice(cache, b, 1)
            kivi.kivi_prefill(part.layout, kt[b:b + 1], vt[b:b + 1], n, part)
            states[b] = part.state()
        before = bytes(states), {n: x.clone() for n, x in cache.buffers.items()}
        outs = [torch.zeros(batch, hq, 128, dtype=torch.float32, device="cuda") for _ in range(2)]
        if rows is not None and rows < need:
            with pytest.raises(kivi.KiviError, match="WORKSPACE"):
                kivi.kivi_decode_step_ragged(layout, cache, states, *new, q, w.softmax_scale, outs[0])
            torch.cuda.synchronize()
            assert bytes(states) == before[0]
            assert all(torch.equal(cache.buffers[n], x) for n, x in before[1].items())
        else:
            kivi.kivi_decode_step_ragged(layout, cache, states, *new, q, w.softmax_scale, outs[0])
            assert [s.n_kq for s in states] == [416, 224, 32]
        if rows is None or rows >= 2:
            kivi.kivi_decode_attention_ragged(layout, cache, states, q, w.softmax_scale, outs[1])
        else:
            with pytest.raises(kivi.KiviError, match="WORKSPACE"):
                kivi.kivi_decode_attention_ragged(layout, cache, states, q, w.softmax_scale, outs[1])
        torch.cuda.synchronize()
        assert (room[size:] == 0x5A).all()
        results[rows] = [o.cpu().numpy() for o in outs]
        if rows is not None and rows >= need:
            for got, ref in zip(results[rows], results[None]):
                assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max(), f"{rows} rows"


@pytest.mark.parametrize("hq,hkv,bits,quantised", [(14, 2, 4, 640), (8, 1, 4, 0), (7, 1, 2, 96)])
def test_tiles_large_window(hq, hkv, bits, quantised):
    """A window of 8192 fp16 tokens and few units: the rows may take no more than half of a unit's parts.  Against the oracle,
    tolerance as in test_tiles."""
    gh.require_gpu()
    w = scaled(CONFIGS["mistral_gqa"], name="tileswindow", batch=1, n_q_heads=hq, n_kv_heads=hkv, bits=bits, residual=8192, seed=5 * hq)
    tokens = 8192 + quantised
    print(f"case tiles window hq={hq} hkv={hkv} bits={bits} L={tokens}", flush=True)
    k, v, q = workloads.keys(w, tokens), workloads.values(w, tokens), workloads.queries(w)
    heads = [(0, h) for h in range(hkv)]
    ref = gh.oracle_attention_for_heads(w, gh.oracle_cache_for_heads(w, k, v, heads, "window"), q, heads)
    scale = float(np.abs(v.astype(np.float32)).max())
    layout, cache = gh.gpu_prefill(w, k, v, W, kivi.KIVI_DECODE_AUTO)
    assert cache.c.n_kq == quantised
    err = np.abs(gh.pick_heads(gh.gpu_attention(layout, cache, q, w.softmax_scale), w, heads) - ref).max()
    assert err <= 1e-4 * scale, f"{err:.3e} against {1e-4 * scale:.3e}"


@pytest.mark.parametrize("path", [kivi.KIVI_DECODE_MFMA, kivi.KIVI_DECODE_MFMA_TWO], ids=["mfma", "mfma2"])
@pytest.mark.parametrize("outlier,size,every", [(40000, 2.0 ** -4, 5000), (1000, 2.0 ** -8, 5000), (40000, 2.0 ** -4, 32), (1000, 2.0 ** -8, 320)])
@pytest.mark.parametrize("hq,hkv,bits,group,policy", [(8, 2, 2, 32, W), (16, 2, 4, 32, W), (6, 2, 2, 32, A), (10, 2, 4, 64, W), (4, 2, 4, 32, W)])
def test_value_outliers(hq, hkv, bits, group, policy, outlier, size, every, path):
    """Tokens with very large values and no probability take no bits from the others.  Tolerance: p (z + s code) of an
    ordinary token keeps 21 bits of p and 22 of the product, and sums add no more than 2^-22 of the largest share:
    2^-20 of the largest ordinary value."""
    gh.require_gpu()
    tokens = 1500
    w = scaled(CONFIGS["mistral_gqa"], name="outliers", batch=1, n_q_heads=hq, n_kv_heads=hkv, bits=bits, group=group, residual=128, seed=3 * hq + bits)
    print(f"case value outliers hq={hq} hkv={hkv} bits={bits} G={group} policy={policy} {outlier} among {size} every {every} path={path}", flush=True)
    k, v, q = workloads.keys(w, tokens), workloads.values(w, tokens), workloads.queries(w)
    q = np.broadcast_to(q[:, :1] * np.float16(0.3), q.shape).copy()          # all heads alike, so that one key suits no head
    v = (v.astype(np.float32) * size).astype(np.float16)
    largest = float(np.abs(v.astype(np.float32)).max())
    for t in range(7, tokens - 128, every):
        k[:, :, t] = -40 * np.sign(q[0, 0].astype(np.float32))
        v[:, :, t] = outlier * np.sign(v[:, :, t].astype(np.float32))
    heads = [(0, h) for h in range(hkv)]
    oc = gh.oracle_cache_for_heads(w, k, v, heads, "window" if policy == W else "alg1")
    ref = gh.oracle_attention_for_heads(w, oc, q, heads)
    layout, cache = gh.gpu_prefill(w, k, v, policy, path)
    err = np.abs(gh.pick_heads(gh.gpu_attention(layout, cache, q, w.softmax_scale), w, heads) - ref).max()
    assert err <= 2.0 ** -20 * largest, f"{err:.3e} against {2.0 ** -20 * largest:.3e}"


@pytest.mark.parametrize("large,small,looks", [(1000, 2.0 ** -5, 0), (1000, 2.0 ** -5, 1), (4000, 2.0 ** -3, 0)])
@pytest.mark.parametrize("hq,hkv,bits,group,policy", [(8, 2, 2, 32, W), (16, 2, 4, 32, W), (6, 2, 2, 32, A), (10, 2, 4, 64, W), (4, 2, 4, 32, W)])
def test_key_outliers(hq, hkv, bits, group, policy, large, small, looks):
    """A key channel 2^15 times larger than the others, at which the queries hardly look, takes no bits from them, also where
    another head of the group looks at it (`looks`).  Tolerance as in test_value_outliers: logits of up to about 4 carry
    2^-22 of their largest product, and fp32's rounding, into the probabilities."""
    gh.require_gpu()
    tokens = 1500
    w = scaled(CONFIGS["mistral_gqa"], name="keyoutliers", batch=1, n_q_heads=hq, n_kv_heads=hkv, bits=bits, group=group, residual=128, seed=5 * hq + bits)
    print(f"case key outliers hq={hq} hkv={hkv} bits={bits} G={group} policy={policy} {large} among {small} looks={looks}", flush=True)
    rng = np.random.default_rng(hq + bits)
    k = (rng.standard_normal((1, hkv, tokens, 128)) * small).astype(np.float16)
    k[..., 5] = (rng.uniform(-1, 1, (1, hkv, tokens)) * large).astype(np.float16)
    v, q = workloads.values(w, tokens), (rng.standard_normal((1, hq, 128)) / small).astype(np.float16)
    q[..., 5] = q[..., 5] * np.float16(small / large)
    if looks:                                           # the first head of every group
        q[:, ::w.q_per_kv, 5] = 0.01
    heads = [(0, h) for h in range(hkv)]
    oc = gh.oracle_cache_for_heads(w, k, v, heads, "window" if policy == W else "alg1")
    ref = gh.oracle_attention_for_heads(w, oc, q, heads)
    layout, cache = gh.gpu_prefill(w, k, v, policy, kivi.KIVI_DECODE_MFMA)
    err = np.abs(gh.pick_heads(gh.gpu_attention(layout, cache, q, w.softmax_scale), w, heads) - ref)
    if looks:
        err = err[:, 1:]                                # (the looking head's probabilities hang on logits of thousands)
    bound = 2.0 ** -20 * float(np.abs(v.astype(np.float32)).max())
    assert err.max() <= bound, f"{err.max():.3e} against {bound:.3e}"


@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("hq,bits", [(1, 2), (1, 4), (2, 2), (4, 4), (7, 2), (8, 4)])
def test_unwritten_scales(hq, bits, group):
    """Values that end inside a tile (Algorithm 1's policy): what the packed arrays hold past them does not count, be it
    zeros or NaN.  Same bytes out."""
    torch = gh.require_gpu()
    print(f"case unwritten scales hq={hq} bits={bits} G={group}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(hq + group)
    for tokens in (256 + 1, 256 + 31, 256 + 77, 256 + 128):
        k, v = (torch.randn(2, 1, tokens, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
        q = torch.randn(2, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
        outs = []
        for fill in (0, 0xFF):
            layout = kivi.make_layout(2, hq, 1, bits, 128, 512, 256, group=group)
            cache = kivi.Cache(layout)
            for buf in cache.buffers.values():
                buf.fill_(fill)
            kivi.kivi_prefill(layout, k, v, tokens, cache, A)
            assert cache.c.n_vq == tokens - 128 and cache.c.n_kq != cache.c.n_vq or tokens == 384
            out = torch.empty(2, hq, 128, dtype=torch.float32, device="cuda")
            kivi.kivi_decode_attention(layout, cache, q, 128 ** -0.5, out)
            torch.cuda.synchronize()
            outs.append(out)
        assert torch.isfinite(outs[1]).all() and torch.equal(outs[0], outs[1]), f"{tokens} tokens"
