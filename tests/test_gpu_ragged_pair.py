"""Batches of different lengths: the first launch (fp16 rows, flush, tables; one query head per kv-head: flush and tables)
and the second against the run-by-run vector path, which has kernels of its own for all of it."""
import pytest

import gpu_harness as gh
from paper_2402_02750_amd import kivi

pytestmark = pytest.mark.gpu

# (query heads, kv-heads, bits, G, R, tokens of every sequence, steps, launches)
LONG = [31, 64, 95, 96, 127, 128, 159, 222, 223, 1000, 4127]
CASES = [
    (8, 2, 2, 32, 64, LONG, 70, 2),                     # every sequence flushes twice, the rings (96 slots) wrap
    (24, 4, 4, 32, 64, LONG, 70, 2),                    # six heads, 4 bits
    (3, 1, 2, 32, 0, [40, 33, 500], 3, None),           # no window: the flush takes the new token itself
    (4, 2, 2, 64, 128, [191, 500, 64, 1900], 66, 2),    # two heads, G = 64
    (12, 2, 4, 128, 128, [300, 255, 1, 2500], 3, 2),    # six heads, G = 128; a sequence without quantised tokens
    (8, 1, 2, 64, 192, [333, 3000], 3, 2),              # eight heads, seven tiles of rows
    (10, 1, 2, 32, 96, [127, 700], 3, 4),               # ten heads: a pair of launches per eight
    (17, 1, 4, 32, 96, [127, 700, 64], 34, 2),          # seventeen: runs of eight as units, the rows in two
    (71, 1, 2, 64, 128, [900, 191], 3, 2),
    (128, 1, 2, 32, 64, [400, 95], 2, 2),
    (9, 3, 2, 32, 480, [520, 600, 2000], 3, 2),         # a window of sixteen tiles
    (6, 2, 4, 32, 32, [63 + i for i in range(192)], 2, 2),      # as many sequences as the arguments hold: flushes among them
    (6, 2, 2, 32, 32, [63 + i for i in range(193)], 2, 2),      # one more
    (4, 2, 2, 32, 64, LONG, 70, 2),                     # two heads
    (2, 2, 2, 32, 64, LONG, 70, 2),                     # one head: several workgroups per unit
    (3, 3, 4, 32, 64, LONG, 70, 2),
    (40, 40, 2, 32, 64, [64 + 67 * i for i in range(24)], 33, 2),       # ... whole units, the longest in parts
    (40, 40, 4, 32, 64, [4100, 64, 95, 100, 3000] + [200] * 20, 33, 2),
    (2, 2, 2, 64, 128, [191, 500, 64, 1900], 66, 2),
    (26, 26, 2, 32, 64, [8000 - 190 * i for i in range(7)], 2, 2),      # nearly one length: 182 units, four parts each
    (53, 53, 4, 32, 64, [6400 - 190 * i for i in range(5)], 2, 2),      # ... 265 units, five
    (1, 1, 4, 128, 128, [300, 255, 1, 2500, 20000], 3, 2),
    (2, 2, 2, 32, 480, [520, 600, 2000], 3, 2),         # a window of sixteen tiles
    (1, 1, 2, 32, 32, [63 + i for i in range(192)], 2, 2),
    (1, 1, 4, 32, 32, [63 + i for i in range(193)], 2, 1),      # counters copied, no first launch; two levels of the search
    (1, 1, 2, 32, 32, [40 + 7 * (i % 97) for i in range(500)], 2, 1),   # the copy in two pieces
    (2, 1, 2, 32, 32, [40 + 7 * (i % 97) for i in range(500)], 2, 2),   # the tables made out of copied counters
    (8, 2, 4, 64, 64, [70 + 9 * (i % 59) for i in range(250)], 2, 2),
    (10, 1, 2, 32, 64, [70 + 9 * (i % 59) for i in range(250)], 2, 4),
    (17, 1, 2, 32, 64, [70 + 9 * (i % 59) for i in range(200)], 2, 2),
    (32, 1, 2, 64, 64, [700] * 97, 66, 2),              # all alike, too many units for one call
]


@pytest.mark.parametrize("hq,hkv,bits,group,residual,tokens,steps,launches", CASES)
def test_pair(hq, hkv, bits, group, residual, tokens, steps, launches):
    """Outputs within the repository's tolerance, every byte of the cache the same."""
    torch = gh.require_gpu()
    print(f"case ragged pair hq={hq} hkv={hkv} bits={bits} G={group} R={residual} {len(tokens)} sequences", flush=True)
    batch, total = len(tokens), max(tokens) + steps
    gen = torch.Generator(device="cuda").manual_seed(hq + bits)
    k, v = (torch.randn(batch, hkv, total, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    k[..., 7] *= 9
    at = {}
    for path in (kivi.KIVI_DECODE_AUTO, kivi.KIVI_DECODE_VALU):
        layout = kivi.make_layout(batch, hq, hkv, bits, residual, gh.round_up(total, group), gh.round_up(residual + group, 32), group=group,
                                  decode_path=path)
        cache = kivi.Cache(layout)
        for buf in cache.buffers.values():
            buf.zero_()
        states = kivi.make_states(batch)
        for b, n in enumerate(tokens):
            part = kivi.CacheSlice(cache, b, 1)
            kivi.kivi_prefill(part.layout, k[b:b + 1], v[b:b + 1], n, part)
            states[b] = part.state()
        at[path] = layout, cache, states
    for step in range(steps):
        rows = torch.tensor([n + step for n in tokens], device="cuda")
        new = [x[torch.arange(batch, device="cuda"), :, rows].contiguous() for x in (k, v)]
        q = torch.randn(batch, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
        outs = []
        for layout, cache, states in at.values():
            out = torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda")
            kivi.kivi_decode_step_ragged(layout, cache, states, *new, q, 128 ** -0.5, out)
            outs.append(out)
        torch.cuda.synchronize()
        gh.check_close(outs[0].cpu().numpy(), outs[1].cpu().numpy(), f"step {step}")
        (l0, c0, s0), (_, c1, s1) = at.values()
        assert bytes(s0) == bytes(s1), f"step {step}"
        for name in c0.buffers:
            assert torch.equal(c0.buffers[name], c1.buffers[name]), f"step {step}: {name}"
        if launches:
            assert kivi.kivi_decode_launches_ragged(l0, s0) == launches


@pytest.mark.parametrize("hq,hkv,bits,group,more", [
    (9, 1, 2, 64, 1), (32, 2, 4, 128, 5), (24, 2, 2, 64, 200)])        # `more` groups: the last case has three runs, 13 000 tokens in one
def test_few_runs_of_wide_groups(hq, hkv, bits, group, more):
    """G > 32, 9 to 16 heads, two or three runs of equal sequences: kivi_decode_step's own outputs and bytes for each."""
    torch = gh.require_gpu()
    print(f"case ragged, few runs hq={hq} hkv={hkv} bits={bits} G={group}", flush=True)
    short = 128 + 3 * group - 2
    runs = [(2, short), (1, short + more * group)] + ([(1, short)] if more == 200 else [])
    batch, total, steps = sum(n for n, _ in runs), max(t for _, t in runs) + 5, 5
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(batch, hkv, total, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    layout = kivi.make_layout(batch, hq, hkv, bits, 128, gh.round_up(total, group), 128 + group, group=group)
    ragged, states, parts, at = kivi.Cache(layout), kivi.make_states(batch), [], 0
    for buf in ragged.buffers.values():
        buf.zero_()
    for n, tokens in runs:
        sub = kivi.make_layout(n, hq, hkv, bits, 128, layout.cap_q_tokens, layout.cap_r_tokens, group=group)
        own, rows = kivi.Cache(sub), slice(at, at + n)
        for buf in own.buffers.values():
            buf.zero_()
        part = kivi.CacheSlice(ragged, at, n)
        kivi.kivi_prefill(part.layout, k[rows], v[rows], tokens, part)
        kivi.kivi_prefill(sub, k[rows], v[rows], tokens, own)
        for b in range(at, at + n):
            states[b] = part.state()
        parts.append((sub, own, rows, tokens))
        at += n
    assert kivi.kivi_decode_launches_ragged(layout, states) == len(runs)
    for step in range(steps):
        new = [torch.cat([x[r, :, t + step] for _, _, r, t in parts]).contiguous() for x in (k, v)]
        q = torch.randn(batch, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
        outs = [torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
        kivi.kivi_decode_step_ragged(layout, ragged, states, *new, q, 128 ** -0.5, outs[0])
        for sub, own, r, _ in parts:
            kivi.kivi_decode_step(sub, own, new[0][r], new[1][r], q[r], 128 ** -0.5, outs[1][r])
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1]), f"step {step}"
        for name in ragged.buffers:
            whole = ragged.view(name)
            for _, own, r, _ in parts:
                assert torch.equal(whole[r], own.view(name)), f"step {step}: {name}"


@pytest.mark.parametrize("hq,hkv,bits,group", [(2, 2, 2, 64), (4, 2, 4, 128), (8, 1, 2, 64), (17, 1, 4, 64)])
def test_large_groups_alike(hq, hkv, bits, group):
    """G > 32, sequences all alike: kivi_decode_step's own outputs and bytes, over steps with and without a flush."""
    torch = gh.require_gpu()
    print(f"case ragged, all alike hq={hq} hkv={hkv} bits={bits} G={group}", flush=True)
    batch, tokens, steps = 3, 128 + 3 * group - 2, 5
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(batch, hkv, tokens + steps, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    layout = kivi.make_layout(batch, hq, hkv, bits, 128, gh.round_up(tokens + steps, group), 128 + group, group=group)
    uniform, ragged, states = kivi.Cache(layout), kivi.Cache(layout), kivi.make_states(batch)
    for cache in (uniform, ragged):
        for buf in cache.buffers.values():
            buf.zero_()
        kivi.kivi_prefill(layout, k, v, tokens, cache)
    for b in range(batch):
        states[b] = kivi.CacheSlice(ragged, b, 1).state()
    for step in range(steps):
        new = [x[:, :, tokens + step].contiguous() for x in (k, v)]
        q = torch.randn(batch, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
        outs = [torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
        kivi.kivi_decode_step(layout, uniform, *new, q, 128 ** -0.5, outs[0])
        kivi.kivi_decode_step_ragged(layout, ragged, states, *new, q, 128 ** -0.5, outs[1])
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1]), f"step {step}"
        for name in uniform.buffers:
            assert torch.equal(uniform.buffers[name], ragged.buffers[name]), f"step {step}: {name}"
    assert all(s.n_kq == uniform.c.n_kq for s in states) and uniform.c.n_kq > 2 * group


@pytest.mark.parametrize("hq,hkv", [(2, 2), (4, 2), (8, 2), (8, 1), (17, 1)])
@pytest.mark.parametrize("ragged", [True, False])
@pytest.mark.parametrize("rows", [1, 33])
def test_row_without_weight(hq, hkv, ragged, rows):
    """A tile of fp16 rows whose logits are all -inf (one token, a key of -inf; alone or after another tile) counts for nothing in the
    launch of the rows: the output of a key whose probability underflows to 0."""
    torch = gh.require_gpu()
    print(f"case row without weight hq={hq} hkv={hkv} ragged={ragged} rows={rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(2, hkv, 224, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    q = torch.randn(2, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
    q[..., 3] = 1 + q[..., 3].abs()
    path = kivi.KIVI_DECODE_AUTO if ragged else kivi.KIVI_DECODE_MFMA_TWO
    layout = kivi.make_layout(2, hq, hkv, 2, 32, 224, 64, decode_path=path)
    cache, states, outs = kivi.Cache(layout), kivi.make_states(2), []
    for buf in cache.buffers.values():
        buf.zero_()
    kivi.kivi_prefill(layout, k, v, 224, cache)
    for name in ("k_resid", "v_resid"):
        cache.view(name).normal_(generator=gen)
    for row in (-60000.0, float("-inf")):
        cache.view("k_resid")[:, :, rows - 1] = 1
        cache.view("k_resid")[:, :, rows - 1, 3] = row
        outs.append(torch.full((2, hq, 128), float("nan"), dtype=torch.float32, device="cuda"))
        if ragged:
            for b, n in enumerate((160, 192)):
                states[b] = kivi.kivi_seq_state_t(n, n, 0, rows, 0, rows)
            kivi.kivi_decode_attention_ragged(layout, cache, states, q, 128 ** -0.5, outs[-1])
        else:
            c = cache.c
            c.n_kq = c.n_vq = 192
            c.n_kr = c.n_vr = rows
            c.k_r_start = c.v_r_start = 0
            kivi.kivi_decode_attention(layout, cache, q, 128 ** -0.5, outs[-1])
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("batch", [4096, 4097])
@pytest.mark.parametrize("hq", [1, 2, 4])
def test_many_sequences(hq, batch):
    """As many sequences as the first launch makes tables for, and one more: attention against the vector path."""
    torch = gh.require_gpu()
    print(f"case many sequences hq={hq} B={batch}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(batch, 1, 224, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    q = torch.randn(batch, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
    outs = []
    for path in (kivi.KIVI_DECODE_AUTO, kivi.KIVI_DECODE_VALU):
        layout = kivi.make_layout(batch, hq, 1, 2, 32, 224, 64, decode_path=path)
        cache, states = kivi.Cache(layout), kivi.make_states(batch)
        kivi.kivi_prefill(layout, k, v, 224, cache)
        for b in range(batch):                  # what is there of a sequence differs from its neighbours'
            n_q, n_r = 32 * (b * 5 % 7), 1 + b * 3 % 32
            states[b] = kivi.kivi_seq_state_t(n_q, n_q, 0, n_r, 0, n_r)
        outs.append(torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda"))
        kivi.kivi_decode_attention_ragged(layout, cache, states, q, 128 ** -0.5, outs[-1])
    torch.cuda.synchronize()
    assert kivi.kivi_decode_launches_ragged(kivi.make_layout(batch, hq, 1, 2, 32, 224, 64), states) == (1 if hq == 1 else 2)
    gh.check_close(outs[0].cpu().numpy(), outs[1].cpu().numpy())


@pytest.mark.parametrize("hq,hkv", [(16, 4), (4, 4)])
def test_pair_is_deterministic(hq, hkv):
    """The same step on copies of one cache: the same bytes (sums in the same order, whichever workgroup comes last)."""
    torch = gh.require_gpu()
    print(f"case ragged pair: repetitions hq={hq} hkv={hkv}", flush=True)
    tokens = [95, 700, 223, 3000, 5000]
    gen = torch.Generator(device="cuda").manual_seed(5)
    k, v = (torch.randn(5, hkv, max(tokens) + 1, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    q, kn, vn = (torch.randn(5, h, 128, dtype=torch.float16, device="cuda", generator=gen) for h in (hq, hkv, hkv))
    layout = kivi.make_layout(5, hq, hkv, 2, 64, 5024, 96)
    outs = []
    for _ in range(6):
        cache, states = kivi.Cache(layout), kivi.make_states(5)
        for b, n in enumerate(tokens):
            part = kivi.CacheSlice(cache, b, 1)
            kivi.kivi_prefill(part.layout, k[b:b + 1], v[b:b + 1], n, part)
            states[b] = part.state()
        outs.append(torch.empty(5, hq, 128, dtype=torch.float32, device="cuda"))
        kivi.kivi_decode_step_ragged(layout, cache, states, kn, vn, q, 128 ** -0.5, outs[-1])
    torch.cuda.synchronize()
    assert all(torch.equal(outs[0], o) for o in outs[1:])


@pytest.mark.parametrize("hq,hkv,batch,bits,group,residual,tokens", [
    (3, 1, 3, 2, 32, 32, 95),           # one tile quantised in the first step; windows of one and two tiles
    (8, 2, 2, 4, 32, 128, 700),         # four heads
    (40, 8, 5, 2, 32, 64, 1055),        # five: the flush rides too
    (16, 2, 2, 4, 32, 160, 2000),       # eight heads, six tiles of rows
    (24, 2, 2, 2, 32, 64, 300),         # twelve: two pairs of launches, the first flushes and appends
    (10, 2, 2, 2, 64, 128, 800),        # G = 64: a launch for the flush
])
def test_one_length_in_two_launches(hq, hkv, batch, bits, group, residual, tokens):
    """A batch of one length whose fp16 rows (and flush) have a launch of their own: 40 steps against the vector path; outputs within
    the repository's tolerance, every byte of the cache the same."""
    torch = gh.require_gpu()
    print(f"case one length, two launches hq={hq} hkv={hkv} bits={bits} G={group} R={residual} L={tokens}", flush=True)
    steps = 40
    gen = torch.Generator(device="cuda").manual_seed(hq)
    k, v = (torch.randn(batch, hkv, tokens + steps, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    caches = []
    for path in (kivi.KIVI_DECODE_MFMA_TWO, kivi.KIVI_DECODE_VALU):
        layout = kivi.make_layout(batch, hq, hkv, bits, residual, gh.round_up(tokens + steps, group), gh.round_up(residual + group, 32), group=group,
                                  decode_path=path)
        cache = kivi.Cache(layout)
        for buf in cache.buffers.values():
            buf.zero_()
        kivi.kivi_prefill(layout, k, v, tokens, cache)
        caches.append((layout, cache))
    for step in range(steps):
        q = torch.randn(batch, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
        new = [x[:, :, tokens + step].contiguous() for x in (k, v)]
        outs = [torch.full((batch, hq, 128), float("nan"), dtype=torch.float32, device="cuda") for _ in caches]
        for (layout, cache), out in zip(caches, outs):
            kivi.kivi_decode_step(layout, cache, *new, q, 128 ** -0.5, out)
        torch.cuda.synchronize()
        gh.check_close(outs[0].cpu().numpy(), outs[1].cpu().numpy(), f"step {step}")
        for name in caches[0][1].buffers:
            assert torch.equal(caches[0][1].buffers[name], caches[1][1].buffers[name]), f"step {step}: {name}"
