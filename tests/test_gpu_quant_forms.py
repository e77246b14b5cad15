"""The one-launch prefill and the flush against the separate quantise entry points, byte for byte:
both token orders, prompts that end inside tiles, both policies (values that do not fill their last tile), rings
at every kind of start, and the group sizes that keep the general forms."""
import numpy as np
import pytest

import gpu_harness as gh
from paper_2402_02750_amd import kivi, workloads
from paper_2402_02750_amd.workloads import CONFIGS, scaled

pytestmark = pytest.mark.gpu
W, A = kivi.KIVI_FLUSH_WINDOW, kivi.KIVI_FLUSH_ALG1


def _bytes(cache, names):
    return {n: cache.buffers[n].cpu().numpy().tobytes() for n in names}


def _zeroed(layout):
    cache = kivi.Cache(layout)
    for buf in cache.buffers.values():
        buf.zero_()
    return cache


PACKED = ("k_codes", "k_scale", "k_zero", "v_codes", "v_scale", "v_zero")


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("policy", [W, A], ids=["window", "alg1"])
@pytest.mark.parametrize("order", ["bhtd", "bthd"])
@pytest.mark.parametrize("batch,heads,tokens,group", [(1, 1, 64, 32), (2, 3, 65, 32), (1, 2, 160, 32), (2, 2, 421, 32), (1, 1, 2085, 32), (1, 2, 421, 64)])
def test_prefill(batch, heads, tokens, group, order, policy, bits):
    torch = gh.require_gpu()
    print(f"case prefill B={batch} H={heads} L={tokens} G={group} {order} policy={policy} bits={bits}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(tokens + bits)
    shape = (batch, heads, tokens, 128) if order == "bhtd" else (batch, tokens, heads, 128)
    k, v = (torch.randn(shape, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    k[..., 7] *= 12
    if order == "bthd":
        k, v = k.transpose(1, 2), v.transpose(1, 2)
    residual = max(group, 32)
    layout = kivi.make_layout(batch, heads, heads, bits, residual, gh.round_up(tokens, group), gh.round_up(residual + group, 32), group=group)
    one, parts = _zeroed(layout), _zeroed(layout)
    kivi.kivi_prefill(layout, k, v, tokens, one, policy)
    nk, nv = one.c.n_kq, one.c.n_vq
    if nk:
        kivi.kivi_quantize_key_groups(layout, k, nk, parts)
    if nv:
        kivi.kivi_quantize_value_tokens(layout, v, nv, parts)
    torch.cuda.synchronize()
    assert _bytes(one, PACKED) == _bytes(parts, PACKED)
    assert torch.equal(one.view("k_resid")[:, :, :tokens - nk], k[:, :, nk:])
    assert torch.equal(one.view("v_resid")[:, :, :tokens - nv], v[:, :, nv:])


@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("batch,heads,group", [(1, 1, 32), (3, 5, 32), (1, 2, 64), (149, 3, 32), (128, 7, 32), (299, 3, 32)])
def test_flush(batch, heads, group, bits):
    """A step's flush out of rings whose oldest row is at slot 0, 32, 64, ... (wrapping): the packed arrays equal
    those of one pass over the whole prompt.  Few units (a workgroup per tile) and many (a wavefront each; from 448 on, at 4 bits from
    896 on)."""
    torch = gh.require_gpu()
    print(f"case flush B={batch} H={heads} G={group} bits={bits}", flush=True)
    residual = max(group, 32)
    start, steps = residual + 3, 4 * group
    total = start + steps
    gen = torch.Generator(device="cuda").manual_seed(7 * batch + bits)
    k, v = (torch.randn(batch, heads, total, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    layout = kivi.make_layout(batch, heads, heads, bits, residual, gh.round_up(total, group), gh.round_up(residual + group, 32), group=group)
    stepped, whole = _zeroed(layout), _zeroed(layout)
    kivi.kivi_prefill(layout, k, v, start, stepped, W)
    flushes = 0
    for t in range(start, total):
        kivi.kivi_append_residual(layout, stepped, k[:, :, t].contiguous(), v[:, :, t].contiguous())
        flushes += kivi.kivi_flush_residual(layout, stepped, W)[0] > 0
    kivi.kivi_quantize_key_groups(layout, k, stepped.c.n_kq, whole)
    kivi.kivi_quantize_value_tokens(layout, v, stepped.c.n_vq, whole)
    torch.cuda.synchronize()
    assert flushes == 4
    assert _bytes(stepped, PACKED) == _bytes(whole, PACKED)


@pytest.mark.parametrize("batch,hq,hkv,tokens,residual,bits", [
    (1, 4, 4, 63, 32, 2),           # the first flush: nothing was quantised before
    (1, 4, 2, 1023, 32, 4),         # two heads per kv-head, few units
    (2, 3, 3, 4095, 128, 2),
    (1, 2, 1, 1024 + 479 + 32, 480, 2),     # fifteen tiles of fp16 rows after the flush
    (24, 16, 8, 1055, 128, 2),      # two heads, 192 and 320 units: the tile kernel's only launch carries the flush
    (40, 16, 8, 1023, 128, 4),
    (49, 16, 8, 1055, 128, 2),      # 392 units, or 384 and 40 000 tiles: the rows' launch carries it
    (49, 16, 8, 1055, 128, 4),
    (48, 16, 8, 3359, 128, 2),
    (24, 64, 8, 1055, 128, 2),      # eight heads, one launch
    (64, 32, 8, 1055, 128, 4),      # four heads: the rows' launch carries the flush for the tile kernel
    (64, 32, 8, 1024 + 479 + 32, 480, 2),   # sixteen tiles of rows for four heads: the most that such a launch takes
    (64, 24, 8, 1023, 32, 2),       # three of four slots, one tile of fp16 rows
    (64, 24, 8, 1023, 96, 4),       # two tiles
])
def test_flush_step(batch, hq, hkv, tokens, residual, bits):
    """A step that flushes, by the automatic choice and in the single-launch form, against append, flush and attention as calls of
    their own.  Cache arrays equal byte for byte; outputs as far apart as two launch forms of one attention."""
    torch = gh.require_gpu()
    print(f"case flush step B={batch} heads {hq}/{hkv} L={tokens} R={residual} bits={bits}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(tokens + bits)
    k, v = (torch.randn(batch, hkv, tokens + 1, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    q = torch.randn(batch, hq, 128, dtype=torch.float16, device="cuda", generator=gen)
    new = [x[:, :, tokens].contiguous() for x in (k, v)]
    caches, outs = [], []
    for apart, path in ((True, kivi.KIVI_DECODE_AUTO), (False, kivi.KIVI_DECODE_AUTO), (False, kivi.KIVI_DECODE_MFMA_ONE)):
        layout = kivi.make_layout(batch, hq, hkv, bits, residual, gh.round_up(tokens + 1, 32), gh.round_up(residual + 32, 32), decode_path=path)
        cache, out = _zeroed(layout), torch.empty(batch, hq, 128, dtype=torch.float32, device="cuda")
        kivi.kivi_prefill(layout, k, v, tokens, cache, W)
        before = cache.c.n_kq
        if apart:
            kivi.kivi_append_residual(layout, cache, *new)
            kivi.kivi_flush_residual(layout, cache, W)
            kivi.kivi_decode_attention(layout, cache, q, 128 ** -0.5, out)
        else:
            kivi.kivi_decode_step(layout, cache, *new, q, 128 ** -0.5, out, W)
        torch.cuda.synchronize()
        assert cache.c.n_kq == before + 32
        caches.append(cache)
        outs.append(out.cpu().numpy())
    for cache, out, what in zip(caches[1:], outs[1:], ("automatic", "one launch")):
        assert _bytes(cache, PACKED + ("k_resid", "v_resid")) == _bytes(caches[0], PACKED + ("k_resid", "v_resid")), what
        gh.check_close(out, outs[0], what)
