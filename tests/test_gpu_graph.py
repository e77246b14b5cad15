"""The decode-attention launch under HIP graph capture: a serving loop replays one captured
launch per layer and step.  The kernel must be capturable as it is (no allocation, no memset
node: its workspace counters return to zero by themselves) and every replay must give what the
eager call gives, also after eager launches on the same workspace in between."""
import numpy as np
import pytest

import gpu_harness as gh
from paper_2402_02750_amd import kivi, workloads
from paper_2402_02750_amd.workloads import CONFIGS, scaled

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("path", [kivi.KIVI_DECODE_VALU, kivi.KIVI_DECODE_MFMA, kivi.KIVI_DECODE_MFMA_TWO], ids=["valu", "mfma", "mfma2"])
def test_replayed_launch_matches_eager(path):
    torch = gh.require_gpu()
    # 2 x 2 units of 6000 tokens: several workgroups per unit, so the cross-workgroup merge and
    # its counters are part of the captured launch
    w = scaled(CONFIGS["mistral_gqa"], name="graph", batch=2, n_q_heads=8, n_kv_heads=2, seed=321)
    length = 6000
    k, v = workloads.keys(w, length), workloads.values(w, length)
    layout, cache = gh.gpu_prefill(w, k, v, kivi.KIVI_FLUSH_WINDOW, path)
    heads = [(0, 0), (1, 1)]
    oc = gh.oracle_cache_for_heads(w, k, v, heads, "window")
    qs = [workloads.queries(w, step) for step in range(4)]
    q_static = torch.from_numpy(qs[0]).cuda()
    out_static = torch.empty(w.batch, w.n_q_heads, 128, dtype=torch.float32, device="cuda")
    out_eager = torch.empty_like(out_static)

    kivi.kivi_decode_attention(layout, cache, q_static, w.softmax_scale, out_eager)     # warm-up outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kivi.kivi_decode_attention(layout, cache, q_static, w.softmax_scale, out_static,
                                   stream=torch.cuda.current_stream())
    for trial, q in enumerate(qs):
        print(f"case graph path={path} replay {trial}", flush=True)
        q_static.copy_(torch.from_numpy(q).cuda())
        graph.replay()
        torch.cuda.synchronize()
        got = out_static.cpu().numpy().copy()
        # eager launch on the same cache and workspace between the replays
        kivi.kivi_decode_attention(layout, cache, q_static, w.softmax_scale, out_eager)
        torch.cuda.synchronize()
        assert np.array_equal(got, out_eager.cpu().numpy()), f"replay {trial} differs from the eager launch"
        gh.check_close(gh.pick_heads(got, w, heads), gh.oracle_attention_for_heads(w, oc, q, heads), f"replay {trial}")


@pytest.mark.parametrize("bits,group,policy,tokens", [
    (2, 32, kivi.KIVI_FLUSH_WINDOW, 2047),      # one query head per kv-head: a tile leaves the window in the captured step
    (4, 32, kivi.KIVI_FLUSH_WINDOW, 2047),
    (2, 64, kivi.KIVI_FLUSH_ALG1, 2000),        # ... a value token
])
def test_replayed_flushing_step_matches_eager(bits, group, policy, tokens):
    """A whole step that flushes, captured with one query head per kv-head (one launch with several workgroups per unit): every replay
    gives the eager step's bits, with attention calls on the same workspace in between."""
    torch = gh.require_gpu()
    print(f"case graph flushing step bits={bits} G={group} policy={policy}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(bits + tokens)
    heads, residual = 4, 128
    k, v = (torch.randn(2, heads, tokens + 1, 128, dtype=torch.float16, device="cuda", generator=gen) for _ in range(2))
    q = torch.randn(2, heads, 128, dtype=torch.float16, device="cuda", generator=gen)
    new = [x[:, :, tokens].contiguous() for x in (k, v)]
    layout = kivi.make_layout(2, heads, heads, bits, residual, gh.round_up(tokens + 1, 128), gh.round_up(residual + group, 32), group=group)
    fields = ("n_kq", "n_vq", "k_r_start", "n_kr", "v_r_start", "n_vr")

    def start():
        cache = kivi.Cache(layout)
        for buf in cache.buffers.values():
            buf.zero_()
        kivi.kivi_prefill(layout, k, v, tokens, cache, policy)
        return cache, [getattr(cache.c, f) for f in fields]

    cache, _ = start()
    expected, again, out = (torch.empty(2, heads, 128, dtype=torch.float32, device="cuda") for _ in range(3))
    kivi.kivi_decode_step(layout, cache, *new, q, 128 ** -0.5, expected, policy)        # eager
    torch.cuda.synchronize()
    arrays = {name: buf.clone() for name, buf in cache.buffers.items()}

    cache, before = start()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        kivi.kivi_decode_step(layout, cache, *new, q, 128 ** -0.5, out, policy, stream=torch.cuda.current_stream())
    assert cache.c.n_vq > before[1]
    for replay in range(4):
        out.fill_(float("nan"))
        graph.replay()                                 # (the rings still hold what left the window: a replay flushes it again)
        torch.cuda.synchronize()
        assert torch.equal(out, expected), f"replay {replay}"
        assert all(torch.equal(buf, arrays[name]) for name, buf in cache.buffers.items()), f"replay {replay}"
        kivi.kivi_decode_attention(layout, cache, q, 128 ** -0.5, again)
        torch.cuda.synchronize()
        gh.check_close(again.cpu().numpy(), expected.cpu().numpy(), f"attention after replay {replay}")
