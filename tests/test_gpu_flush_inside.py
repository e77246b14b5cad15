"""GPU parity of the flush that rides in decode_tiles_kernel's launch: two and more query heads per kv-head, one tile leaving the
window, with windows of few and many tiles, one and several workgroups for the rows, runs of heads that share a kv-head (only
one of them stores), and the first tile there is."""
import pytest

from test_gpu_one_head import run_steps

pytestmark = pytest.mark.gpu

# (kv-heads, query heads per kv-head, batch, bits, residual, prompt tokens, steps)
CASES = [
    (2, 2, 1, 2, 32, 62, 3),            # the first quantised tile, one tile of rows
    (2, 4, 1, 4, 64, 94, 3),
    (2, 3, 2, 2, 128, 1023, 3),         # four tiles of rows beside the flush
    (1, 8, 1, 4, 128, 4095, 3),
    (8, 4, 4, 2, 128, 2047, 2),
    (8, 8, 4, 2, 96, 2047, 2),
    (2, 2, 2, 4, 1024, 3007, 3),        # a large window
    (1, 9, 2, 2, 64, 1055, 3),          # runs of heads
    (1, 71, 2, 2, 128, 511, 3),
    (1, 20, 3, 4, 32, 500, 40),         # two flushes, the ring wraps
    (40, 8, 16, 2, 32, 127, 2),         # many units
]


@pytest.mark.parametrize("heads,rep,batch,bits,residual,tokens,steps", CASES)
def test_flush_inside(heads, rep, batch, bits, residual, tokens, steps):
    """Outputs within the bound of decode_tiles_kernel's arithmetic (see test_one_head); codes, scales and zero-points exactly."""
    run_steps(heads, batch, bits, 32, residual, tokens, steps, 1, 1, "window", rep)
