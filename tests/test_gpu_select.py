"""Selection of the support: what is counted and kept around it."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_gpu_ctx
from paper_2501_02379_amd import synth, tgrad as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,ranks", [
    ((16, 16, 8, 5), (8, 8, 4, 3)),                        # the first digit picked by every workgroup that needs it
    ((128, 128, 32, 33), (128, 128, 32, 33)),              # ... by a launch of its own (17.3 M numbers; no Gram of them)
])
def test_check_counts_nan_of_either_sign(shape, ranks):
    """A NaN keeps its sign bit in |g|^2 (an x86 processor makes negative ones), and with it the top bit of its key."""
    print("[case] check", shape, flush=True)
    g = synth.small_case(shape, 32).copy()
    bits = g.reshape(-1).view(np.uint32)                   # (re, im) of element e at 2 e, 2 e + 1
    bits[[10, 101, 2000]] = 0xFFC00000                     # negative quiet NaN
    bits[500] = 0xFFFFFFFF
    bits[[700, 901]] = 0x7FC00000
    bits[3000] = 0xFF800000                                # -inf: its square is +inf
    ctx = make_gpu_ctx(T, shape, ranks, 103, refresh_every=0)
    for _ in range(2):
        ctx.tgrad_refresh_factors(T.to_device_grad(g))
        assert ctx.tgrad_check() == 7
    ctx.tgrad_destroy()
