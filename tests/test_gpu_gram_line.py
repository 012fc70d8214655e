"""Gram matrices of all modes in one launch of equal parts: whole numbers, so that every sum is exact in any order, on tensors whose
parts begin and end inside modes, with fewer tiles than workgroups, modes of all kernel variants and modes of more than 128 entries
(a launch each) among them."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_gpu_ctx
from oracle import tgrad_oracle as O
from paper_2501_02379_amd import tgrad as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["c64", "cbf16"])
@pytest.mark.parametrize("shape,ranks", [
    ((2, 3), (1, 2)), ((17, 33, 65), (2, 3, 4)),                          # a tile per workgroup
    ((34, 33, 20, 9), (5, 33, 6, 2)),                                     # about as many tiles as workgroups; a mode left out
    ((100, 20, 40, 17), (9, 5, 7, 3)), ((128, 17, 33, 65), (5, 4, 3, 2)),
    ((16, 16, 16, 16, 17), (4, 4, 4, 4, 4)), ((5, 3, 4, 2, 6, 7), (2, 2, 2, 1, 3, 3)),
    ((130, 64, 33), (6, 5, 4)), ((17, 200, 150), (3, 4, 5)), ((129, 30), (4, 3)),
    ((127, 96, 48, 30), (4, 5, 6, 7))])                                   # 17.6 M numbers
def test_every_mode_exactly(shape, ranks, dt):
    print("[case] gram line", shape, dt, flush=True)
    rng = np.random.default_rng(len(shape) + shape[0])
    g = (rng.integers(-7, 8, shape) + 1j * rng.integers(-7, 8, shape)).astype(np.complex64)
    k = g.size // 50
    gd = O.complex_to_bf16_pairs(g) if dt == "cbf16" else g
    ctx = make_gpu_ctx(T, shape, ranks, k, refresh_every=0, grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    ctx.tgrad_refresh_factors(T.to_device_grad(gd))
    g.reshape(-1)[ctx.tgrad_get_state(T.STATE_INDICES)] = 0
    for m in range(len(shape)):
        if ranks[m] == shape[m]:
            continue
        a = np.moveaxis(g, m, 0).reshape(shape[m], -1)
        want = np.zeros((shape[m], shape[m]), np.complex128)
        for part in np.array_split(a, max(1, a.shape[1] // 50_000), axis=1):   # (single precision holds 2 x 49 x 50 000 exactly)
            want += part @ part.conj().T
        assert np.array_equal(ctx.tgrad_get_state(T.STATE_GRAM0 + m), want), m
    ctx.tgrad_destroy()
