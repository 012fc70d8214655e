"""Selection of the support: what is counted and kept around it."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import make_gpu_ctx
from oracle import tgrad_oracle as O
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


@pytest.mark.parametrize("shape,ranks,rule", [
    ((16, 16, 8, 5), (8, 8, 4, 3), T.TGRAD_SELECT_TOPK_MAG), ((40, 30, 13, 9), (9, 7, 5, 3), T.TGRAD_SELECT_TOPK_MAG),
    ((40, 30, 13, 9), (9, 7, 5, 3), T.TGRAD_SELECT_RANDOM), ((20, 16, 36, 20), (5, 4, 34, 18), T.TGRAD_SELECT_TOPK_MAG)])
def test_refresh_reads_nothing_that_an_earlier_call_left(shape, ranks, rule):
    """Refreshing at every step, a context may find anything in its workspace: another one's scratch, or a fill."""
    import torch
    print("[case] workspace", shape, rule, flush=True)
    k = int(np.prod(shape)) // 50
    kw = dict(refresh_every=1, lr=2e-3, select_rule=rule, select_seed=5)
    ctx, ref = (make_gpu_ctx(T, shape, ranks, k, **kw) for _ in range(2))
    W0 = synth.small_case(shape, 40) * np.float32(0.02)
    w, wref = T.to_device_weight(W0), T.to_device_weight(W0)
    rng = np.random.default_rng(6)
    for t, fill in enumerate((0x00, 0xFF, 0x01, None, 0x7F)):
        g = T.to_device_grad(synth.small_case(shape, 50 + t, outlier_frac=(1, 100)))
        if fill is None:
            ctx.ws_buf.copy_(torch.from_numpy(rng.integers(0, 256, ctx.ws_buf.numel(), dtype=np.uint8)))
        else:
            ctx.ws_buf.fill_(fill)
        ctx.tgrad_step(w, g)
        ref.tgrad_step(wref, g)
        assert np.array_equal(ctx.tgrad_get_state(T.STATE_INDICES), ref.tgrad_get_state(T.STATE_INDICES)), fill
        assert torch.equal(ctx.state_buf, ref.state_buf) and torch.equal(w, wref), fill
    ctx.tgrad_destroy()
    ref.tgrad_destroy()


def test_support_where_a_wavefront_walks_the_longest_run():
    """143 M numbers: runs of 1024 words of the masks, more of them than the 4224 that shorter runs are limited to; keys of
    bf16 numbers, so that entries equal to the last one taken are many."""
    import torch
    shape, ranks = (256, 256, 64, 34), (256, 256, 2, 2)
    print("[case] long runs", shape, flush=True)
    k = 100_003
    g = torch.randn(shape + (2,), generator=torch.Generator(device="cuda:0").manual_seed(3), device="cuda:0").bfloat16()
    ctx = make_gpu_ctx(T, shape, ranks, k, grad_dtype=T.TGRAD_CBF16, refresh_every=0)
    ctx.tgrad_refresh_factors(g)
    got = torch.from_numpy(ctx.tgrad_get_state(T.STATE_INDICES)).to("cuda:0")
    ctx.tgrad_destroy()
    del ctx
    re, im = g.view(-1, 2).unbind(1)
    key = re.float().square_()
    key += im.float().square_()
    least = key.topk(k).values[-1]
    above = (key > least).nonzero().reshape(-1)
    equal = (key == least).nonzero().reshape(-1)
    assert equal.numel() > k - above.numel() > 0           # (a tie that the lower index decides)
    want = torch.cat((above, equal[:k - above.numel()])).sort().values
    assert torch.equal(got, want)


@pytest.mark.parametrize("shape", [(16, 16, 8, 5), (31, 24, 5, 9)])
def test_equal_keys_go_by_index(shape):
    """Numbers on a circle whose |g|^2 = fl(fl(re re) + fl(im im)) is the same float32: with the first square unrounded it is not."""
    print("[case] equal keys", shape, flush=True)
    rng = np.random.default_rng(17)
    n = int(np.prod(shape))
    a = rng.uniform(0, 2 * np.pi, 40 * n)
    z = (np.sqrt(2.4) * np.exp(1j * a)).astype(np.complex64)
    key = O.selection_key(z)
    z = z[key == np.float32(2.4)][:n]
    assert z.size == n
    fused = (z.real.astype(np.float64) ** 2 + np.multiply(z.imag, z.imag, dtype=np.float32)).astype(np.float32)
    assert np.unique(fused).size > 1
    ctx = make_gpu_ctx(T, shape, shape, n // 3, refresh_every=0)
    ctx.tgrad_refresh_factors(T.to_device_grad(z.reshape(shape)))
    assert np.array_equal(ctx.tgrad_get_state(T.STATE_INDICES), np.arange(n // 3))
    ctx.tgrad_destroy()


def test_last_entry_of_many():
    """8 M numbers, 800 979 of them in the support, the last two with one key between them: the lower index has it."""
    shape = (59, 59, 59, 39)
    print("[case] last entry", shape, flush=True)
    g = synth.small_case(shape, 710, outlier_frac=(1, 100))
    k = int(np.ceil(0.1 * g.size))
    ctx = make_gpu_ctx(T, shape, (2, 2, 2, 2), k, refresh_every=0)
    ctx.tgrad_refresh_factors(T.to_device_grad(g))
    assert np.array_equal(ctx.tgrad_get_state(T.STATE_INDICES), O.sparse_indices(g, k))
    ctx.tgrad_destroy()
