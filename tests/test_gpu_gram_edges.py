"""Gram matrices of every mode against float64 sums, at the extents where the kernel variants and their tile rows begin
and end, with the mode first, in the middle and last, and with the support masked."""
import numpy as np
import pytest

from oracle import tgrad_oracle as O
from paper_2501_02379_amd import synth
from paper_2501_02379_amd import tgrad as T
from helpers import make_gpu_ctx

pytestmark = pytest.mark.gpu

EXTENTS = [2, 15, 16, 17, 18, 32, 33, 34, 48, 64, 65, 66, 112, 113, 128, 130]


@pytest.mark.parametrize("n", EXTENTS)
@pytest.mark.parametrize("dt", ["c64", "cbf16"])
def test_gram_at_tile_edges(n, dt):
    for shape in ((n, 9, 31), (5, n, 21), (7, 19, n), (2, 3, n, 2)):
        print("[case]", shape, dt, flush=True)
        g = synth.small_case(shape, 40 + n, outlier_frac=(1, 50), dtype=dt)
        k = int(np.prod(shape)) // 40
        ctx = make_gpu_ctx(T, shape, [max(1, e // 2) for e in shape], k, refresh_every=0,
                           grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
        ctx.tgrad_refresh_factors(T.to_device_grad(g))
        x = np.array(O.to_complex128(g))
        x.reshape(-1)[ctx.tgrad_get_state(T.STATE_INDICES)] = 0
        for m in range(len(shape)):
            if shape[m] == max(1, shape[m] // 2):
                continue
            a = np.moveaxis(x, m, 0).reshape(shape[m], -1)
            want = a @ a.conj().T
            got = ctx.tgrad_get_state(T.STATE_GRAM0 + m)
            d = np.sqrt(np.real(np.diag(want)))
            # a sum of J products in float64, in whatever order: J 2^-53 times the product of the row norms; the real
            # and imaginary parts are sums of two and of three such sums, on either side
            bound = 8 * a.shape[1] * 2.0 ** -53 * np.outer(d, d)
            assert np.all(np.abs(got - want) <= bound), (shape, m, np.max(np.abs(got - want) / bound))
            assert np.all(np.imag(np.diag(got)) == 0) and np.array_equal(got, got.conj().T)
        ctx.tgrad_destroy()
