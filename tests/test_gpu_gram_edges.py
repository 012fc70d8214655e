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


# shape, mode: every chunk of tensor columns is four staged tiles or more (a tile is 256 / RT columns), the last tile
# ragged; columns behind the mode (B) far above, just above and below a tile, and none
LOOP_CASES = [
    ((17, 457, 431), 0), ((767, 17, 257), 1), ((199, 32, 17, 31), 2), ((457, 431, 17), 2),
    ((33, 331, 298), 0), ((763, 33, 129), 1), ((199, 17, 33, 30), 2), ((331, 298, 33), 2),
    ((65, 223, 221), 0), ((757, 65, 65), 1), ((83, 41, 65, 15), 2), ((223, 221, 65), 2),
    ((66, 157, 157), 0), ((745, 66, 33), 1), ((59, 60, 66, 7), 2),
    ((157, 112, 157), 1), ((113, 157, 157), 0), ((157, 157, 113), 2),
    ((128, 157, 157), 0), ((797, 128, 31), 1), ((157, 157, 128), 2),
]


def _whole_numbers(shape, seed, dt):
    """A gradient of whole numbers: every product and every sum of its Gram matrices is exact in float64, in any order."""
    rng = np.random.default_rng(seed)
    g = (rng.integers(-7, 8, shape) + 1j * rng.integers(-7, 8, shape)).astype(np.complex64)
    return O.complex_to_bf16_pairs(g) if dt == "cbf16" else g


def _check_exact(shape, ranks, k, dt, seed):
    g = _whole_numbers(shape, seed, dt)
    ctx = make_gpu_ctx(T, shape, ranks, k, refresh_every=0, grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    ctx.tgrad_refresh_factors(T.to_device_grad(g))
    x = np.array(O.to_complex128(g))
    om = ctx.tgrad_get_state(T.STATE_INDICES)
    assert np.array_equal(om, O.sparse_indices(g, k))
    x.reshape(-1)[om] = 0
    for m in range(len(shape)):
        if ranks[m] < shape[m]:
            a = np.moveaxis(x, m, 0).reshape(shape[m], -1)
            assert np.array_equal(ctx.tgrad_get_state(T.STATE_GRAM0 + m), a @ a.conj().T), (shape, m)
    ctx.tgrad_destroy()


@pytest.mark.parametrize("shape,mode", LOOP_CASES)
def test_gram_over_several_tiles_of_a_chunk(shape, mode):
    """The steady state of the kernel's loop (one tile multiplied, one committed, one fetched), one mode compressed."""
    dt = "cbf16" if (shape[mode] + mode) % 2 else "c64"
    print("[case]", shape, mode, dt, flush=True)
    ranks = [max(1, e // 4) if m == mode else e for m, e in enumerate(shape)]
    _check_exact(shape, ranks, int(np.prod(shape)) // 30, dt, 60 + mode)


@pytest.mark.parametrize("shape", [(128, 13, 31, 29), (17, 66, 34, 33), (10, 11, 12, 9, 113)])
def test_gram_of_several_modes_over_several_tiles(shape):
    print("[case]", shape, flush=True)
    _check_exact(shape, [max(1, e // 4) for e in shape], int(np.prod(shape)) // 30, "c64", 70)
