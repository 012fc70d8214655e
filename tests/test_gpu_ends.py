"""The first and last kernel of a step on 16 x 16 tiles (modes N-1 and N in one pass, any extent of mode N-1):
one step per shape against the oracle, at the edges of its tiles and of its size classes."""
import numpy as np
import pytest

from oracle import tgrad_oracle as O
from paper_2501_02379_amd import synth
from paper_2501_02379_amd import tgrad as T
from helpers import check_parity, run_both, run_both_bf16_weights

pytestmark = pytest.mark.gpu

# shape, ranks, k, gradient dtype
SHAPES = [
    ((5, 7, 13, 5), (3, 4, 5, 2), 200, "c64"),          # odd slabs: tiles that start off a 16-byte boundary
    ((6, 9, 4, 7), (3, 4, 1, 3), 40, "c64"),            # the shortest slabs they take
    ((6, 9, 3, 7), (3, 4, 3, 3), 40, "c64"),            # ... and one row less
    ((11, 6, 16, 2), (3, 4, 16, 2), 40, "c64"),         # shortest rows, a full tile of rows, full ranks
    ((9, 8, 33, 33), (3, 4, 17, 9), 700, "c64"),        # two tiles (32 + 1 rows), lone last column, two tiles of each rank
    ((9, 8, 48, 34), (3, 4, 16, 8), 500, "c64"),        # 16-row tiles from here on, padded rows
    ((4, 5, 21, 65), (3, 4, 9, 16), 300, "c64"),        # 16 + 5 rows, lone last column
    ((4, 3, 70, 68), (3, 3, 32, 16), 900, "c64"),       # longest rows, five tiles shared by four wavefronts
    ((40, 30, 35, 9), (4, 5, 6, 8), 3000, "c64"),       # slabs enough for whole ones per wavefront, two tiles each
    ((36, 31, 5, 4), (4, 5, 2, 3), 5500, "c64"),        # ... of five rows; support entries everywhere
    ((5, 7, 13, 5), (3, 4, 5, 2), 2000, "cbf16"),       # odd slabs of 4-byte elements, most entries in the support
    ((37, 29, 19, 21), (4, 5, 7, 6), 2000, "cbf16"),
    ((50, 33, 24), (12, 20, 7), 300, "c64"),            # three-way: one slab per leading index
    ((4, 3, 5, 6, 11), (2, 2, 3, 4, 5), 90, "c64"),     # five-way
]


@pytest.mark.parametrize("shape,ranks,k,dt", SHAPES)
def test_end_kernels_small_tiles(shape, ranks, k, dt):
    print("[case]", shape, ranks, k, dt, flush=True)
    grads = [synth.small_case(shape, 300 + t, outlier_frac=(1, 100), dtype=dt) for t in range(4)]
    rng = np.random.default_rng(5)
    W0 = ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02).astype(np.complex64)
    info = run_both(T, shape, ranks, k, grads, W0, refresh_every=3, lr=2e-3, weight_decay=0.01,
                    grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    assert all(info["omega_equal"])
    check_parity(info, W0)


@pytest.mark.parametrize("shape,ranks,k,dt", [SHAPES[0], SHAPES[4], SHAPES[6], SHAPES[10], SHAPES[11]])
def test_end_kernels_bf16_weights(shape, ranks, k, dt):
    """Four-element pieces of W: tiles that start and end inside a piece (bounds as in test_bf16_weights_single_steps)."""
    print("[case]", shape, ranks, k, dt, flush=True)
    grads = [synth.small_case(shape, 400 + t, outlier_frac=(1, 100), dtype=dt) for t in range(4)]
    rng = np.random.default_rng(6)
    W0 = O.complex_to_bf16_pairs((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02)
    info = run_both_bf16_weights(T, shape, ranks, k, grads, W0, resync=True, refresh_every=3, lr=2e-3,
                                 weight_decay=0.01, grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    for worst, frac in info["stats"]:
        assert worst <= 1
        assert frac <= max(5e-3, 2.0 / (2 * int(np.prod(shape))))


# shape, ranks: slabs that two or four wavefronts of the last kernel walk together, more of them than it has wavefronts for at a
# time (2 to 4 workgroups of 4 a compute unit), in numbers that do not divide the grid; the last tile of every slab is a partial one
SHARED_SLABS = [
    ((46, 46, 126, 20), (3, 4, 5, 6)),                  # four wavefronts, four tiles of 32 rows
    ((46, 45, 115, 33), (3, 4, 16, 8)),                 # ... lone last column
    ((46, 46, 61, 40), (3, 4, 9, 12)),                  # ... tiles of 16 rows, two operands of the last rank
    ((51, 51, 125, 34), (3, 4, 6, 10)),                 # ... eight tiles
    ((46, 46, 63, 20), (3, 4, 5, 6)),                   # two wavefronts, two tiles
    ((46, 46, 63, 34), (3, 4, 20, 8)),                  # ... four tiles, two operands of mode N-1's rank
    ((51, 51, 95, 34), (3, 4, 20, 10)),                 # ... six tiles
    ((34, 33, 39, 19), (3, 4, 16, 11)),                 # ... 561 workgroups: not whole rounds of the eight XCDs
    ((34, 32, 39, 19), (3, 4, 16, 11)),                 # ... 544: whole ones
    ((51, 51, 39, 19), (3, 4, 16, 11)),                 # a wavefront for every slab again: 2601 of two tiles
    ((60, 60, 43, 18), (3, 4, 5, 6)),                   # ... 3600, a second tile of 11 rows
    ((60, 60, 44, 18), (3, 4, 5, 6)),                   # two again: of 12
    ((37, 37, 115, 19), (3, 4, 30, 7)),                 # ... ranks of 17 and more, 1369 slabs
]


@pytest.mark.parametrize("shape,ranks", SHARED_SLABS)
def test_slabs_walked_by_several_wavefronts(shape, ranks):
    print("[case] shared slabs", shape, ranks, flush=True)
    grads = [synth.small_case(shape, 320 + t, outlier_frac=(1, 100)) for t in range(2)]
    rng = np.random.default_rng(8)
    W0 = ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02).astype(np.complex64)
    info = run_both(T, shape, ranks, int(np.prod(shape)) // 40, grads, W0, refresh_every=3, lr=2e-3, weight_decay=0.01)
    assert all(info["omega_equal"])
    check_parity(info, W0)


# shape, ranks, fused: modes N-1 and N in one pass (False: separate kernels, 8192 slabs or more of few rows)
SHORT_SLABS = [
    ((91, 90, 4, 5), (9, 8, 2, 2), True),               # 8190 slabs
    ((91, 91, 4, 5), (9, 8, 2, 2), False),              # 8281
    ((128, 64, 8, 5), (9, 8, 3, 2), False),             # 8192, one tile in four filled
    ((128, 64, 16, 5), (9, 8, 3, 2), True),             # ... half filled
    ((128, 128, 9, 3), (9, 8, 3, 2), False),            # 16384: the further line
    ((128, 128, 9, 9), (9, 8, 3, 9), True),             # ... a full last rank: its result is as long as the row
    ((40, 30, 9, 36, 2), (4, 5, 3, 18, 1), False),      # 10800 slabs of one tile and four rows, two tiles of rank
    ((32, 16, 16, 32, 3), (4, 5, 3, 18, 1), True),      # 8192 slabs of one whole tile
]


@pytest.mark.parametrize("shape,ranks,fused", SHORT_SLABS)
def test_short_slabs_in_large_numbers(shape, ranks, fused):
    """Both sides of the line from which on short slabs are left to separate kernels; launches and values."""
    print("[case]", shape, ranks, fused, flush=True)
    grads = [synth.small_case(shape, 350 + t, outlier_frac=(1, 100)) for t in range(2)]
    rng = np.random.default_rng(7)
    W0 = ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02).astype(np.complex64)
    info = run_both(T, shape, ranks, int(np.prod(shape)) // 50, grads, W0, refresh_every=5, lr=2e-3, weight_decay=0.01)
    assert all(info["omega_equal"])
    check_parity(info, W0)
    ctx = info["ctx"]
    ctx.tgrad_set_profiling(True)
    ctx.tgrad_step(T.to_device_weight(W0), T.to_device_grad(grads[0]))
    times = ctx.tgrad_get_kernel_times()
    between = len(shape) - 2 - (1 if fused else 0)       # stages between the first kernel and the core kernel, each way
    if shape[0] * shape[1] <= 1600:                      # (small leading modes: two of them inside the core kernel)
        between -= 1
    assert times["project"]["launches"] == between and times["backproject"]["launches"] == between
