"""The kernels whose float32 products run on split bf16 operands, one step or two per shape against the oracle, at the edges
of their operands (16 rows or elements at a time), their tables and the lines between them and the kernels beside them."""
import numpy as np
import pytest

from oracle import tgrad_oracle as O
from paper_2501_02379_amd import synth
from paper_2501_02379_amd import tgrad as T
from helpers import check_parity, run_both, run_both_bf16_weights

pytestmark = pytest.mark.gpu


def _weights(shape, seed):
    rng = np.random.default_rng(seed)
    return (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 0.02


MID_SHAPES = [
    ((96, 140, 20, 9), (4, 70, 20, 9), 900),       # nine quads: two chunks of the table; a rank of five tiles, two launch rows
    ((96, 256, 20, 9), (4, 60, 20, 9), 900),       # sixteen quads; an expansion whose table is cut after eight tiles
    ((96, 128, 20, 9), (4, 16, 20, 9), 900),       # the table of one tile, all of it at once
    ((250, 17, 16, 9), (4, 9, 16, 9), 900),        # one element past the last whole quad
    ((250, 30, 29, 16), (4, 28, 29, 16), 900),     # 3625 groups of column pairs: several for some workgroups
]


@pytest.mark.parametrize("shape,ranks,k", MID_SHAPES)
def test_middle_stages(shape, ranks, k):
    print("[case]", shape, ranks, flush=True)
    grads = [synth.small_case(shape, 700 + t, outlier_frac=(1, 200)) for t in range(2)]
    W0 = _weights(shape, 21).astype(np.complex64)
    info = run_both(T, shape, ranks, k, grads, W0, refresh_every=4, lr=2e-3, weight_decay=0.01)
    assert all(info["omega_equal"])
    check_parity(info, W0)


@pytest.mark.parametrize("shape,ranks,k", [
    ((96, 100, 20, 9), (4, 40, 20, 9), 900),       # 21 items of an expansion's table: a whole batch of the wavefronts and a part
    ((96, 200, 20, 9), (4, 20, 20, 9), 900),       # 26, for eight wavefronts
    ((250, 144, 16, 9), (4, 20, 16, 9), 900),      # ... 18, pairs of columns
    ((250, 70, 16, 16), (4, 20, 16, 16), 900),     # 10 for four: a part of a batch; pairs of columns
    ((96, 128, 20, 9), (4, 32, 20, 9), 900),       # 16: a whole one
    ((96, 64, 20, 9), (4, 20, 20, 9), 900),        # 8: columns first
])
def test_expansion_tables_past_the_first_requests(shape, ranks, k):
    test_middle_stages(shape, ranks, k)


# The core kernel: four wavefronts or eight, tiles of rank, rows in one batch or several, one group of 16 columns or several
# for a workgroup.
CORE_SHAPES = [
    ((20, 40, 40, 12), (7, 40, 40, 12)),           # one tile of rank, four wavefronts; 1200 groups: two for some workgroups
    ((64, 42, 40, 5), (16, 42, 40, 5)),            # ... as many rows as these hold
    ((65, 42, 40, 5), (16, 42, 40, 5)),            # ... eight
    ((140, 16, 16, 15), (16, 16, 16, 15)),         # ... more rows than these hold: 240 groups
    ((140, 16, 16, 17), (16, 16, 16, 17)),         # ... 272 groups: four
    ((100, 30, 20, 9), (50, 30, 20, 9)),           # four tiles, eight wavefronts: operands partly in LDS, 338 groups
    ((200, 24, 20, 9), (64, 24, 20, 9)),           # ... in several batches, fetched again for every group
    ((256, 12, 12, 9), (33, 12, 12, 9)),           # ... the longest
]


@pytest.mark.parametrize("shape,ranks", CORE_SHAPES)
def test_core_kernel(shape, ranks):
    print("[case]", shape, ranks, flush=True)
    grads = [synth.small_case(shape, 800 + t, outlier_frac=(1, 200)) for t in range(2)]
    W0 = _weights(shape, 28).astype(np.complex64)
    info = run_both(T, shape, ranks, 900, grads, W0, refresh_every=4, lr=2e-3, weight_decay=0.01)
    assert all(info["omega_equal"])
    check_parity(info, W0)


# shape, ranks, k, gradient dtype, packed: whether the 32 x 32 kernels (which have a factor packed for them) serve it
END_SHAPES = [
    ((64, 32, 32, 17), (4, 4, 17, 9), 6000, "c64", False),      # 2048 slabs: the first with full ranks
    ((89, 23, 32, 17), (4, 4, 17, 9), 6000, "c64", True),       # ... 2047
    ((46, 45, 40, 33), (4, 4, 20, 12), 9000, "c64", False),     # coefficients in LDS, two tiles in flight, half a tile last
    ((46, 45, 40, 33), (4, 4, 20, 12), 200000, "cbf16", False), # ... more than 64 support entries in a tile
    ((46, 45, 24, 65), (3, 4, 17, 16), 9000, "c64", False),     # 16-row tiles in pairs
    ((46, 45, 40, 65), (3, 4, 17, 16), 9000, "cbf16", False),   # ... three to a slab: the last alone
    ((20, 20, 40, 50), (3, 4, 9, 9), 3000, "c64", False),       # ... a tile per wavefront: never in pairs
    ((33, 32, 24, 42), (3, 4, 9, 6), 3000, "cbf16", False),     # three quads, no remainder
    ((33, 32, 21, 25), (3, 4, 9, 8), 3000, "c64", False),       # two quads, the second of nine elements
    ((13, 10, 250, 34), (3, 4, 20, 10), 9000, "c64", False),    # a table that leaves one workgroup to a compute unit
    ((40, 30, 230, 20), (3, 4, 18, 7), 9000, "c64", False),     # ... with whole slabs: eight wavefronts
    ((10, 10, 250, 34), (3, 4, 20, 10), 9000, "c64", False),    # ... fewer slabs
    ((9, 3, 232, 15), (3, 2, 32, 2), 900, "c64", False),        # ... too few for it: separate kernels
    ((9, 3, 205, 54), (3, 2, 17, 9), 900, "c64", False),        # ... the other line of those
    ((29, 29, 220, 50), (3, 3, 26, 12), 9000, "c64", False),    # four wavefronts per compute unit, 841 slabs: separate kernels
    ((27, 93, 70, 38), (6, 23, 31, 8), 9000, "c64", False),     # five tiles to a slab, 2511: single tiles in the last kernel
    ((20, 128, 70, 38), (6, 23, 31, 9), 9000, "c64", False),    # ... 2560: whole slabs
    ((20, 128, 70, 38), (6, 23, 31, 8), 9000, "c64", False),    # ... up to eight columns of rank single ones
    ((32, 32, 256, 13), (4, 5, 20, 5), 9000, "c64", False),     # 1024 slabs, whole 32-row tiles
]


@pytest.mark.parametrize("shape,ranks,k,dt,packed", END_SHAPES)
def test_end_kernels(shape, ranks, k, dt, packed):
    print("[case]", shape, ranks, dt, flush=True)
    grads = [synth.small_case(shape, 720 + t, outlier_frac=(1, 200), dtype=dt) for t in range(2)]
    W0 = _weights(shape, 22).astype(np.complex64)
    info = run_both(T, shape, ranks, k, grads, W0, refresh_every=4, lr=2e-3, weight_decay=0.01,
                    grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    assert all(info["omega_equal"])
    check_parity(info, W0)
    ctx = info["ctx"]
    ctx.tgrad_set_profiling(True)
    ctx.tgrad_refresh_factors(T.to_device_grad(grads[0]))
    assert ("factor_pack" in ctx.tgrad_get_kernel_times()) == packed


@pytest.mark.parametrize("shape,ranks,k", [(s, r, k) for s, r, k, dt, _ in END_SHAPES if dt == "cbf16"])
def test_end_kernels_bf16_weights(shape, ranks, k):
    """(Bounds as in test_bf16_weights_single_steps.)"""
    print("[case]", shape, ranks, flush=True)
    grads = [synth.small_case(shape, 740 + t, outlier_frac=(1, 200), dtype="cbf16") for t in range(2)]
    info = run_both_bf16_weights(T, shape, ranks, k, grads, O.complex_to_bf16_pairs(_weights(shape, 23)), resync=True,
                                 refresh_every=4, lr=2e-3, weight_decay=0.01, grad_dtype=T.TGRAD_CBF16)
    for worst, frac in info["stats"]:
        assert worst <= 1
        assert frac <= max(5e-3, 2.0 / (2 * int(np.prod(shape))))


# Fewer than 1024 slabs whose last mode has many coefficients: one tile per wavefront while slabs have four tiles at most or
# all of them are resident, coefficients in registers for complex64 beyond that; last kernel: one tile per wavefront up to
# 768 tiles (rank above 8) or 3072.
# shape, ranks, k, gradient dtype
FEW_TILES = [
    ((11, 9, 29), (4, 2, 9), 60, "c64"),                    # one tile of nine rows
    ((40, 33, 22), (6, 32, 10), 800, "cbf16"),              # 32 + 1 rows, two tiles of rank each
    ((9, 10, 37), (4, 2, 16), 90, "cbf16"),                 # 16-row tiles, one to a slab
    ((12, 17, 34), (5, 16, 9), 200, "c64"),                 # 16 + 1 rows: an even tile and an odd one, padded rows
    ((7, 64, 52), (3, 17, 8), 500, "c64"),                  # four tiles, three quads and a remainder step
    ((7, 65, 68), (3, 9, 16), 500, "cbf16"),                # ... five, the last of one row
    ((6, 128, 53), (3, 32, 5), 900, "c64"),                 # ... eight
    ((6, 129, 53), (3, 20, 5), 900, "c64"),                 # ... nine: one more than that takes
    ((9, 150, 26), (3, 20, 12), 900, "c64"),                # five tiles of 32 rows (9 x 26 > 150: a Gram matrix of full rank)
    ((31, 33, 20, 33), (4, 5, 7, 12), 3000, "c64"),         # 1023 slabs of one tile
    ((32, 32, 20, 33), (4, 5, 7, 12), 3000, "c64"),         # 1024: whole slabs
    ((24, 32, 12, 44), (4, 5, 5, 9), 3000, "cbf16"),        # 768 tiles for the last kernel
    ((27, 29, 12, 44), (4, 5, 5, 9), 3000, "cbf16"),        # ... 783
    ((24, 32, 60, 34), (4, 5, 9, 6), 9000, "c64"),          # 3072 tiles, rank 6
    ((25, 31, 60, 34), (4, 5, 9, 6), 9000, "c64"),          # ... 3100
    ((19, 20, 86, 61), (4, 5, 19, 5), 9000, "c64"),         # 380 slabs of six tiles: coefficients in registers, shared slabs
    ((21, 21, 97, 53), (5, 5, 7, 11), 9000, "c64"),         # ... of seven, one tile of rank
    ((17, 18, 82, 36), (4, 4, 6, 9), 9000, "c64"),          # ... no remainder
    ((13, 30, 118, 30), (3, 7, 23, 5), 9000, "c64"),        # the class whose table alone leaves one workgroup to a compute unit
    ((13, 30, 118, 30), (3, 7, 23, 5), 9000, "cbf16"),      # ... in bf16 there is room
]


@pytest.mark.parametrize("shape,ranks,k,dt", FEW_TILES)
def test_few_tiles_of_many_coefficients(shape, ranks, k, dt):
    print("[case]", shape, ranks, dt, flush=True)
    grads = [synth.small_case(shape, 780 + t, outlier_frac=(1, 200), dtype=dt) for t in range(2)]
    W0 = _weights(shape, 26).astype(np.complex64)
    info = run_both(T, shape, ranks, k, grads, W0, refresh_every=4, lr=2e-3, weight_decay=0.01,
                    grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    assert all(info["omega_equal"])
    check_parity(info, W0)


@pytest.mark.parametrize("shape,ranks,k", [(s, r, k) for s, r, k, dt in FEW_TILES if dt == "cbf16"])
def test_few_tiles_bf16_weights(shape, ranks, k):
    """(Bounds as in test_bf16_weights_single_steps.)"""
    print("[case]", shape, ranks, flush=True)
    grads = [synth.small_case(shape, 790 + t, outlier_frac=(1, 200), dtype="cbf16") for t in range(2)]
    info = run_both_bf16_weights(T, shape, ranks, k, grads, O.complex_to_bf16_pairs(_weights(shape, 27)), resync=True,
                                 refresh_every=4, lr=2e-3, weight_decay=0.01, grad_dtype=T.TGRAD_CBF16)
    for worst, frac in info["stats"]:
        assert worst <= 1
        assert frac <= max(5e-3, 2.0 / (2 * int(np.prod(shape))))


# Slabs of five to eight tiles, fewer than 1024 of them but more than the chip has places for: a workgroup of the first kernel
# stays for several of them (bf16 gradients, or a table too large for two workgroups).  Rows of an even number of elements are
# padded in LDS, and what lies there meets zero coefficients: it has to be a finite number in the gradient's type, after the
# wavefronts have exchanged their sums through the same place too.
# shape, ranks, k, gradient dtype, order
SHARED_SLABS = [
    ((28, 28, 80, 64), (6, 6, 16, 16), 9000, "cbf16", T.TGRAD_ORDER_US_LR),
    ((43, 16, 99, 50), (14, 5, 32, 16), 9000, "cbf16", T.TGRAD_ORDER_US_LR),
    ((43, 16, 99, 49), (14, 5, 32, 16), 9000, "cbf16", T.TGRAD_ORDER_US_LR),     # nothing to pad
    ((24, 23, 114, 54), (6, 5, 32, 9), 9000, "c64", T.TGRAD_ORDER_US_LR),
    ((31, 31, 141, 38), (7, 7, 24, 6), 9000, "cbf16", T.TGRAD_ORDER_US_LR),      # coefficients in registers
    ((30, 30, 80, 48), (8, 8, 12, 12), 9000, "cbf16", T.TGRAD_ORDER_US_LR),
    ((30, 30, 80, 48), (8, 8, 12, 12), 9000, "cbf16", T.TGRAD_ORDER_SUM),
    ((24, 24, 136, 32), (6, 6, 20, 9), 9000, "cbf16", T.TGRAD_ORDER_US_LR),      # 32-row tiles, a remainder step past the end
    ((24, 24, 136, 32), (6, 6, 20, 9), 9000, "cbf16", T.TGRAD_ORDER_LR_US),
    ((24, 24, 136, 26), (6, 6, 20, 12), 9000, "cbf16", T.TGRAD_ORDER_US_LR),     # ... two quads and no remainder
]


def _head_lds(K, r, I2, r2, elem_dwords):
    """LDS bytes of a workgroup of the first kernel for shared slabs (coefficients, staging slices, table of conj(U))."""
    steps = next(t for t in (3, 5, 7, 9, 13, 17) if t >= (K + 3) // 4)
    quads = steps // 4 + (steps % 4 >= 2)
    rows, pieces = (32, steps) if steps <= 9 else (16, (steps + 1) // 2)
    pad = 1 - K % 2
    elems = max(pieces * 128 + pad * (pieces * 128 // K + 1), rows * (K + pad)) + 16 * quads + 4
    piece_slice = 4 * (-(-max(elem_dwords * elems, 1024) // 4) * 4)
    fixed = (quads * 2 * 3072 if r > 8 else 0) + -(-I2 // 32) * (1 if r2 <= 16 else 2) * 6144
    lds = lambda W: fixed + W * piece_slice
    most = 4 if lds(4) <= 80 * 1024 or lds(8) > 160 * 1024 else 8
    return lds(min(most, -(-I2 // rows)))


@pytest.mark.parametrize("shape,ranks,k,dt,order", SHARED_SLABS)
def test_workgroups_that_stay_for_several_slabs(shape, ranks, k, dt, order):
    import torch
    print("[case]", shape, ranks, dt, order, flush=True)
    places = (160 * 1024) // _head_lds(shape[3], ranks[3], shape[2], ranks[2], 1 if dt == "cbf16" else 2)
    units = torch.cuda.get_device_properties(0).multi_processor_count
    assert shape[0] * shape[1] > max(places, 2) * units          # (2: the most that one tile per wavefront gets in)
    grads = [synth.small_case(shape, 760 + t, outlier_frac=(1, 200), dtype=dt) for t in range(2)]
    W0 = _weights(shape, 25).astype(np.complex64)
    info = run_both(T, shape, ranks, k, grads, W0, refresh_every=4, lr=2e-3, weight_decay=0.01, order=order,
                    grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64)
    assert all(info["omega_equal"])
    check_parity(info, W0)


# Every kernel whose operands are split, in its variants: first and last kernel with coefficients in registers, in LDS, for one
# tile, for shared slabs; compressions and expansions of one, two and four tiles, with one column per lane and two; the core
# kernel of one, two and four tiles on four wavefronts and eight.
EXACT_SHAPES = [
    ((24, 20, 40, 33), (4, 5, 9, 8), "c64"),
    ((42, 42, 44), (13, 13, 14), "c64"),                   # one tile per wavefront; core (1, 4)
    ((19, 20, 86, 61), (4, 5, 19, 5), "c64"),              # shared slabs, registers
    ((28, 28, 80, 64), (6, 6, 16, 16), "cbf16"),           # ... LDS
    ((48, 44, 40, 34), (30, 20, 20, 12), "c64"),           # whole slabs, LDS; core (2, 4)
    ((48, 44, 40, 34), (12, 20, 20, 12), "cbf16"),
    ((110, 60, 40, 16), (12, 50, 30, 15), "c64"),          # compression and expansion of four tiles, one column; core (1, 8)
    ((96, 80, 40, 16), (40, 24, 30, 14), "c64"),           # ... of two, two columns; core (4, 8)
    ((100, 96, 20, 16), (20, 12, 18, 14), "c64"),          # ... of one; core (2, 8)
    ((64, 140, 20, 10), (44, 70, 18, 8), "c64"),           # expansion of more rows than registers hold; core (4, 4)
]


@pytest.mark.parametrize("shape,ranks,dt", EXACT_SHAPES)
def test_selecting_factors_are_exact(shape, ranks, dt):
    """Factors of one unit entry (1, i, -1 or -i) per column select entries of G: every product is exact, so is the core
    gradient, bit for bit, up to the largest float32 (whose nearest bf16 is infinite).  The way back multiplies each entry of
    N once: 16 roundings of 2^-24 are more than AdamUpdate and the products make, and where the third part of an operand is
    lost 2^-17 remain."""
    print("[case]", shape, ranks, dt, flush=True)
    rng = np.random.default_rng(29)
    bits = rng.integers(0, 1 << 24, shape + (2,), dtype=np.uint32)                  # sign and 23 bits of mantissa
    expo = rng.integers(-100, 128, shape + (2,)).astype(np.int64) + 127
    g = (((bits >> np.uint32(23)) << np.uint32(31)) | (expo.astype(np.uint32) << np.uint32(23)) |
         (bits & np.uint32(0x7FFFFF))).view(np.float32)
    if dt == "cbf16":
        g = (g.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)
    g = g.reshape(-1).view(np.complex64).reshape(shape)
    g.reshape(-1)[:4] = np.finfo(np.float32).max * np.complex64(1 - 1j) if dt == "c64" else 1.0
    lr, eps, tau = 1e-3, 1e-8, 4
    ctx = T.Context(T.make_config(shape, ranks, 1, lr=lr, eps=eps, refresh_every=0,
                                  grad_dtype=T.TGRAD_CBF16 if dt == "cbf16" else T.TGRAD_C64))
    ctx.tgrad_set_state(T.STATE_STEP, tau - 1)
    ctx.tgrad_set_state(T.STATE_INDICES, np.zeros(1, np.int64))
    rows, phases = [], []
    for n, (i, r) in enumerate(zip(shape, ranks)):
        # (row 0 of the last mode's neighbours of the support is among the selected ones)
        rows.append(np.concatenate([[0], 1 + rng.permutation(i - 1)[:r - 1]]) if n < len(shape) - 1 else
                    np.concatenate([[1, 2, 3], 4 + rng.permutation(i - 4)[:r - 3]]))
        phases.append(np.array([1, 1j, -1, -1j], np.complex64)[rng.integers(0, 4, r)])
        u = np.zeros((i, r), np.complex64)
        u[rows[n], np.arange(r)] = phases[n]
        ctx.tgrad_set_state(T.STATE_FACTOR0 + n, u)
    gd = g if dt == "c64" else O.complex_to_bf16_pairs(g)
    W = T.to_device_weight(np.zeros(shape, np.complex64))
    ctx.tgrad_step(W, T.to_device_grad(gd))
    phase = phases[0]
    for p in phases[1:]:
        phase = np.multiply.outer(phase, p)
    want = g[np.ix_(*rows)] * phase.conj()
    assert np.array_equal(ctx.tgrad_get_state(T.STATE_CORE_G), want)
    m, v = ctx.tgrad_get_state(T.STATE_CORE_M), ctx.tgrad_get_state(T.STATE_CORE_V)
    with np.errstate(over="ignore"):
        d = 1.0 / (np.sqrt(np.float32(1 / (1 - float(np.float32(0.999)) ** tau)) * v) + np.float32(eps)).astype(np.float64)
    N = m.astype(np.complex128) / (1 - float(np.float32(0.9)) ** tau) * d * phase
    got = T.weight_to_host(W).astype(np.complex128)
    back = got[np.ix_(*rows)]
    for a, b in ((back.real, N.real), (back.imag, N.imag)):
        worst = np.max(np.abs(a + float(np.float32(lr)) * b) / (float(np.float32(lr)) * np.abs(b) + 1e-30))
        print("way back: %.2e" % worst, flush=True)
        assert worst < 16 * 2.0 ** -24
    got[np.ix_(*rows)] = 0
    got.reshape(-1)[0] = 0
    assert not got.any()
    ctx.tgrad_destroy()


def test_products_keep_float32_accuracy():
    """A step's core gradient at entries of G between 2^-60 and 2^60, against 64 bits: every part of a float32 counts, so the
    error stays that of float32 sums (16 roundings of 2^-24 at the depth of these chains), where two parts of three would
    leave 2^-17."""
    shape, ranks = (24, 20, 40, 33), (4, 5, 9, 8)
    rng = np.random.default_rng(24)
    for scale in (2.0 ** -60, 1.0, 2.0 ** 60):
        g = ((rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * scale).astype(np.complex64)
        ctx = T.Context(T.make_config(shape, ranks, 1, lr=1e-3, refresh_every=0), device="cuda:0")
        ctx.tgrad_set_state(T.STATE_STEP, 3)
        ctx.tgrad_set_state(T.STATE_INDICES, np.zeros(1, np.int32))
        us = []
        for n, (i, r) in enumerate(zip(shape, ranks)):
            u = np.linalg.qr(rng.standard_normal((i, r)) + 1j * rng.standard_normal((i, r)))[0].astype(np.complex64)
            ctx.tgrad_set_state(T.STATE_FACTOR0 + n, u)
            us.append(u.astype(np.complex128))
        ctx.tgrad_step(T.to_device_weight(np.zeros(shape, np.complex64)), T.to_device_grad(g))
        x = g.astype(np.complex128)
        x.reshape(-1)[0] = 0
        for n, u in enumerate(us):
            x = np.moveaxis(np.tensordot(u.conj(), x, axes=([0], [n])), 0, n)
        m = ctx.tgrad_get_state(T.STATE_CORE_M).reshape(ranks).astype(np.complex128) / float(np.float32(1) - np.float32(0.9))
        err = np.linalg.norm(m - x) / np.linalg.norm(x)
        print("scale %g error %.2e" % (scale, err), flush=True)
        assert err < 16 * 2.0 ** -24
        ctx.tgrad_destroy()
